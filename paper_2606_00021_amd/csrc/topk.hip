// Per-query top-k of the similarity scores (Sec. 3.1 Eq. 3: the retriever
// returns the N most relevant continuations; Sec. 3.2 Eq. 7 "top-N'") and
// the gather of each hit's continuation into the draft batch (the (k_i, s_i)
// pairs of Sec. 3.2).
//
// Order: score descending, then row index ascending.  Each (score, row) pair
// is packed into one unique 64-bit key (order-preserving score bits in the
// high word, the complemented row in the low word), so "top-k" is "the k
// largest keys" and ties need no special handling.
//
// Selection is hierarchical.  A block of 512 threads takes a chunk of 8192
// keys into registers (16 per thread; a single chunk of at most 4096 keys
// takes 8 per thread, since every phase costs its per-thread key loop).
// The block is one compute unit, so every per-key instruction counts.  One
// reduction gives the number of real (non-padding) keys and the AND and OR
// of them: the bits above the highest bit where they differ are shared by
// all, so the radix select starts right below them (survivors of a level
// share their sign and most of their exponent, which a fixed top-down start
// would spend a whole pass on).  For a chunk of raw scores the AND and OR
// come from the score words alone, the row words being a contiguous range.
// A chunk of raw scores holds both signs, so the first level also bounds the
// k-th largest key from below by the smallest of k or more group maxima and
// starts below the bits that this bound and the largest key share: every
// key of the top k lies between them.  Each pass builds a 256-bin LDS
// histogram of the next 8-bit digit among the keys that still match the
// chosen prefix, then one wave totals the waves' histograms and finds the
// digit holding the k-th key with a suffix scan; the loop stops as soon as
// that digit's bucket is taken whole.  The taken keys are compacted by ballot prefix sums (no atomics).
// The k survivors of every chunk form the next level's input until one
// chunk remains; its keys are put in order by rank (each key counts the
// keys above it, all reads LDS broadcasts) and written out together with
// the gathered continuations.
#include "internal.h"
#include "topk_device.h"

namespace sense {
namespace {

constexpr int kThreads = 512;

constexpr int kWaves = kThreads / 64;
constexpr int kPer = kSelectChunk / kThreads;   // keys per thread

// One block per (chunk, query).  FROM_SCORES: input is the fp32 score matrix
// (nq x count, row index = position); otherwise packed keys (nq x count).
// FINAL: exactly one chunk per query; writes sorted ids/scores and drafts.
// P keys per thread: chunks of kThreads * P keys (kSelectChunk for P = 16;
// a smaller P serves a single chunk of fewer keys with less work).
template <bool FROM_SCORES, bool FINAL, int P>
__global__ __launch_bounds__(kThreads) void select_kernel(
    const float* __restrict__ scores, const uint64_t* __restrict__ in_keys, int64_t count,
    int k, uint64_t* __restrict__ out_keys, int64_t* __restrict__ out_ids,
    float* __restrict__ out_scores, int32_t* __restrict__ out_drafts,
    int32_t* __restrict__ out_draft_len, const int32_t* __restrict__ spans,
    const int32_t* __restrict__ span_len, int max_span, int64_t span_stride) {
    __shared__ uint64_t s_sel[kMaxK];
    __shared__ uint64_t s_sorted[FINAL ? kMaxK : 1];
    __shared__ __align__(16) uint32_t s_hist[kWaves * 256];   // read 16 bytes at a time
    __shared__ uint32_t s_info[4];
    __shared__ uint32_t s_nzw[kWaves], s_wc[kWaves];
    __shared__ uint64_t s_andw[kWaves], s_orw[kWaves];
    __shared__ uint32_t s_loww[kWaves], s_highw[kWaves];

    constexpr int CH = kThreads * P;
    const int tid = threadIdx.x;
    const int q = blockIdx.y;
    const int64_t start = (int64_t)blockIdx.x * CH;
    const int64_t remain = count - start;
    const int len = (int)(remain < CH ? remain : CH);
    const int kk = k < CH ? k : CH;

    // Key i of the chunk is held by thread i % kThreads; slots past the chunk
    // hold the padding key 0.  Scores are loaded unconditionally (positions
    // past the chunk re-read its last one, a chunk is never empty here) so
    // that all loads are in flight at once: a load under a branch makes the
    // thread wait for it before issuing the next.
    // The group-maxima bound pays where a chunk holds raw scores of both
    // signs (its keys share no leading bits), first levels and single-chunk
    // finals alike; later levels hold survivors that already share them.
    constexpr bool kBound = FROM_SCORES;
    const StatsLds lds{s_nzw, s_andw, s_orw, s_loww, s_highw};
    uint64_t key[P];
    ChunkStats cs;
    if constexpr (FROM_SCORES) {
        const float* src = scores + (int64_t)q * count + start;
        const int last = len > 0 ? len - 1 : 0;
        float sv[P];
#pragma unroll
        for (int e = 0; e < P; ++e) {
            const int i = tid + e * kThreads;
            sv[e] = src[i < len ? i : last];
        }
        uint32_t sw[P];
#pragma unroll
        for (int e = 0; e < P; ++e) {
            const int i = tid + e * kThreads;
            sw[e] = score_key(sv[e]);
            key[e] = i < len ? (((uint64_t)sw[e] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)(start + i)))
                             : 0ull;
        }
        cs = score_stats<kThreads, P>(sw, key, kk, start, len, lds);
    } else {
#pragma unroll
        for (int e = 0; e < P; ++e) {
            const int i = tid + e * kThreads;
            key[e] = i < len ? in_keys[(int64_t)q * count + start + i] : 0;
        }
        cs = chunk_stats<kThreads, P, kBound>(key, kk, lds);
    }

    // Keys taken: every real (non-zero) one if there are no more than kk,
    // else the kk largest (then more than kk keys are real, as the radix
    // select needs); both as (key & mask) >= prefix.
    SelectState st{1ull, ~0ull};
    const bool all = cs.nz <= (uint32_t)kk;
    if (!all) st = radix_select<kThreads, P, kBound>(key, kk, cs, s_hist, s_info);

    if constexpr (!FINAL) {
        uint64_t* out = out_keys + ((int64_t)q * gridDim.x + blockIdx.x) * kk;
        const uint32_t tot = compact_taken<kThreads, P>(key, st.mask, st.prefix, out, kk, s_wc);
        const int nt = (int)tot < kk ? (int)tot : kk;
        for (int i = nt + tid; i < kk; i += kThreads) out[i] = 0;  // padding key
    } else {
        const uint32_t tot = compact_taken<kThreads, P>(key, st.mask, st.prefix, s_sel, kk, s_wc);
        const int nt = (int)tot < kk ? (int)tot : kk;
        final_output<kThreads>(s_sel, s_sorted, nt, k, q, out_ids, out_scores, out_drafts,
                               out_draft_len, spans, span_len, max_span, span_stride);
    }
}

// One block per query over a key list whose length is a per-query count on
// the device (candidate buffers: most of the capacity is unused): rounds of
// kStreamThreads * P keys, each holding the running top k and the next new
// keys, reduced to the top k by the same radix select; then the final
// output.  P (keys per thread) is chosen per query from its count, so a short
// list is walked with less work; a count that fits one round of the largest
// P is one round, and any count is exact.
constexpr int kStreamThreads = 1024;
constexpr int kStreamPer = kPer;                       // the largest P

struct StreamLds {
    uint32_t* s_hist;
    uint32_t* s_info;
    uint32_t* s_nzw;
    uint32_t* s_wc;
    uint64_t* s_andw;
    uint64_t* s_orw;
};

template <int P>
__device__ int stream_rounds(const uint64_t* __restrict__ src, int64_t count, int64_t cnt_q,
                             int kk, uint64_t* s_sel, const StreamLds& L) {
    constexpr int R = kStreamThreads * P;              // keys per round
    const int tid = threadIdx.x;
    int nt = 0;                                        // running top keys in s_sel
    int64_t pos = 0;
    do {
        const int64_t left = cnt_q - pos;
        const int take = (int)((R - nt) < left ? (R - nt) : left);
        // New keys on clamped positions (no branch around a load), the
        // running ones from LDS.
        uint64_t key[P];
#pragma unroll
        for (int e = 0; e < P; ++e) {
            const int i = tid + e * kStreamThreads;
            const int64_t j = pos + (i - nt);
            const int64_t jc = j < 0 ? 0 : (j < count ? j : count - 1);
            key[e] = src[jc];
        }
#pragma unroll
        for (int e = 0; e < P; ++e) {
            const int i = tid + e * kStreamThreads;
            if (i < nt) key[e] = s_sel[i];
            else if (i - nt >= take) key[e] = 0;
        }
        __syncthreads();                               // s_sel read before it is rewritten
        const ChunkStats cs = chunk_stats<kStreamThreads, P, false>(
            key, kk, StatsLds{L.s_nzw, L.s_andw, L.s_orw, nullptr, nullptr});
        SelectState st{1ull, ~0ull};                   // all real keys, as above
        const bool all = cs.nz <= (uint32_t)kk;
        if (!all)
            st = radix_select<kStreamThreads, P, false>(key, kk, cs, L.s_hist, L.s_info);
        const uint32_t tot =
            compact_taken<kStreamThreads, P>(key, st.mask, st.prefix, s_sel, kk, L.s_wc);
        nt = (int)tot < kk ? (int)tot : kk;
        pos += take;
        __syncthreads();                               // s_sel complete for the next round
    } while (pos < cnt_q);
    return nt;
}

__global__ __launch_bounds__(kStreamThreads) void select_stream_kernel(
    const uint64_t* __restrict__ in_keys, int64_t count, int k,
    const int32_t* __restrict__ dev_count, int64_t* __restrict__ out_ids,
    float* __restrict__ out_scores, int32_t* __restrict__ out_drafts,
    int32_t* __restrict__ out_draft_len, const int32_t* __restrict__ spans,
    const int32_t* __restrict__ span_len, int max_span, int64_t span_stride) {
    constexpr int W = kStreamThreads / 64;
    __shared__ uint64_t s_sel[kMaxK];
    __shared__ uint64_t s_sorted[kMaxK];
    __shared__ __align__(16) uint32_t s_hist[W * 256];        // read 16 bytes at a time
    __shared__ uint32_t s_info[4];
    __shared__ uint32_t s_nzw[W], s_wc[W];
    __shared__ uint64_t s_andw[W], s_orw[W];
    const StreamLds L{s_hist, s_info, s_nzw, s_wc, s_andw, s_orw};
    const int q = blockIdx.x;
    const int kk = k;                                  // k <= kMaxK < kStreamThreads * 4
    int64_t cnt_q = dev_count ? (int64_t)dev_count[q] : count;
    cnt_q = cnt_q < 0 ? 0 : (cnt_q > count ? count : cnt_q);
    const uint64_t* src = in_keys + (int64_t)q * count;
    // The branch is uniform over the block.
    int nt;
    if (cnt_q <= (int64_t)kStreamThreads * 4)
        nt = stream_rounds<4>(src, count, cnt_q, kk, s_sel, L);
    else if (cnt_q <= (int64_t)kStreamThreads * 8)
        nt = stream_rounds<8>(src, count, cnt_q, kk, s_sel, L);
    else
        nt = stream_rounds<kStreamPer>(src, count, cnt_q, kk, s_sel, L);
    final_output<kStreamThreads>(s_sel, s_sorted, nt, k, q, out_ids, out_scores, out_drafts,
                                 out_draft_len, spans, span_len, max_span, span_stride);
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The final level over one chunk of keys (count <= kSelectChunk): eight
// keys per thread when they fit.
void launch_final_keys(const uint64_t* keys, int64_t count, int nq, int k, const int32_t* spans,
                       const int32_t* span_len, int max_span, int64_t span_stride,
                       int64_t* out_ids, float* out_scores, int32_t* out_drafts,
                       int32_t* out_draft_len, hipStream_t stream) {
    if (count <= (int64_t)kThreads * 8)
        hipLaunchKernelGGL((select_kernel<false, true, 8>), dim3(1, nq), dim3(kThreads), 0,
                           stream, nullptr, keys, count, k, nullptr, out_ids, out_scores,
                           out_drafts, out_draft_len, spans, span_len, max_span, span_stride);
    else
        hipLaunchKernelGGL((select_kernel<false, true, kPer>), dim3(1, nq), dim3(kThreads), 0,
                           stream, nullptr, keys, count, k, nullptr, out_ids, out_scores,
                           out_drafts, out_draft_len, spans, span_len, max_span, span_stride);
}

}  // namespace

// One of the two key buffers of the selection levels, 256-byte rounded.
static size_t key_buffer_bytes(int64_t n, int nq, int k) {
    const int64_t chunks = ceil_div(n, kSelectChunk);
    const int64_t kk = k < kSelectChunk ? k : kSelectChunk;
    return ((size_t)nq * (size_t)chunks * (size_t)kk * sizeof(uint64_t) + 255) / 256 * 256;
}

size_t topk_workspace_bytes(int64_t n, int nq, int k) {
    const int64_t chunks = ceil_div(n, kSelectChunk);
    if (chunks <= 1) return 0;
    const int64_t kk = k < kSelectChunk ? k : kSelectChunk;
    const size_t one = (size_t)nq * (size_t)chunks * (size_t)kk * sizeof(uint64_t);
    return 2 * ((one + 255) / 256 * 256);                // the two key buffers
}

hipError_t launch_topk_gather(const float* scores, int64_t n, int nq, int k,
                              const int32_t* spans, const int32_t* span_len, int max_span,
                              int64_t span_stride, int64_t* out_ids, float* out_scores, int32_t* out_drafts,
                              int32_t* out_draft_len, void* workspace, hipStream_t stream) {
    const int64_t kk = k < kSelectChunk ? k : kSelectChunk;
    int64_t chunks = ceil_div(n, kSelectChunk);
    if (chunks <= 2) {
        // One block: up to kThreads * 8 scores take eight per thread, up to
        // two chunks' worth 32 (one launch instead of a level and a final).
        if (n > kSelectChunk) {
            hipLaunchKernelGGL((select_kernel<true, true, 2 * kPer>), dim3(1, nq), dim3(kThreads),
                               0, stream, scores, nullptr, n, k, nullptr, out_ids, out_scores,
                               out_drafts, out_draft_len, spans, span_len, max_span, span_stride);
            return hipGetLastError();
        }
        if (n <= (int64_t)kThreads * 8)
            hipLaunchKernelGGL((select_kernel<true, true, 8>), dim3(1, nq), dim3(kThreads), 0,
                               stream, scores, nullptr, n, k, nullptr, out_ids, out_scores,
                               out_drafts, out_draft_len, spans, span_len, max_span, span_stride);
        else
            hipLaunchKernelGGL((select_kernel<true, true, kPer>), dim3(1, nq), dim3(kThreads), 0,
                               stream, scores, nullptr, n, k, nullptr, out_ids, out_scores,
                               out_drafts, out_draft_len, spans, span_len, max_span, span_stride);
        return hipGetLastError();
    }
    const size_t one = key_buffer_bytes(n, nq, k);
    uint64_t* buf[2] = {(uint64_t*)workspace, (uint64_t*)((char*)workspace + one)};
    hipLaunchKernelGGL((select_kernel<true, false, kPer>), dim3((unsigned)chunks, nq), dim3(kThreads),
                       0, stream, scores, nullptr, n, k, buf[0], nullptr, nullptr, nullptr,
                       nullptr, nullptr, nullptr, 0, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int64_t count = chunks * kk;
    int cur = 0;
    while ((chunks = ceil_div(count, kSelectChunk)) > 1) {
        hipLaunchKernelGGL((select_kernel<false, false, kPer>), dim3((unsigned)chunks, nq),
                           dim3(kThreads), 0, stream, nullptr, buf[cur], count, k, buf[cur ^ 1],
                           nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        count = chunks * kk;
        cur ^= 1;
    }
    launch_final_keys(buf[cur], count, nq, k, spans, span_len, max_span, span_stride, out_ids,
                      out_scores, out_drafts, out_draft_len, stream);
    return hipGetLastError();
}

hipError_t launch_topk_keys(const uint64_t* keys, int64_t count, int nq, int k,
                            const int32_t* spans, const int32_t* span_len, int max_span,
                            int64_t span_stride, int64_t* out_ids, float* out_scores,
                            int32_t* out_drafts, int32_t* out_draft_len,
                            const int32_t* dev_count, hipStream_t stream) {
    // A count known here that fits one chunk takes the smaller block.
    if (!dev_count && count <= kSelectChunk) {
        launch_final_keys(keys, count, nq, k, spans, span_len, max_span, span_stride, out_ids,
                          out_scores, out_drafts, out_draft_len, stream);
        return hipGetLastError();
    }
    // One block per query walks its own count.
    hipLaunchKernelGGL(select_stream_kernel, dim3(nq), dim3(kStreamThreads), 0, stream, keys,
                       count, k, dev_count, out_ids, out_scores, out_drafts, out_draft_len, spans,
                       span_len, max_span, span_stride);
    return hipGetLastError();
}

}  // namespace sense
