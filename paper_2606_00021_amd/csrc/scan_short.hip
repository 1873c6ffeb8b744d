// Batched similarity scan of short keys (d <= 64, e.g. the 64-dim PCA keys)
// on the matrix cores, every score or the best of each group of rows (Sec. 3.2
// Eq. 8 for a batch of queries; the top-N' retrieval of Eq. 7).
//
// A 64-dim key is 128 bytes, so the long-key MFMA design (a ring of key
// stages walking d) has nothing to pipeline across.  Here every wave keeps
// the whole query batch (up to 64 queries x 64 dims, hi and lo halves) in
// registers as A fragments and streams 16-key tiles as B fragments straight
// from HBM: lane l loads 16 bytes of key (base + l%16) at dims 8*(l/16) and
// 32 + 8*(l/16), so one tile is 16 contiguous rows (2 KiB at d = 64).  Four
// tiles are in flight per wave.  Per tile: 4 query tiles x 2 k-steps x
// (hi, lo) MFMA 16x16x32 instructions.
//
// The 64 x n score matrix would be 256 MB at n = 1M: writing it and reading
// it back for the top-k costs more than reading the keys.  So a large store is
// cut into groups of 16 to 64 consecutive rows, and the scan stores each
// query's best score per group only (scan_groups_kernel).  The k best groups by
// (score descending, group ascending) hold the k best rows by (score
// descending, row ascending): the best rows of those k groups precede any row
// of another group.  The rows of these groups are scored again
// (score_groups_kernel) and their top k is the result.  Both passes and the
// plain scan form a score with the same instructions, hence the same bits.
#include "internal.h"
#include "lds_dma.h"
#include "topk_device.h"

#include <type_traits>

namespace sense {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kShortThreads = 256;
constexpr int kShortDepth = 4;     // 16-key tiles in flight per wave

template <int KT>
__device__ __forceinline__ f32x4 mfma(const u32x4& a, const u32x4& b, const f32x4& c) {
    if constexpr (KT == DT_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// NT query tiles of 16, KS k-steps of 32 dims (d <= 32 * KS).
template <int KT, int NT, int KS, bool SPLIT>
__global__ __launch_bounds__(kShortThreads, 2) void scan_short_kernel(ShortScan s,
                                                                  int64_t rows_per_wave) {
    // The scales 1/|q| in LDS (read in the epilogue without a wait on the key
    // loads in flight, and without registers).
    __shared__ float s_qn[64];
    if (threadIdx.x < 64) s_qn[threadIdx.x] = threadIdx.x < 16 * NT ? s.inv_qn[threadIdx.x] : 0.0f;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    // The wave index is uniform: the row loop below is then a scalar loop.
    const int64_t wave = (int64_t)blockIdx.x * (kShortThreads / 64) +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r0 = wave * rows_per_wave;
    if (r0 >= s.n_rows) return;                      // uniform over the wave
    const int64_t r1 = (r0 + rows_per_wave < s.n_rows) ? r0 + rows_per_wave : s.n_rows;
    const int col = lane & 15, grp = lane >> 4;

    // Query fragments: A[m = col][k = 8*grp + 32*ks], for every query tile.
    u32x4 ahi[NT][KS], alo[NT][KS];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int dim = 8 * grp + 32 * ks;
            const int64_t qrow = 16 * t + col;
            const bool ok = dim < s.d;
            ahi[t][ks] = ok ? *(const u32x4*)(s.qhi + qrow * s.d + dim) : u32x4{0u, 0u, 0u, 0u};
            if constexpr (SPLIT)
                alo[t][ks] = ok ? *(const u32x4*)(s.qlo + qrow * s.d + dim) : u32x4{0u, 0u, 0u, 0u};
        }
    }
    // This lane's key row advances by 16 rows per tile: pointers step by a
    // fixed stride (no 64-bit multiplies per tile).  Every load is issued
    // unconditionally, so the compiler can count the loads in flight exactly
    // (a load under a branch makes it wait for all of them): rows past r1
    // re-read the lane's last row (their scores are discarded), dims past d
    // read dim 0 and are zeroed before use.  Everything an iteration reads
    // comes in with the tile (keys and the key norm): a load issued later and
    // consumed earlier would make the wave wait for all the tiles in flight
    // before it.
    const int64_t key_step = 16 * s.ld;
    const int64_t norm_step = s.inv_norm ? 16 : 0;
    const int64_t row_first = (r0 + col < r1) ? r0 + col : r1 - 1;
    const uint16_t* kp = (const uint16_t*)s.keys + row_first * s.ld;
    // Without key norms the norm load reads a fixed valid word (unused).
    const float* np = s.inv_norm ? s.inv_norm + row_first : s.inv_qn;
    const bool dim0 = 8 * grp < s.d;                 // this lane's dims hold key elements
    const bool dim1 = 8 * grp + 32 < s.d;            // ... in the second k-step
    const int off0 = dim0 ? 8 * grp : 0;
    const int off1 = dim1 ? 8 * grp + 32 : 0;
    int64_t lr = r0 + col;                           // row of the next tile to load
    auto load_tile = [&](u32x4 (&b)[KS], float& kn) {
        b[0] = __builtin_nontemporal_load((const u32x4*)(kp + off0));
        if constexpr (KS == 2) b[1] = __builtin_nontemporal_load((const u32x4*)(kp + off1));
        kn = *np;
        lr += 16;
        if (lr < r1) {                               // the next load stays on a valid row
            kp += key_step;
            np += norm_step;
        }
    };
    // The products of one tile; the tile's registers are free afterwards.
    auto products = [&](const u32x4 (&bt)[KS], f32x4 (&acc)[NT]) {
        u32x4 b[KS];
        b[0] = dim0 ? bt[0] : u32x4{0u, 0u, 0u, 0u};
        if constexpr (KS == 2) b[1] = dim1 ? bt[1] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                acc[t] = mfma<KT>(ahi[t][ks], b[ks], acc[t]);
                if constexpr (SPLIT) acc[t] = mfma<KT>(alo[t][ks], b[ks], acc[t]);
            }
        }
    };
    // Scores of row r (this lane's key) for every query.
    auto epilogue = [&](int64_t r, const f32x4 (&acc)[NT], float kn) {
        float v[NT][4];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[t][i] = acc[t][i];
                if (s.inv_norm) v[t][i] = v[t][i] * kn;
                v[t][i] = v[t][i] * s_qn[16 * t + 4 * grp + i];
            }
        if (r >= r1) return;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = 16 * t + 4 * grp + i;
                if (q < s.nq) s.scores[(int64_t)q * s.n_rows + r] = v[t][i];
            }
    };

    u32x4 buf[kShortDepth][KS];
    float kn[kShortDepth];
    // The first tiles in the loop's own order (keys, then norm, per tile):
    // the wait at the loop head is computed for both ways in, so a
    // different order here would make every iteration wait for more tiles.
#pragma unroll
    for (int u = 0; u < kShortDepth; ++u) {
        load_tile(buf[u], kn[u]);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int64_t base = r0; base < r1; base += 16 * kShortDepth) {
#pragma unroll
        for (int u = 0; u < kShortDepth; ++u) {
            // The slot's next tile is requested before the epilogue, whose
            // branches would otherwise keep the load behind them.
            f32x4 acc[NT];
            products(buf[u], acc);
            const float knu = kn[u];
            load_tile(buf[u], kn[u]);
            epilogue(base + 16 * u + col, acc, knu);
        }
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x),
                                                                 CTRL, 0xF, 0xF, false));
}

// Maxima that pass over a quiet NaN (every operand here is a product or one of
// these); as instructions, since fmaxf quiets each operand first.
__device__ __forceinline__ float max_f(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max3_f(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// One step of a transposing maximum over lane pairs (the lanes that CTRL swaps
// differ in `bit`): of each two values a lane keeps one and gives the other
// away, the lane with the bit set keeps the second.
template <int CTRL, int N>
__device__ __forceinline__ void swap_max(float (&v)[16], bool bit) {
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
        const float keep = bit ? v[2 * j + 1] : v[2 * j], give = bit ? v[2 * j] : v[2 * j + 1];
        v[j] = max_f(keep, dpp_f<CTRL>(give));
    }
}

// The best score of every group of group_rows rows (a multiple of 16) for each
// query, gmax[q * n_groups + g]; NaN where no row of the group has a number.
//
// Reading the matrix-core operand layout straight from HBM (as above) takes 64
// bytes of each of 16 rows per load instruction, a pattern this device serves
// below its streaming rate, and holds every tile in flight in registers.  Here
// global_load_lds_dwordx4 moves whole rows (8 per instruction) into a private
// ring of kRing tile slots per wave, kRing - 1 tiles ahead of the products, and
// each lane reads its operand from LDS: lane L = 8p + w of an instruction
// writes entry w of row p and fetches unit (w + p) mod 8 of that row (unit u of
// row p sits at entry (u - p) mod 8, rows 8-15 at entries 64 + ...), so the 8
// rows a matrix-core read touches in each half fall on 8 distinct 16-byte
// groups.  Units past a row shorter than 64 dims re-read its first and are
// zeroed as operands.  A tile's 16 key norms come the same way (inner product
// loads a valid dummy word and uses a scale of 1).  Every iteration issues the
// same three loads (tiles past the end reload the last one), so the wait for a
// tile is a fixed count.
//
// A lane keeps the running maxima of its key column for its 4 * NT queries (one
// product and one maximum per score); at a group's end 16 columns meet in four
// transposing steps that leave each lane one query's maximum.  The query's
// scale, a factor >= 0, goes on the maximum: rounding is monotone, so that is
// the maximum of the scaled scores, but for a scale of 0 (a query whose squared
// norm is beyond fp32) on an infinite maximum.  Such a wave goes over its rows
// again with the scale on every score.
//
// Bound: the read of the keys, 34 us for 1M x 64 bf16 and 64 queries (4.1 TB/s;
// 33 without the products: loads alone, norms and stores of the maxima), of
// which a wave's start is about 6.  Four slots and twice the waves: 36-38 us.
// With the selection, rescore and top-k behind it 100 -> 75.7 us a search
// against a strided sample's k-th best as the threshold of a filtered pass.
constexpr int kRing = 8;           // tile slots per wave
constexpr int kDmaOps = 3;         // loads per tile: two key halves, the norms

template <int KT, int NT, bool SPLIT>
__global__ __launch_bounds__(kShortThreads, 2) void scan_groups_kernel(ShortScan s,
                                                                       int64_t groups_per_wave) {
    __shared__ __attribute__((aligned(16))) u32x4 s_key[kShortThreads / 64][kRing][128];
    __shared__ __attribute__((aligned(16))) float s_norm[kShortThreads / 64][kRing][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t wave = (int64_t)blockIdx.x * (kShortThreads / 64) + wv;
    const int64_t g0 = wave * groups_per_wave;
    const int64_t r0 = g0 * s.group_rows;
    if (r0 >= s.n_rows) return;                      // uniform over the wave
    const int64_t r_end = (g0 + groups_per_wave) * s.group_rows;
    const int64_t r1 = r_end < s.n_rows ? r_end : s.n_rows;
    const int ntiles = (int)((r1 - r0 + 15) / 16);
    const int col = lane & 15, grp = lane >> 4;
    const bool dim0 = 8 * grp < s.d, dim1 = 8 * grp + 32 < s.d;   // this lane's dims exist

    // This lane's sources: its unit of rows dp and 8 + dp of the next tile to
    // request, and its column's norm; they step by a tile at a time and stay on
    // the last one.
    const uint16_t* keys = (const uint16_t*)s.keys;
    const bool cosine = s.inv_norm != nullptr;
    const int dp = lane >> 3;                        // row within a load instruction
    int du = ((lane & 7) + dp) & 7;                  // 16-byte unit it fetches
    du = 8 * du < s.d ? du : 0;
    const int64_t step = 16 * s.ld, nstep = cosine ? 16 : 0;
    const uint16_t* src[2];
    const float* nsrc;
    auto at_tile = [&](int t) {                      // on clamped rows
        const int64_t base = r0 + 16 * (int64_t)t;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t row = base + 8 * i + dp;
            src[i] = keys + (row < r1 ? row : r1 - 1) * s.ld + du * 8;
        }
        const int64_t nrow = base + col;
        nsrc = cosine ? s.inv_norm + (nrow < r1 ? nrow : r1 - 1) : s.inv_qn;
    };
    at_tile(0);
    int req = 0;                                     // the tile src stands on
    const bool ragged = r0 + 16 * (int64_t)ntiles > r1;
    auto issue = [&](int slot) {
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16_nt(src[i], &s_key[wv][slot][64 * i]);
        dma4(nsrc, &s_norm[wv][slot][0]);
        if (++req < ntiles) {
            if (ragged && req == ntiles - 1) {
                at_tile(req);
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i) src[i] += step;
                nsrc += nstep;
            }
        }
    };
    // Operand entry of this lane in a tile for k-step ks: row col, unit
    // grp + 4 ks.
    auto entry = [&](int ks) {
        const int p = col & 7;
        return 64 * (col >> 3) + 8 * p + (((grp + 4 * ks) - p) & 7);
    };
    const int e0 = entry(0), e1 = entry(1);

#pragma unroll
    for (int t = 0; t < kRing - 1; ++t) issue(t);
    // Query fragments A[m = col][k = 8*grp + 32*ks], requested behind the
    // first tiles and taken into registers before the loop.
    u32x4 ahi[NT][2], alo[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bool in = ks ? dim1 : dim0;
            const int64_t qoff = (int64_t)(16 * t + col) * s.d + (in ? 8 * grp + 32 * ks : 0);
            ahi[t][ks] = *(const u32x4*)(s.qhi + qoff);
            if constexpr (SPLIT) alo[t][ks] = *(const u32x4*)(s.qlo + qoff);
            if (!in) {
                ahi[t][ks] = u32x4{0u, 0u, 0u, 0u};
                if constexpr (SPLIT) alo[t][ks] = u32x4{0u, 0u, 0u, 0u};
            }
        }
    // The query this lane stores: value 4 t + i of its group's 16 ends up in
    // the lane whose column is that number with its bits reversed.
    const int mine = (int)(__builtin_bitreverse32((uint32_t)col) >> 28);
    const int oq = 16 * (mine >> 2) + 4 * grp + (mine & 3);
    const bool out = oq < s.nq;
    float scale = s.inv_qn[out ? oq : 0];
    float* dst = s.gmax + (int64_t)(out ? oq : 0) * s.n_groups + g0;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            asm volatile("" : "+v"(ahi[t][ks]));
            if constexpr (SPLIT) asm volatile("" : "+v"(alo[t][ks]));
        }
    asm volatile("" : "+v"(scale));

    float m[NT][4];
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) m[q][i] = __builtin_nanf("");
    // Tile t's operands and column scale, after its three loads are complete.
    // Inner product scales by 1 (x * 1 is x: the same bits as no scale); rows
    // past the last one score NaN, which no maximum takes.
    auto take = [&](int t, u32x4& b0, u32x4& b1, float& ks) {
        const int slot = t % kRing;
        b0 = s_key[wv][slot][e0];
        b1 = s_key[wv][slot][e1];
        const float kn = s_norm[wv][slot][col];
        if (s.d < 64) {                              // uniform
            if (!dim0) b0 = u32x4{0u, 0u, 0u, 0u};
            if (!dim1) b1 = u32x4{0u, 0u, 0u, 0u};
        }
        ks = cosine ? kn : 1.0f;
        if (ragged && t == ntiles - 1 && r0 + 16 * (int64_t)t + col >= r1) ks = __builtin_nanf("");
    };
    // Scores of TN tiles (each its own sums, query tiles between the steps of
    // one sum), into the maxima.
    auto score = [&](auto tn, const u32x4 (&b)[2][2], const float (&ks)[2]) {
        constexpr int TN = decltype(tn)::value;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            f32x4 acc[TN];
#pragma unroll
            for (int u = 0; u < TN; ++u)
                acc[u] = mfma<KT>(ahi[q][0], b[u][0], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
            if constexpr (SPLIT)
#pragma unroll
                for (int u = 0; u < TN; ++u) acc[u] = mfma<KT>(alo[q][0], b[u][0], acc[u]);
#pragma unroll
            for (int u = 0; u < TN; ++u) acc[u] = mfma<KT>(ahi[q][1], b[u][1], acc[u]);
            if constexpr (SPLIT)
#pragma unroll
                for (int u = 0; u < TN; ++u) acc[u] = mfma<KT>(alo[q][1], b[u][1], acc[u]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (TN == 2)
                    m[q][i] = max3_f(m[q][i], acc[0][i] * ks[0], acc[1][i] * ks[1]);
                else
                    m[q][i] = max_f(m[q][i], acc[0][i] * ks[0]);
            }
        }
    };
    const int per_group = s.group_rows / 16;
    int left = per_group;                            // tiles to the end of the group
    bool over = false;                               // this lane's query had an infinite maximum
    for (int t = 0; t < ntiles;) {
        u32x4 b[2][2];
        float ks[2];
        if (left >= 2 && t + 2 <= ntiles) {
            wait_vmcnt<(kRing - 3) * kDmaOps>();       // tiles t and t + 1 are in LDS
            take(t, b[0][0], b[0][1], ks[0]);
            take(t + 1, b[1][0], b[1][1], ks[1]);
            issue((t + kRing - 1) % kRing);          // the slot read last
            score(std::integral_constant<int, 2>{}, b, ks);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // tile t was read
            issue((t + kRing) % kRing);
            t += 2;
            left -= 2;
        } else {
            wait_vmcnt<(kRing - 2) * kDmaOps>();
            take(t, b[0][0], b[0][1], ks[0]);
            issue((t + kRing - 1) % kRing);
            score(std::integral_constant<int, 1>{}, b, ks);
            t += 1;
            left -= 1;
        }
        if (left == 0 || t == ntiles) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[4 * q + i] = q < NT ? m[q < NT ? q : 0][i] : 0.0f;
                    if (q < NT) m[q < NT ? q : 0][i] = __builtin_nanf("");
                }
            swap_max<0x140, 16>(v, col & 8);         // row mirror
            swap_max<0x141, 8>(v, col & 4);          // half-row mirror
            swap_max<0x4E, 4>(v, col & 2);           // quad xor 2
            swap_max<0xB1, 2>(v, col & 1);           // quad xor 1
            if (out) *dst = v[0] * scale;
            over |= v[0] == __builtin_inff();
            ++dst;
            left = per_group;
        }
    }
    wait_vmcnt<0>();
    if (!__ballot(out && over && scale == 0.0f)) return;
    // A finite product of the query makes the row's score 0, another NaN.
    float* again = s.gmax + (int64_t)(out ? oq : 0) * s.n_groups + g0;
    for (int64_t r = r0; r < r1; r += s.group_rows, ++again) {
        const int64_t r_top = r + s.group_rows < r1 ? r + s.group_rows : r1;
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = __builtin_nanf("");
        for (int64_t base = r; base < r_top; base += 16) {
            const bool row_in = base + col < r_top;
            const int64_t row = row_in ? base + col : r_top - 1;
            const uint16_t* kp = keys + row * s.ld;
            u32x4 b0 = *(const u32x4*)(kp + (dim0 ? 8 * grp : 0));
            u32x4 b1 = *(const u32x4*)(kp + (dim1 ? 8 * grp + 32 : 0));
            const float kn = cosine ? s.inv_norm[row] : 1.0f;
            if (!dim0) b0 = u32x4{0u, 0u, 0u, 0u};
            if (!dim1) b1 = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                f32x4 acc = mfma<KT>(ahi[q][0], b0, f32x4{0.0f, 0.0f, 0.0f, 0.0f});
                if constexpr (SPLIT) acc = mfma<KT>(alo[q][0], b0, acc);
                acc = mfma<KT>(ahi[q][1], b1, acc);
                if constexpr (SPLIT) acc = mfma<KT>(alo[q][1], b1, acc);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (row_in && __builtin_fabsf(acc[i] * kn) < __builtin_inff()) v[4 * q + i] = 0.0f;
            }
        }
        swap_max<0x140, 16>(v, col & 8);
        swap_max<0x141, 8>(v, col & 4);
        swap_max<0x4E, 4>(v, col & 2);
        swap_max<0xB1, 2>(v, col & 1);
        if (out && scale == 0.0f) *again = v[0];
    }
}

// The scores of the rows of each query's best groups: one wave per (query,
// group), its tiles from the store in the operand layout, every row of A the
// one query, so that lane (grp, col) has row col of each tile and stores that
// of tile grp.  keys[q * count + j * group_rows + row], count = n_hits *
// group_rows; 0 (a padding key) past the store and for a missing group.
template <int KT, bool SPLIT>
__global__ __launch_bounds__(kShortThreads) void score_groups_kernel(
    ShortScan s, const int64_t* __restrict__ ids, int k, int n_hits,
    uint64_t* __restrict__ out_keys) {
    const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
    const int q = blockIdx.y;
    const int j = blockIdx.x * (kShortThreads / 64) +
                  __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (j >= n_hits) return;                         // uniform over the wave
    const int64_t id = ids[(int64_t)q * k + j];
    const bool dim[2] = {8 * grp < s.d, 8 * grp + 32 < s.d};
    u32x4 ahi[2], alo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int64_t qoff = (int64_t)q * s.d + (dim[ks] ? 8 * grp + 32 * ks : 0);
        ahi[ks] = *(const u32x4*)(s.qhi + qoff);
        if constexpr (SPLIT) alo[ks] = *(const u32x4*)(s.qlo + qoff);
        if (!dim[ks]) {
            ahi[ks] = u32x4{0u, 0u, 0u, 0u};
            if constexpr (SPLIT) alo[ks] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    const float qn = s.inv_qn[q];
    const int64_t r0 = (id < 0 ? 0 : id) * s.group_rows;
    u32x4 b[4][2];
    float kn[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {                    // tiles past the group re-read rows
        int64_t r = r0 + 16 * t + col;
        r = r < s.n_rows ? r : s.n_rows - 1;
        const uint16_t* row = (const uint16_t*)s.keys + r * s.ld;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            b[t][ks] = *(const u32x4*)(row + (dim[ks] ? 8 * grp + 32 * ks : 0));
        kn[t] = s.inv_norm ? s.inv_norm[r] : 1.0f;
    }
    float mine = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            if (!dim[ks]) b[t][ks] = u32x4{0u, 0u, 0u, 0u};
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            acc = mfma<KT>(ahi[ks], b[t][ks], acc);
            if constexpr (SPLIT) acc = mfma<KT>(alo[ks], b[t][ks], acc);
        }
        const float v = (acc[0] * kn[t]) * qn;
        mine = grp == t ? v : mine;
    }
    const int64_t r = r0 + lane;                     // row 16 grp + col
    if (lane < s.group_rows)
        out_keys[((int64_t)q * n_hits + j) * s.group_rows + lane] =
            (id >= 0 && r < s.n_rows) ? pack_key(mine, (uint32_t)r) : 0ull;
}

// score_groups_kernel and the selections on either side of it in one block per
// query: the n_hits best of at most 16384 group maxima, the scores of their
// rows (at most kTailRows) straight into registers, and the top k of those with
// its output.
//
// Bound: latency (one compute unit per query; loads, barriers and histogram
// passes in turn), which is why more rows are scored by all compute units and
// selected in launches of their own: whole search, 64 queries over 131072 x 64,
// k = 100 (1600 rows) 48.4 us so and 55.0 in three launches; over 1M, k = 64
// (4096 rows) 79.3 so and 75.7 in three.
constexpr int kTailThreads = 1024;
constexpr int kTailGroups = (int)kSelectGroups;
constexpr int kTailRows = 2048;

template <int KT, bool SPLIT>
__global__ __launch_bounds__(kTailThreads) void best_groups_kernel(
    ShortScan s, int n_hits, int k, int64_t* __restrict__ out_ids,
    float* __restrict__ out_scores, int32_t* __restrict__ out_drafts,
    int32_t* __restrict__ out_draft_len, const int32_t* __restrict__ spans,
    const int32_t* __restrict__ span_len, int max_span, int64_t span_stride) {
    constexpr int W = kTailThreads / 64;
    constexpr int GP = kTailGroups / kTailThreads, P = kTailRows / kTailThreads;
    __shared__ uint64_t s_sel[kMaxK];
    __shared__ uint64_t s_sorted[kMaxK];
    __shared__ __align__(16) uint32_t s_hist[W * 256];        // read 16 bytes at a time
    __shared__ uint32_t s_info[4];
    __shared__ uint32_t s_nzw[W], s_wc[W];
    __shared__ uint64_t s_andw[W], s_orw[W];
    __shared__ uint32_t s_loww[W], s_highw[W];
    const StatsLds lds{s_nzw, s_andw, s_orw, s_loww, s_highw};
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;

    // The query, every row of A (see score_groups_kernel).
    const bool dim[2] = {8 * grp < s.d, 8 * grp + 32 < s.d};
    u32x4 ahi[2], alo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int64_t qoff = (int64_t)q * s.d + (dim[ks] ? 8 * grp + 32 * ks : 0);
        ahi[ks] = *(const u32x4*)(s.qhi + qoff);
        if constexpr (SPLIT) alo[ks] = *(const u32x4*)(s.qlo + qoff);
    }
    const float qn = s.inv_qn[q];

    // The best groups, in any order.
    {
        const float* src = s.gmax + (int64_t)q * s.n_groups;
        const int len = (int)s.n_groups;
        float sv[GP];
#pragma unroll
        for (int e = 0; e < GP; ++e) {
            const int i = tid + e * kTailThreads;
            sv[e] = src[i < len ? i : len - 1];
        }
        uint32_t sw[GP];
        uint64_t key[GP];
#pragma unroll
        for (int e = 0; e < GP; ++e) {
            const int i = tid + e * kTailThreads;
            sw[e] = score_key(sv[e]);
            key[e] = i < len ? (((uint64_t)sw[e] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i))
                             : 0ull;
        }
        const ChunkStats cs = score_stats<kTailThreads, GP>(sw, key, n_hits, 0, len, lds);
        SelectState st{1ull, ~0ull};
        if (cs.nz > (uint32_t)n_hits)
            st = radix_select<kTailThreads, GP, true>(key, n_hits, cs, s_hist, s_info);
        compact_taken<kTailThreads, GP>(key, st.mask, st.prefix, s_sel, n_hits, s_wc);
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        if (!dim[ks]) {
            ahi[ks] = u32x4{0u, 0u, 0u, 0u};
            if constexpr (SPLIT) alo[ks] = u32x4{0u, 0u, 0u, 0u};
        }

    // Their rows, four tiles of 16 per wave and key slot: lane (grp, col) keeps
    // row col of tile grp.
    const int per = s.group_rows / 16;               // tiles per group
    const int tiles = n_hits * per;
    uint64_t key[P];
#pragma unroll
    for (int e = 0; e < P; ++e) {
        const int c0 = 4 * (wv + W * e);
        u32x4 b[4][2];
        float kn[4];
        int64_t my_row = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {                // tiles past the last re-read it
            const int c = c0 + t < tiles ? c0 + t : tiles - 1;
            const int hit = c / per;
            const int64_t r = (int64_t)key_row(s_sel[hit]) * s.group_rows +
                              16 * (c - hit * per) + col;
            const int64_t rc = r < s.n_rows ? r : s.n_rows - 1;
            const uint16_t* row = (const uint16_t*)s.keys + rc * s.ld;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                b[t][ks] = *(const u32x4*)(row + (dim[ks] ? 8 * grp + 32 * ks : 0));
            kn[t] = s.inv_norm ? s.inv_norm[rc] : 1.0f;
            my_row = grp == t ? r : my_row;
        }
        float mine = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                if (!dim[ks]) b[t][ks] = u32x4{0u, 0u, 0u, 0u};
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                acc = mfma<KT>(ahi[ks], b[t][ks], acc);
                if constexpr (SPLIT) acc = mfma<KT>(alo[ks], b[t][ks], acc);
            }
            const float v = (acc[0] * kn[t]) * qn;
            mine = grp == t ? v : mine;
        }
        key[e] = (c0 + grp < tiles && my_row < s.n_rows) ? pack_key(mine, (uint32_t)my_row) : 0ull;
    }
    const ChunkStats cs = chunk_stats<kTailThreads, P, true>(key, k, lds);
    SelectState st{1ull, ~0ull};
    if (cs.nz > (uint32_t)k)
        st = radix_select<kTailThreads, P, true>(key, k, cs, s_hist, s_info);
    const uint32_t tot = compact_taken<kTailThreads, P>(key, st.mask, st.prefix, s_sel, k, s_wc);
    const int nt = (int)tot < k ? (int)tot : k;
    final_output<kTailThreads>(s_sel, s_sorted, nt, k, q, out_ids, out_scores, out_drafts,
                               out_draft_len, spans, span_len, max_span, span_stride);
}

__global__ void short_tau_kernel(const int64_t* __restrict__ ids, const float* __restrict__ scores,
                                 int nq, int k, int64_t row_step, int32_t slot_area,
                                 const float* __restrict__ margin, uint64_t* __restrict__ tau,
                                 int32_t* __restrict__ counts) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const int64_t id = ids[(int64_t)q * k + (k - 1)];
    // A sample shorter than k leaves a padding id: then every row passes.
    // With approximate scores the threshold is lowered by the margin.
    float s = scores[(int64_t)q * k + (k - 1)];
    if (margin) s = s - margin[q];
    tau[q] = id < 0 ? 0ull : pack_key(s, (uint32_t)(id * row_step));
    counts[q] = slot_area;          // overflow entries follow the wave slots
}

// Two resident waves per SIMD (scan_short_kernel's register use allows two).
int64_t short_rows_per_wave(int64_t n_rows) {
    const int64_t waves_max = (int64_t)device_cus() * 8;
    int64_t rpw = (n_rows + waves_max - 1) / waves_max;
    return (rpw + 16 * kShortDepth - 1) / (16 * kShortDepth) * (16 * kShortDepth);
}

unsigned blocks_of(int64_t waves) {
    return (unsigned)((waves + (kShortThreads / 64) - 1) / (kShortThreads / 64));
}

template <int KT, int NT, int KS>
hipError_t launch_mode(const ShortScan& s, hipStream_t stream) {
    const int64_t rpw = short_rows_per_wave(s.n_rows);
    const dim3 grid(blocks_of((s.n_rows + rpw - 1) / rpw));
    if (s.split)
        hipLaunchKernelGGL((scan_short_kernel<KT, NT, KS, true>), grid, dim3(kShortThreads), 0,
                           stream, s, rpw);
    else
        hipLaunchKernelGGL((scan_short_kernel<KT, NT, KS, false>), grid, dim3(kShortThreads), 0,
                           stream, s, rpw);
    return hipGetLastError();
}

template <int KT, int NT>
hipError_t launch_groups(const ShortScan& s, hipStream_t stream) {
    // One resident round (two waves per SIMD: the ring's LDS): a wave's start
    // (query fragments, first tiles) costs as much as several groups.
    const int64_t waves_max = (int64_t)device_cus() * 8;
    const int64_t gpw = (s.n_groups + waves_max - 1) / waves_max;
    const dim3 grid(blocks_of((s.n_groups + gpw - 1) / gpw));
    if (s.split)
        hipLaunchKernelGGL((scan_groups_kernel<KT, NT, true>), grid, dim3(kShortThreads), 0,
                           stream, s, gpw);
    else
        hipLaunchKernelGGL((scan_groups_kernel<KT, NT, false>), grid, dim3(kShortThreads), 0,
                           stream, s, gpw);
    return hipGetLastError();
}

template <int KT>
hipError_t launch_score_groups_t(const ShortScan& s, const int64_t* ids, int k, int n_hits,
                                 uint64_t* keys, hipStream_t stream) {
    const dim3 grid(blocks_of(n_hits), (unsigned)s.nq);
    if (s.split)
        hipLaunchKernelGGL((score_groups_kernel<KT, true>), grid, dim3(kShortThreads), 0, stream,
                           s, ids, k, n_hits, keys);
    else
        hipLaunchKernelGGL((score_groups_kernel<KT, false>), grid, dim3(kShortThreads), 0, stream,
                           s, ids, k, n_hits, keys);
    return hipGetLastError();
}

template <int KT, bool SPLIT>
hipError_t launch_best_groups_t(const ShortScan& s, int n_hits, const TopkOut& o,
                                hipStream_t stream) {
    hipLaunchKernelGGL((best_groups_kernel<KT, SPLIT>), dim3((unsigned)s.nq), dim3(kTailThreads),
                       0, stream, s, n_hits, o.k, o.ids, o.scores, o.drafts, o.draft_len, o.spans, o.span_len, o.max_span,
                       o.span_stride);
    return hipGetLastError();
}

template <int KT, int KS>
hipError_t launch_tiles(const ShortScan& s, hipStream_t stream) {
    switch ((s.nq + 15) / 16) {
        case 1: return launch_mode<KT, 1, KS>(s, stream);
        case 2: return launch_mode<KT, 2, KS>(s, stream);
        case 3: return launch_mode<KT, 3, KS>(s, stream);
        default: return launch_mode<KT, 4, KS>(s, stream);
    }
}

}  // namespace

hipError_t launch_scan_short(const ShortScan& s, hipStream_t stream) {
    const bool two = s.d > 32;
    if (s.key_dtype == DT_BF16)
        return two ? launch_tiles<DT_BF16, 2>(s, stream) : launch_tiles<DT_BF16, 1>(s, stream);
    return two ? launch_tiles<DT_F16, 2>(s, stream) : launch_tiles<DT_F16, 1>(s, stream);
}

template <int KT>
static hipError_t launch_groups_t(const ShortScan& s, hipStream_t stream) {
    switch ((s.nq + 15) / 16) {
        case 1: return launch_groups<KT, 1>(s, stream);
        case 2: return launch_groups<KT, 2>(s, stream);
        case 3: return launch_groups<KT, 3>(s, stream);
        default: return launch_groups<KT, 4>(s, stream);
    }
}

hipError_t launch_scan_groups(const ShortScan& s, hipStream_t stream) {
    return s.key_dtype == DT_BF16 ? launch_groups_t<DT_BF16>(s, stream)
                                  : launch_groups_t<DT_F16>(s, stream);
}

bool best_groups_fit(const ShortScan& s, int n_hits) {
    return s.n_groups <= kTailGroups && n_hits * s.group_rows <= kTailRows;
}

hipError_t launch_best_groups(const ShortScan& s, int n_hits, const TopkOut& o,
                              hipStream_t stream) {
    if (s.key_dtype == DT_BF16)
        return s.split ? launch_best_groups_t<DT_BF16, true>(s, n_hits, o, stream)
                       : launch_best_groups_t<DT_BF16, false>(s, n_hits, o, stream);
    return s.split ? launch_best_groups_t<DT_F16, true>(s, n_hits, o, stream)
                   : launch_best_groups_t<DT_F16, false>(s, n_hits, o, stream);
}

hipError_t launch_score_groups(const ShortScan& s, const int64_t* ids, int k, int n_hits,
                               uint64_t* keys, hipStream_t stream) {
    return s.key_dtype == DT_BF16 ? launch_score_groups_t<DT_BF16>(s, ids, k, n_hits, keys, stream)
                                  : launch_score_groups_t<DT_F16>(s, ids, k, n_hits, keys, stream);
}

hipError_t launch_short_tau(const int64_t* ids, const float* scores, int nq, int k,
                            int64_t row_step, int32_t slot_area, const float* margin,
                            uint64_t* tau, int32_t* counts, hipStream_t stream) {
    hipLaunchKernelGGL(short_tau_kernel, dim3((unsigned)((nq + 63) / 64)), dim3(64), 0, stream,
                       ids, scores, nq, k, row_step, slot_area, margin, tau, counts);
    return hipGetLastError();
}

}  // namespace sense
