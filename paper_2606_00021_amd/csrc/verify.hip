// Soft-gated evaluation (Sec. 3.3 Eqs. 12-18; Alg. 4) of a candidate draft
// batch against the target's aligned logits.
//
// The cost is one read of the logits of every live (candidate, position)
// row; everything else is per-row scalars.  Two kernels:
//
// verify_rows: one block of 256 threads per (row, vocabulary slice).  A
//   thread takes four 16-byte words of the slice per step, the next step's
//   words requested before this one's are used, so a block's loads stay in
//   flight through its arithmetic, and no step waits for another wave.  Every
//   lane keeps its own running maximum m2 (times log2 e), and with
//   t = x log2 e - m2
//       S   = sum 2^t,   T2 = sum 2^t * t;
//   beside them the wave counts
//       cnt = #{v : x_v > x_d} + #{v < d : x_v = x_d},  x_d the draft token's
//             logit, as x_v >= x_d left of d and x_v >= next(x_d) from d on.
//   The lanes, then the waves, are brought to one maximum at the end, and the
//   block stores one 16-byte partial (m2, S, T2, cnt) per (row, slice).  With
//   p = softmax(x), E = -sum p ln p = ln S - ln2 * T2 / S.  The draft token
//   is the first argmax exactly when cnt = 0 and is in the top-k set exactly
//   when cnt < k, so neither an argmax nor a sort of the vocabulary is needed.
//   Sums are formed in a fixed order (DPP butterflies, then the waves in
//   order), so results are deterministic.
//   Rows may start at any element: the elements before the first 16-byte word
//   of memory and behind the last go to single lanes.
//
//   Bound: the read of the rows; per 16-bit logit 6.5 vector issues (half of one
//   for the maximum, unpack, fma, exp2 at half rate, add, fma; 10.1 instructions
//   counted at 64 x 8 rows of 152064, the count of the judged logit, the state's
//   changes, prologue and reduction with them), one more where a logit of the wave reaches the judged one and one more
//   where a masked (-inf) one is among them.  64 x 8 of 152064 bf16 with a third
//   of the vocabulary masked: 31.4 us clamped throughout, 41.4 where every step
//   first forms the sums without the clamp, 31.6 so.
//   16 x 64 x 8 rows of 32000 fp32, ragged (half judged): 108 -> 77 us, 6.8
//   TB/s, most of it from dealing the judged rows evenly to the XCDs.  64 x 8 of
//   152064 bf16: 26 us before and after, 6.0 TB/s with launch and ramp; rows
//   of 151937, which start anywhere: 50 us one element at a time, 26 so.
//
// verify_finalize: one block per candidate group.  Phase 1 gives every
//   (candidate, position) row its own thread, which merges the row's slices
//   in slice order and forms the exact-match / entropy / top-k bits; phase 2
//   gives every row a thread again, which counts its window's mismatches
//   with one popcount over the candidate's 64-bit exact-match mask and forms
//   its gate bit; phase 3 gives every candidate a thread that takes the
//   leading run of its gate mask; the block then picks the group's first
//   longest candidate.
#include "internal.h"

namespace sense {
namespace {

constexpr int kRowThreads = kVerifyRowThreads;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kNV = 4;             // 16-byte words per thread and step
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct Partial {
    float m2;
    float s;
    float t2;
    int cnt;
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <int CTRL>
__device__ __forceinline__ int dpp_i(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __builtin_bit_cast(float, dpp_i<CTRL>(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ float lane_f(float x, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}

// Wave-uniform sum / max over 64 lanes in a fixed order.
__device__ __forceinline__ float wave_sum_f(float x) {
    x += dpp_f<0xB1>(x);
    x += dpp_f<0x4E>(x);
    x += dpp_f<0x141>(x);
    x += dpp_f<0x140>(x);
    return (lane_f(x, 0) + lane_f(x, 16)) + (lane_f(x, 32) + lane_f(x, 48));
}
__device__ __forceinline__ int wave_sum_i(int x) {
    x += dpp_i<0xB1>(x);
    x += dpp_i<0x4E>(x);
    x += dpp_i<0x141>(x);
    x += dpp_i<0x140>(x);
    return (__builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16)) +
           (__builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48));
}
__device__ __forceinline__ float wave_max_f(float x) {
    x = __builtin_fmaxf(x, dpp_f<0xB1>(x));
    x = __builtin_fmaxf(x, dpp_f<0x4E>(x));
    x = __builtin_fmaxf(x, dpp_f<0x141>(x));
    x = __builtin_fmaxf(x, dpp_f<0x140>(x));
    return __builtin_fmaxf(__builtin_fmaxf(lane_f(x, 0), lane_f(x, 16)),
                           __builtin_fmaxf(lane_f(x, 32), lane_f(x, 48)));
}

template <int LT>
__device__ __forceinline__ float bits_f32(uint32_t bits) {
    if constexpr (LT == DT_BF16) return __builtin_bit_cast(float, bits << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}

template <int LT>
__device__ __forceinline__ float load_one(const char* base, int64_t i) {
    if constexpr (LT == DT_F32) return ((const float*)base)[i];
    else return bits_f32<LT>(((const uint16_t*)base)[i]);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int LT>
__device__ __forceinline__ void unpack(const u32x4& w, float (&x)[LT == DT_F32 ? 4 : 8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // Copy the lane out first: a bit_cast applied directly to an element
        // of an ext_vector_type is mis-compiled by this hipcc (it reads the
        // wrong element).
        const uint32_t u = w[i];
        if constexpr (LT == DT_F32) {
            x[i] = __builtin_bit_cast(float, u);
        } else if constexpr (LT == DT_BF16) {
            x[2 * i] = __builtin_bit_cast(float, u << 16);
            x[2 * i + 1] = __builtin_bit_cast(float, u & 0xFFFF0000u);
        } else {
            x[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xFFFFu));
            x[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16));
        }
    }
}

// Threshold of "x > x_d" as "x >= next_up(x_d)": the smallest float above a
// finite or -inf x.  Nothing lies above +inf, so there it is NaN, which no
// comparison reaches (elements from d on that equal +inf rank below d, as in
// the stable order); NaN maps to itself.
__device__ __forceinline__ float next_up(float x) {
    if (x != x) return x;
    if (x == __builtin_inff()) return __builtin_nanf("");
    if (x == 0.0f) return __builtin_bit_cast(float, 1u);
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return __builtin_bit_cast(float, x > 0.0f ? u + 1u : u - 1u);
}

// What a lane has seen of a row: m2 = log2 e times the largest logit, and with
// t = x log2 e - m2 the sums S of 2^t and T2 of 2^t t.  Every change of the
// maximum goes through the difference of two rounded m2, so that all of a
// row's terms refer to the same numbers.
struct State {
    float m2 = -__builtin_inff(), s = 0.0f, t2 = 0.0f;
};

// The factor 2^(from - to) and its exponent, for from <= to.  The clamp (where
// 2^d is 0) covers an empty state (-inf) and two of them (NaN).
__device__ __forceinline__ float drop_to(float from, float to, float& d) {
    d = __builtin_fmaxf(from - to, -256.0f);
    return fast_exp2(d);
}

__device__ __forceinline__ void raise_to(State& a, float m2) {
    float d;
    const float f = drop_to(a.m2, m2, d);
    a.t2 = f * __builtin_fmaf(d, a.s, a.t2);
    a.s = f * a.s;
    a.m2 = m2;
}

// Merges the first n (uniform) of N partials into (a, c): to the largest maximum
// at once, so that no factor waits for another.
template <int N>
__device__ __forceinline__ void merge_all(State& a, int& c, const Partial (&q)[N], int n = N) {
    float m2 = a.m2;
#pragma unroll
    for (int u = 0; u < N; ++u)
        if (u < n) m2 = __builtin_fmaxf(m2, q[u].m2);
    raise_to(a, m2);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u < n) {
            State b{q[u].m2, q[u].s, q[u].t2};
            raise_to(b, m2);
            a.s += b.s;
            a.t2 += b.t2;
            c += q[u].cnt;
        }
    }
}

// The constant of t = x log2 e + base.
__device__ __forceinline__ float base_of(float m2) {
    return m2 == -__builtin_inff() ? 0.0f : -m2;
}

typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Makes what was derived from the words be derived again: the unpacked values
// of one path shall not be kept in registers for another.
template <int U>
__device__ __forceinline__ void forget(u32x4 (&buf)[U]) {
#pragma unroll
    for (int k = 0; k < U; ++k) asm volatile("" : "+v"(buf[k]));
}

// The largest of a lane's logits, NaN passed over.  As integers, floats of the
// positive sign keep their order and lie above all of the negative sign, whose
// order is reversed: one signed maximum, on two 16-bit logits at a time or two
// operands of a three-way maximum, settles every lane that holds a logit >= 0
// (half an instruction per logit, without unpacking).  Lanes of negative logits
// take the unsigned minimum, and a NaN that comes out on top the float maximum.
template <int LT, int U>
__device__ __forceinline__ float lane_max(u32x4 (&buf)[U]) {
    constexpr uint32_t kInf = LT == DT_F32 ? 0x7F800000u : (LT == DT_BF16 ? 0x7F80u : 0x7C00u);
    float best;
    bool low, nan;
    if constexpr (LT == DT_F32) {
        int32_t top = INT32_MIN;
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t w = (int32_t)buf[k][i];
                top = w > top ? w : top;
            }
        best = __builtin_bit_cast(float, top);
        low = top < 0;
        nan = top > (int32_t)kInf;
    } else {
        i16x2 top = {INT16_MIN, INT16_MIN};
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t w = buf[k][i];
                top = __builtin_elementwise_max(top, __builtin_bit_cast(i16x2, w));
            }
        const int lo = top.x, hi = top.y;
        const int t = hi > lo ? hi : lo;
        best = bits_f32<LT>((uint32_t)t & 0xFFFFu);
        low = t < 0;
        nan = t > (int)kInf;
    }
    if (__ballot(low)) {
        if constexpr (LT == DT_F32) {
            uint32_t top = 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = buf[k][i];
                    top = w < top ? w : top;
                }
            if (low) {
                best = __builtin_bit_cast(float, top);
                nan = top > (0x80000000u | kInf);
            }
        } else {
            u16x2 top = {0xFFFFu, 0xFFFFu};
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = buf[k][i];
                    top = __builtin_elementwise_min(top, __builtin_bit_cast(u16x2, w));
                }
            const uint32_t lo = top.x, hi = top.y;
            const uint32_t t = hi < lo ? hi : lo;
            if (low) {
                best = bits_f32<LT>(t);
                nan = t > (0x8000u | kInf);
            }
        }
    }
    if (__ballot(nan)) {
        forget(buf);
        best = -__builtin_inff();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            float x[LT == DT_F32 ? 4 : 8];
            unpack<LT>(buf[k], x);
#pragma unroll
            for (int u = 0; u < (LT == DT_F32 ? 4 : 8); ++u) best = __builtin_fmaxf(best, x[u]);
        }
    }
    return best;
}

// Whether a word of 16-bit logits holds -inf (or a NaN of the negative sign).
template <int LT>
__device__ __forceinline__ bool has_low(const u32x4& w) {
    u16x2 top = {0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t u = w[i];
        top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, u));
    }
    const uint32_t lo = top.x, hi = top.y;
    return (hi > lo ? hi : lo) >= (LT == DT_BF16 ? 0xFF80u : 0xFC00u);
}

// The sums over the first `live` words of a lane's logits, and over the wave the
// number of those >= thr (one compare each; the ballot is counted on the scalar
// unit).  CLAMP keeps a -inf or NaN logit at weight 0 and contribution 0; without
// it (every word live) those make t2 NaN and the caller asks again.
template <int LT, int U, bool COUNT, bool CLAMP>
__device__ __forceinline__ void add_up(u32x4 (&buf)[U], int live, float base,
                                       const float (&thr)[U], float& s, float& t2,
                                       uint32_t& wcnt) {
    constexpr int VW = LT == DT_F32 ? 4 : 8;
    s = 0.0f;
    t2 = 0.0f;
    forget(buf);
#pragma unroll
    for (int k = 0; k < U; ++k) {
        if (!CLAMP || k < live) {                    // uniform
            float x[VW];
            unpack<LT>(buf[k], x);
#pragma unroll
            for (int u = 0; u < VW; ++u) {
                float t = __builtin_fmaf(x[u], kLog2e, base);
                if constexpr (CLAMP) t = __builtin_fmaxf(t, -256.0f);
                const float e = fast_exp2(t);
                s += e;
                t2 = __builtin_fmaf(e, t, t2);
                if constexpr (COUNT) wcnt += (uint32_t)__popcll(__ballot(x[u] >= thr[k]));
            }
        }
        __builtin_amdgcn_sched_barrier(0);           // registers: one word's logits
    }
}

// One block per (item, vocabulary slice).  Dense: item = candidate * max_len
// + position, its own logits row, token drafts[item].  TREE: item = group *
// nodes + u, token tree_tokens[item]; it is judged when u < tree_len[group]
// and its parent is a node of the group (or none), and its logits row is
// 1 + parent within the group's 1 + nodes rows.
// ONE: a slice is one step, and the kernel requests no other (requests for the
// two steps behind it, all lanes on the last word, cost as much as the rows:
// 8192 rows of 1000 bf16 40.0 us with them, 18.6 without; of 8192 bf16 32.6 and
// 28.0; one row of 500 6.9 and 6.1).
template <int LT, bool TREE, bool ONE>
__global__ __launch_bounds__(kRowThreads, 5) void verify_rows_kernel(
    const void* __restrict__ logits, int64_t row_stride, const int32_t* __restrict__ drafts,
    const int32_t* __restrict__ draft_len, int max_len, int vocab, int slice_vecs, int n_slices,
    int64_t n_items, Partial* __restrict__ partial, const int32_t* __restrict__ tree_parent,
    const int32_t* __restrict__ tree_len, int nodes) {
    constexpr int VW = (LT == DT_F32) ? 4 : 8;      // elements per 16-byte load
    constexpr int ES = (LT == DT_F32) ? 4 : 2;      // element size
    constexpr int U = kNV;
    int item = blockIdx.x;
    const int slice = blockIdx.y;
    const int tid = threadIdx.x;
    int cand = 0, pos = 0;
    if constexpr (!TREE) {
        // Blocks go to the XCDs in turn, and of ragged drafts the first
        // positions are judged most often: a candidate's positions are dealt
        // out from a place of its own, so that no XCD has position 0 of all.
        cand = item / max_len;
        pos = (int)(((uint32_t)(item - cand * max_len) + ((uint32_t)cand * 0x9E3779B1u >> 16)) %
                    (uint32_t)max_len);
        item = cand * max_len + pos;
    }
    int64_t row = item;
    // The row's token and the loads that decide whether the row is judged
    // are requested together (every index is in range either way).
    const int tok = drafts[item];
    if constexpr (TREE) {
        const int g = item / nodes, u = item - g * nodes;
        const int tl = tree_len[g];
        const int par = tree_parent[item];
        if (u >= tl || par < -1 || par >= nodes) return;   // uniform over the block
        row = (int64_t)g * (nodes + 1) + 1 + par;
    } else {
        int len = draft_len ? draft_len[cand] : max_len;
        len = len < 0 ? 0 : (len > max_len ? max_len : len);
        if (pos >= len) return;          // uniform over the block
    }

    const bool valid = tok >= 0 && tok < vocab;
    const char* rowp = (const char*)logits + row * row_stride * ES;
    const int tk = valid ? tok : -1;                 // -1: the count is unused

    // The row in 16-byte words of memory: `head` elements before the first,
    // `words` of them, the rest behind the last.  This block's share.
    int head = (int)(((0 - (uintptr_t)rowp) & 15) / ES);
    head = head < vocab ? head : vocab;
    const int words = (vocab - head) / VW;
    const int w0 = slice * slice_vecs;
    const int left = words - w0;
    const int nvec = left < 0 ? 0 : (left < slice_vecs ? left : slice_vecs);
    const int v0 = head + w0 * VW;                   // first element of the share's words
    const u32x4* vp = (const u32x4*)(rowp + (int64_t)v0 * ES);
    const int steps = (nvec + U * kRowThreads - 1) / (U * kRowThreads);

    auto load = [&](u32x4 (&buf)[U], int s) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int i = tid + (s * U + k) * kRowThreads;
            buf[k] = __builtin_nontemporal_load(vp + (i < nvec ? i : nvec - 1));
        }
    };
    u32x4 ba[U], bb[U];
    if (steps > 0) load(ba, 0);
    // One element more for some lanes of the first wave: the row's head (first
    // slice), what follows its last word (last slice), and the elements of the
    // judged token's word left of it.
    const int tail0 = head + words * VW;
    const int dword = v0 + (tk < v0 ? 0 : (tk - v0) / VW * VW);
    const bool is_head = slice == 0 && tid < head;
    const bool is_tail = slice == n_slices - 1 && tid >= 8 && tail0 + tid - 8 < vocab;
    const bool is_tie = tid >= 16 && tid < 16 + VW && tk >= v0 && tk < v0 + nvec * VW &&
                        dword + tid - 16 < tk;
    const int at = is_head ? tid : (is_tail ? tail0 + tid - 8 : (is_tie ? dword + tid - 16 : 0));
    const float xe = load_one<LT>(rowp, at);
    const float xd_raw = load_one<LT>(rowp, valid ? tok : 0);
    __builtin_amdgcn_sched_barrier(0);
    // The rank count's thresholds, left of d and from d on.
    const float xd = valid ? xd_raw : __builtin_inff();
    const float thr_lo = xd, thr_hi = next_up(xd);

    State st;
    uint32_t wcnt = 0;                               // per wave
    // Uniform: the clamped form first.  fp32 logits always take it (their read
    // leaves the vector units time, and the kernel is half as long); of 16-bit
    // ones a wave that has met a logit that needs it, which a masked row's first
    // words tell, so that it pays for the clamp alone (7.5 and not 6.5
    // instructions a logit) and not for both forms.
    bool masked = LT == DT_F32;
    const int wfirst = __builtin_amdgcn_readfirstlane(tid & ~63);
    auto absorb = [&](u32x4 (&buf)[U], int s) {
        // Words of this wave's lanes in the share, all of its lanes' or not.
        const int first = wfirst + s * (U * kRowThreads);
        const int live = (nvec - first + kRowThreads - 1) / kRowThreads;
        if (live <= 0) return;                       // uniform over the wave
        const bool whole = first + 63 + (U - 1) * kRowThreads < nvec;
        if (!whole) {                                // -inf past the last word
            constexpr uint32_t kNone = LT == DT_F32    ? 0xFF800000u
                                       : LT == DT_BF16 ? 0xFF80FF80u
                                                       : 0xFC00FC00u;
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (tid + (s * U + k) * kRowThreads >= nvec)
                    buf[k] = u32x4{kNone, kNone, kNone, kNone};
        }
        const float top = lane_max<LT, U>(buf);
        const float m2 = __builtin_fmaxf(st.m2, top * kLog2e);
        raise_to(st, m2);
        const float base = base_of(m2);
        float thr[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            thr[k] = v0 + (tid + (s * U + k) * kRowThreads + 1) * VW <= tk ? thr_lo : thr_hi;
        if constexpr (LT != DT_F32)
            if (s == 0 && __ballot(has_low<LT>(buf[0]))) masked = true;
        float s1, t1;
        // No logit of the wave reaches the judged one: nothing to count.
        const bool count = __ballot(top >= xd) != 0;
        if (LT == DT_F32 || masked || !whole) {
            if (count) add_up<LT, U, true, true>(buf, live, base, thr, s1, t1, wcnt);
            else add_up<LT, U, false, true>(buf, live, base, thr, s1, t1, wcnt);
        } else {
            if (count) add_up<LT, U, true, false>(buf, U, base, thr, s1, t1, wcnt);
            else add_up<LT, U, false, false>(buf, U, base, thr, s1, t1, wcnt);
            if (__ballot(t1 != t1)) {
                masked = true;
                add_up<LT, U, false, true>(buf, U, base, thr, s1, t1, wcnt);
            }
        }
        st.s += s1;
        st.t2 += t1;
    };
    if constexpr (ONE) {
        absorb(ba, 0);
    } else {
        // Loads past the last step all fall on the share's last word.
        for (int s = 0; s < steps; s += 2) {
            load(bb, s + 1);
            __builtin_amdgcn_sched_barrier(0);
            absorb(ba, s);
            load(ba, s + 2);
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < steps) absorb(bb, s + 1);
        }
    }

    int cnt = 0;
    if (is_head || is_tail) {
        const float m2 = __builtin_fmaxf(st.m2, xe * kLog2e);
        raise_to(st, m2);
        const float t = __builtin_fmaxf(__builtin_fmaf(xe, kLog2e, base_of(m2)), -256.0f);
        const float e = fast_exp2(t);
        st.s += e;
        st.t2 = __builtin_fmaf(e, t, st.t2);
        cnt = xe >= (at < tk ? thr_lo : thr_hi) ? 1 : 0;
    } else if (is_tie) {
        // The word holding d was counted with x > x_d throughout; its
        // elements left of d equal to x_d also rank above d.
        cnt = xe == xd ? 1 : 0;
    }

    // Block sums in a fixed order.
    raise_to(st, wave_max_f(st.m2));
    const float ws = wave_sum_f(st.s), wt = wave_sum_f(st.t2);
    const int wc = wave_sum_i(cnt) + (int)wcnt;
    __shared__ Partial s_w[kRowWaves];
    if ((tid & 63) == 0) s_w[tid >> 6] = Partial{st.m2, ws, wt, wc};
    __syncthreads();
    if (tid == 0) {
        State a;
        int c = 0;
        merge_all<kRowWaves>(a, c, s_w);
        partial[(int64_t)slice * n_items + item] = Partial{a.m2, a.s, a.t2, c};
    }
}

constexpr int kFinThreads = 512;
constexpr int kFinChunkRows = 4096;   // (candidate, position) rows per LDS chunk
constexpr int kFinChunkCands = 1024;  // candidates per LDS chunk

__device__ __forceinline__ uint64_t bits_upto(int x) {  // bits 0..x set (x may be -1)
    return (x >= 63) ? ~0ull : ((x < 0) ? 0ull : ((1ull << (x + 1)) - 1ull));
}

// Merge of an item's slice partials in slice order.  Loads go out in
// batches of kMergeBatch (clamped indices, no branch around a load, so none
// waits for the one before it); partials past the last take no part (merged as
// empty ones they cost the finalize of 256 x 8 rows of one slice 8.5 us against
// 5.8).
constexpr int kMergeBatch = 8;

__device__ __forceinline__ void merge_partials(const Partial* p, int64_t n_items, int n_slices,
                                               State* st, int* cnt) {
    if (n_slices == 1) {
        const Partial q = *p;
        *st = State{q.m2, q.s, q.t2};
        *cnt = q.cnt;
        return;
    }
    State a;
    int c = 0;
    for (int s0 = 0; s0 < n_slices; s0 += kMergeBatch) {
        Partial q[kMergeBatch];
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u)
            q[u] = p[((s0 + u < n_slices) ? s0 + u : n_slices - 1) * n_items];
        merge_all(a, c, q, n_slices - s0);
    }
    *st = a;
    *cnt = c;
}

// Row statistics of one item from its merged partials: the entropy score
// and the rank of the judged token; bits em | ent<<1 | topk<<2.
__device__ __forceinline__ uint8_t item_bits(const State& a, int cnt, int tok, int vocab,
                                             const GateParams& gp, float* score, int* rank) {
    const float e_nats = __logf(a.s) - (kLn2 * a.t2) / a.s;
    *score = e_nats * gp.ent_scale;
    const bool valid = tok >= 0 && tok < vocab;
    *rank = valid ? cnt : vocab;
    return (uint8_t)((valid && *rank == 0 ? 1 : 0) | (*score > gp.gamma ? 2 : 0) |
                     (valid && *rank < gp.topk ? 4 : 0));
}

// First candidate with the largest n in the block (all threads call it).
// A thread's (n, i) is one key, n + 1 above the complemented index, so the
// largest key has the largest n and then the smallest i (a thread that saw
// no candidate has n = -1, below every real one); each wave takes its
// maximum with lane swaps and thread 0 the waves'.
__device__ void group_best(int best_n, int best_i, int32_t* out) {
    __shared__ uint64_t s_w[kFinThreads / 64];
    uint64_t key = ((uint64_t)(uint32_t)(best_n + 1) << 32) |
                   (uint64_t)(0xFFFFFFFFu - (uint32_t)best_i);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor(key, off, 64);
        key = o > key ? o : key;
    }
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t m = s_w[0];
#pragma unroll
        for (int w = 1; w < kFinThreads / 64; ++w) m = s_w[w] > m ? s_w[w] : m;
        *out = (int32_t)(0xFFFFFFFFu - (uint32_t)m);
    }
}

// Dense finalize, one block per group, in chunks of candidates.  Phase 1
// gives every (candidate, position) row a thread: the row's bits into LDS
// and its exact-match bit into the candidate's 64-bit mask.  Phase 2 gives
// every row a thread again: the mismatches in its window from the mask (one
// popcount), its gate bit (Alg. 4's cascade) into the candidate's gate
// mask.  Phase 3 gives every candidate a thread: the leading run of the gate
// mask is the accepted length.  No thread walks a draft's positions, so the
// cost does not grow with the draft length.
__global__ __launch_bounds__(kFinThreads) void verify_finalize_kernel(
    const Partial* __restrict__ partial, int n_slices, const int32_t* __restrict__ drafts,
    const int32_t* __restrict__ draft_len, int max_len, int vocab, int group_size,
    GateParams gp, int32_t* __restrict__ out_accept_len, int32_t* __restrict__ out_best,
    float* __restrict__ out_gate_score, uint8_t* __restrict__ out_masks,
    int32_t* __restrict__ out_rank) {
    __shared__ uint8_t s_bits[kFinChunkRows];     // em | ent<<1 | topk<<2 per row
    __shared__ uint8_t s_len[kFinChunkCands];     // clamped draft length per candidate
    __shared__ uint64_t s_em[kFinChunkCands];     // exact-match bit per position
    __shared__ uint64_t s_gate[kFinChunkCands];   // gate bit per position
    const int g = blockIdx.x;
    const int64_t n_items = (int64_t)gridDim.x * group_size * max_len;
    const int by_rows = kFinChunkRows / max_len;
    const int chunk_cands = by_rows < kFinChunkCands ? by_rows : kFinChunkCands;
    const uint64_t in_draft = bits_upto(max_len - 1);
    for (int cl = threadIdx.x; cl < kFinChunkCands; cl += kFinThreads) {
        s_em[cl] = 0ull;
        s_gate[cl] = 0ull;
    }
    __syncthreads();
    int best_n = -1, best_i = 0;
    for (int cc0 = 0; cc0 < group_size; cc0 += chunk_cands) {
        const int ncc = (group_size - cc0 < chunk_cands) ? group_size - cc0 : chunk_cands;
        const int rows = ncc * max_len;
        // Phase 1: the row statistics.
        for (int r = threadIdx.x; r < rows; r += kFinThreads) {
            const int cl = r / max_len, jj = r - cl * max_len;
            const int c = g * group_size + cc0 + cl;
            const int64_t row = (int64_t)c * max_len + jj;
            // Every load of the row first (the partials of a position past
            // the draft were not written and are not used).
            int len = draft_len ? draft_len[c] : max_len;
            const int tok = drafts[row];
            State st;
            int cnt;
            merge_partials(partial + row, n_items, n_slices, &st, &cnt);
            len = len < 0 ? 0 : (len > max_len ? max_len : len);
            uint8_t bits = 0;
            float score = 0.0f;
            int rank = vocab;
            if (jj < len) bits = item_bits(st, cnt, tok, vocab, gp, &score, &rank);
            if (out_gate_score) out_gate_score[row] = score;
            if (out_rank) out_rank[row] = rank;
            s_bits[r] = bits;
            if (jj == 0) s_len[cl] = (uint8_t)len;
            if (bits & 1) atomicOr((unsigned long long*)&s_em[cl], 1ull << jj);
        }
        __syncthreads();
        // Phase 2: each row's window and gate.  Mismatches are 1 - B_em
        // inside the draft (every position past its length included) and
        // W padding ones past the last position.
        for (int r = threadIdx.x; r < rows; r += kFinThreads) {
            const int cl = r / max_len, jj = r - cl * max_len;
            const uint8_t b = s_bits[r];
            const uint64_t notem = ~s_em[cl] & in_draft;
            const int hi = jj + gp.window;
            const int in_hi = hi < max_len - 1 ? hi : max_len - 1;
            const uint64_t range = bits_upto(in_hi) & ~bits_upto(jj);
            const int mis = __popcll(notem & range) + (hi > max_len - 1 ? hi - (max_len - 1) : 0);
            const bool con = mis <= gp.tau;
            const bool bem = b & 1, bent = (b >> 1) & 1, btk = (b >> 2) & 1;
            const bool gate = (jj < (int)s_len[cl]) && (bem || (bent && (btk || con)));
            if (out_masks) {
                const int64_t row = (int64_t)(g * group_size + cc0 + cl) * max_len + jj;
                out_masks[row] = (uint8_t)((int)bem | ((int)bent << 1) | ((int)btk << 2) |
                                           ((int)con << 3) | ((int)gate << 4));
            }
            if (gate) atomicOr((unsigned long long*)&s_gate[cl], 1ull << jj);
        }
        __syncthreads();
        // Phase 3: the accepted length, and the masks cleared for the next
        // chunk (each candidate's words by its own thread).
        for (int cl = threadIdx.x; cl < ncc; cl += kFinThreads) {
            const uint64_t open = ~s_gate[cl];
            const int n = open == 0ull ? 64 : __builtin_ctzll(open);
            out_accept_len[g * group_size + cc0 + cl] = n;
            if (n > best_n) {
                best_n = n;
                best_i = cc0 + cl;
            }
            s_em[cl] = 0ull;
            s_gate[cl] = 0ull;
        }
        __syncthreads();
    }
    group_best(best_n, best_i, out_best + g);
}

// Tree variant, one block per group.  Phase 1 gives every tree node of the
// group a thread (bits, score and rank into LDS).  Then every (draft,
// position) row gets a thread in three phases: its node through Gamma and
// whether that node is judged (into the draft's 64-bit mask); the draft's
// length, the leading run of that mask, and the row's bits and outputs
// (exact-match bit into the draft's mask); its window and gate bit, as in
// the dense finalize.  Last, every draft a thread for the leading run of its
// gate mask.
__global__ __launch_bounds__(kFinThreads) void verify_finalize_tree_kernel(
    const Partial* __restrict__ partial, int n_slices, const int32_t* __restrict__ tree_tokens,
    const int32_t* __restrict__ tree_parent, const int32_t* __restrict__ tree_len,
    const int32_t* __restrict__ gamma, int max_len, int vocab, int group_size, GateParams gp,
    int32_t* __restrict__ out_accept_len, int32_t* __restrict__ out_best,
    float* __restrict__ out_gate_score, uint8_t* __restrict__ out_masks,
    int32_t* __restrict__ out_rank) {
    __shared__ uint8_t s_bits[kMaxNodes];       // em | ent<<1 | topk<<2 | judged<<3 per node
    __shared__ float s_score[kMaxNodes];
    __shared__ int32_t s_rank[kMaxNodes];
    __shared__ int16_t s_node[kMaxNodes];       // per row: its judged node, else -1
    __shared__ uint8_t s_rbits[kMaxNodes];      // per row: its node's bits inside the draft
    __shared__ uint64_t s_run[kMaxGroup];       // per draft: positions with a judged node
    __shared__ uint64_t s_em[kMaxGroup];        // per draft: exact-match bits
    __shared__ uint64_t s_gate[kMaxGroup];      // per draft: gate bits
    __shared__ uint8_t s_len[kMaxGroup];        // per draft: its length
    const int g = blockIdx.x;
    const int nodes = group_size * max_len;
    const int64_t n_items = (int64_t)gridDim.x * nodes;
    const int L = tree_len[g] < nodes ? tree_len[g] : nodes;
    const uint64_t in_draft = bits_upto(max_len - 1);
    for (int cl = threadIdx.x; cl < group_size; cl += kFinThreads) {
        s_run[cl] = 0ull;
        s_em[cl] = 0ull;
        s_gate[cl] = 0ull;
    }
    for (int u = threadIdx.x; u < L; u += kFinThreads) {
        const int item = g * nodes + u;
        // Every load of the node first (the partials of a node that is not
        // judged were not written and are not used).
        const int tok = tree_tokens[item];
        const int par = tree_parent[item];
        State st;
        int cnt;
        merge_partials(partial + item, n_items, n_slices, &st, &cnt);
        uint8_t bits = 0;
        float score = 0.0f;
        int rank = vocab;
        // u < L: the node exists; it is judged when its parent is in range
        // (the rows kernel's test for the same node).
        if (par >= -1 && par < nodes) bits = 8 | item_bits(st, cnt, tok, vocab, gp, &score, &rank);
        s_bits[u] = bits;
        s_score[u] = score;
        s_rank[u] = rank;
    }
    __syncthreads();
    // Rows: the node of each draft position, and whether it is judged.
    for (int r = threadIdx.x; r < nodes; r += kFinThreads) {
        const int cl = r / max_len, jj = r - cl * max_len;
        const int u = gamma[(int64_t)(g * group_size + cl) * max_len + jj];
        const bool judged = u >= 0 && u < L && (s_bits[u] & 8);
        s_node[r] = judged ? (int16_t)u : (int16_t)-1;
        if (judged) atomicOr((unsigned long long*)&s_run[cl], 1ull << jj);
    }
    __syncthreads();
    // Rows: a draft's length is its leading run of judged positions; the
    // bits and outputs of the positions inside it.
    for (int r = threadIdx.x; r < nodes; r += kFinThreads) {
        const int cl = r / max_len, jj = r - cl * max_len;
        const uint64_t unjudged = ~s_run[cl];
        const int len = unjudged == 0ull ? 64 : __builtin_ctzll(unjudged);
        const bool inside = jj < len;
        const int u = s_node[r];
        const uint8_t b = inside ? s_bits[u] : 0;
        const int64_t o = (int64_t)(g * group_size + cl) * max_len + jj;
        if (out_gate_score) out_gate_score[o] = inside ? s_score[u] : 0.0f;
        if (out_rank) out_rank[o] = inside ? s_rank[u] : vocab;
        s_rbits[r] = b;
        if (jj == 0) s_len[cl] = (uint8_t)len;
        if (b & 1) atomicOr((unsigned long long*)&s_em[cl], 1ull << jj);
    }
    __syncthreads();
    // Rows: window and gate.
    for (int r = threadIdx.x; r < nodes; r += kFinThreads) {
        const int cl = r / max_len, jj = r - cl * max_len;
        const uint8_t b = s_rbits[r];
        const uint64_t notem = ~s_em[cl] & in_draft;
        const int hi = jj + gp.window;
        const int in_hi = hi < max_len - 1 ? hi : max_len - 1;
        const uint64_t range = bits_upto(in_hi) & ~bits_upto(jj);
        const int mis = __popcll(notem & range) + (hi > max_len - 1 ? hi - (max_len - 1) : 0);
        const bool con = mis <= gp.tau;
        const bool bem = b & 1, bent = (b >> 1) & 1, btk = (b >> 2) & 1;
        const bool gate = (jj < (int)s_len[cl]) && (bem || (bent && (btk || con)));
        if (out_masks) {
            const int64_t o = (int64_t)(g * group_size + cl) * max_len + jj;
            out_masks[o] = (uint8_t)((int)bem | ((int)bent << 1) | ((int)btk << 2) |
                                     ((int)con << 3) | ((int)gate << 4));
        }
        if (gate) atomicOr((unsigned long long*)&s_gate[cl], 1ull << jj);
    }
    __syncthreads();
    int best_n = -1, best_i = 0;
    for (int cl = threadIdx.x; cl < group_size; cl += kFinThreads) {
        const uint64_t open = ~s_gate[cl];
        const int n = open == 0ull ? 64 : __builtin_ctzll(open);
        out_accept_len[g * group_size + cl] = n;
        if (n > best_n) {
            best_n = n;
            best_i = cl;
        }
    }
    group_best(best_n, best_i, out_best + g);
}

struct Plan {
    int n_slices;
    int slice_vecs;                // 16-byte words per slice: whole steps of a block
};

constexpr int kStepVecs = kRowThreads * kNV;
// Slices: at most 8 steps (128 KiB; longer ones leave the last blocks of a large
// batch alone; 2 to 16 steps within 2 % of each other).  A small batch is cut
// finer, to 4096 slices of two steps or more, since rows of a ragged batch or
// of a trie may be dead (64 + 16 drafts of 8, 152064 bf16, 7 tenths judged:
// 24.8 us with 4 slices a row, 21.8 with 7, 23.4 with 10), and to one step each
// only up to 512 of them (16 x 6 ragged rows of 128256 bf16: 7.8 us in slices
// of one step, 7.3 of two).  Rows shorter than 8 steps are cut to 2048 slices
// only, since each costs a start and an end (256 x 8 rows whole and in two slices,
// dense / ragged: 20000 bf16 24.9 / 19.7 us and 28.2 / 22.4, 32000 30.4 / 24.1 and
// 33.5 / 26.4, 50257 42.9 / 30.2 and 45.2 / 32.1; 64 x 14 rows of 32000 18.2 / 16.8
// and 18.9 / 15.6).
constexpr int64_t kSliceSteps = 8, kFillBlocks = 4096, kFillShort = 2048, kFillSingle = 512;

// The most slices of a row, whatever the logits' type: one step of 16-bit
// logits each.  The workspace holds one partial for each of them.
int most_slices(int vocab) { return (int)(((int64_t)vocab + 8 * kStepVecs - 1) / (8 * kStepVecs)); }

Plan make_plan(int logits_dtype, int64_t n_items, int vocab) {
    const int vw = logits_dtype == DT_F32 ? 4 : 8;
    const int64_t steps = ((int64_t)vocab + (int64_t)vw * kStepVecs - 1) / ((int64_t)vw * kStepVecs);
    const int64_t by_size = (steps + kSliceSteps - 1) / kSliceSteps;
    const int64_t pairs = (steps + 1) / 2;
    const int64_t blocks = steps < kSliceSteps ? kFillShort : kFillBlocks;
    const int64_t fill = (blocks + n_items - 1) / n_items;
    const int64_t single = (kFillSingle + n_items - 1) / n_items;
    int64_t n = fill < pairs ? fill : pairs;
    n = n > by_size ? n : by_size;
    n = n > single ? n : single;
    const int64_t most = most_slices(vocab);
    n = n < most ? n : most;
    const int64_t per = (steps + n - 1) / n;
    return Plan{(int)((steps + per - 1) / per), (int)(per * kStepVecs)};
}

template <int LT, bool TREE>
hipError_t launch_rows_t(const void* logits, int64_t row_stride, const int32_t* tokens,
                         const int32_t* draft_len, int64_t n_items, int max_len, int vocab,
                         const Plan& pl, Partial* part, const int32_t* tree_parent,
                         const int32_t* tree_len, int nodes, hipStream_t stream) {
    const dim3 grid((unsigned)n_items, (unsigned)pl.n_slices);
    auto kern = pl.slice_vecs == kStepVecs ? verify_rows_kernel<LT, TREE, true>
                                           : verify_rows_kernel<LT, TREE, false>;
    hipLaunchKernelGGL(kern, grid, dim3(kRowThreads), 0, stream, logits, row_stride, tokens,
                       draft_len, max_len, vocab, pl.slice_vecs, pl.n_slices, n_items, part,
                       tree_parent, tree_len, nodes);
    return hipGetLastError();
}

template <bool TREE>
hipError_t launch_rows(const void* logits, int logits_dtype, int64_t row_stride,
                       const int32_t* tokens, const int32_t* draft_len, int64_t n_items,
                       int max_len, int vocab, const Plan& pl, Partial* part,
                       const int32_t* tree_parent, const int32_t* tree_len, int nodes,
                       hipStream_t stream) {
    switch (logits_dtype) {
        case DT_F32:
            return launch_rows_t<DT_F32, TREE>(logits, row_stride, tokens, draft_len, n_items,
                                               max_len, vocab, pl, part, tree_parent, tree_len,
                                               nodes, stream);
        case DT_F16:
            return launch_rows_t<DT_F16, TREE>(logits, row_stride, tokens, draft_len, n_items,
                                               max_len, vocab, pl, part, tree_parent, tree_len,
                                               nodes, stream);
        default:
            return launch_rows_t<DT_BF16, TREE>(logits, row_stride, tokens, draft_len, n_items,
                                                max_len, vocab, pl, part, tree_parent, tree_len,
                                                nodes, stream);
    }
}

}  // namespace

size_t verify_workspace_bytes(int n_cand, int max_len, int vocab) {
    return (size_t)n_cand * (size_t)max_len * (size_t)most_slices(vocab) * sizeof(Partial);
}

size_t verify_tree_workspace_bytes(int n_cand, int max_len, int vocab, int n_groups) {
    // One partial per (tree node, slice); a group has at most n_cand / n_groups
    // * max_len nodes, so the dense bound is also the tree bound.
    (void)n_groups;
    return verify_workspace_bytes(n_cand, max_len, vocab);
}

hipError_t launch_verify(const void* logits, int logits_dtype, int64_t row_stride,
                         const int32_t* drafts, const int32_t* draft_len, int n_cand,
                         int max_len, int vocab, int n_groups, const GateParams& gp,
                         int32_t* out_accept_len, int32_t* out_best, float* out_gate_score,
                         uint8_t* out_masks, int32_t* out_rank, void* workspace,
                         hipStream_t stream) {
    if (n_cand == 0) return hipSuccess;
    const Plan pl = make_plan(logits_dtype, (int64_t)n_cand * max_len, vocab);
    Partial* part = (Partial*)workspace;
    hipError_t e = launch_rows<false>(logits, logits_dtype, row_stride, drafts, draft_len,
                                      (int64_t)n_cand * max_len, max_len, vocab, pl, part,
                                      nullptr, nullptr, 0, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(verify_finalize_kernel, dim3((unsigned)n_groups), dim3(kFinThreads), 0,
                       stream, part, pl.n_slices, drafts, draft_len, max_len, vocab,
                       n_cand / n_groups, gp, out_accept_len, out_best, out_gate_score,
                       out_masks, out_rank);
    return hipGetLastError();
}

hipError_t launch_verify_tree(const void* logits, int logits_dtype, int64_t row_stride,
                              const int32_t* tree_tokens, const int32_t* tree_parent,
                              const int32_t* tree_len, const int32_t* gamma, int n_cand,
                              int max_len, int vocab, int n_groups, const GateParams& gp,
                              int32_t* out_accept_len, int32_t* out_best, float* out_gate_score,
                              uint8_t* out_masks, int32_t* out_rank, void* workspace,
                              hipStream_t stream) {
    if (n_cand == 0) return hipSuccess;
    const Plan pl = make_plan(logits_dtype, (int64_t)n_cand * max_len, vocab);
    Partial* part = (Partial*)workspace;
    const int gs = n_cand / n_groups;
    const int nodes = gs * max_len;
    hipError_t e = launch_rows<true>(logits, logits_dtype, row_stride, tree_tokens, nullptr,
                                     (int64_t)n_groups * nodes, max_len, vocab, pl, part,
                                     tree_parent, tree_len, nodes, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(verify_finalize_tree_kernel, dim3((unsigned)n_groups), dim3(kFinThreads),
                       0, stream, part, pl.n_slices, tree_tokens, tree_parent, tree_len, gamma,
                       max_len, vocab, gs, gp, out_accept_len, out_best, out_gate_score,
                       out_masks, out_rank);
    return hipGetLastError();
}

}  // namespace sense
