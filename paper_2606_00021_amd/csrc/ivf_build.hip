// Datastore construction for the inverted file (Sec. 3.2 Eq. 7; App.
// implementation details: IVF-PQ, nlist 4096, pq_m 16 over 64-dim keys):
//   ivf_assign: every key's list = its most similar centroid, a contraction
//     of N keys with nlist centroids on the matrix cores;
//   pq_encode: code j of key i = nearest codebook entry of the j-th slice of
//     the residual key - centroid[list].
#include "internal.h"

namespace sense {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int KT>
__device__ __forceinline__ float elem_f32(uint32_t bits) {
    if constexpr (KT == DT_F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
    return __builtin_bit_cast(float, bits << 16);
}

// ------------------------------------------------------------- assignment
// The better of (b, r) and (ob, orow): the larger score, the lower row on a tie.
__device__ __forceinline__ void take_better(float& b, int& r, float ob, int orow) {
    const bool up = ob > b || (ob == b && orow < r);
    b = up ? ob : b;
    r = up ? orow : r;
}

// The list of one key (the same in every lane) in plain fp32, the definition
// centroid by centroid, by a whole wave: for keys that the matrix-core path
// leaves out.  A lane takes every 64th centroid; a key whose cosine scale is 0
// (its squared norm overflows or vanishes in fp32) scores 0 or NaN, and the
// first 0 ends the search.  Bound: the centroids' read by one wave, 1 MiB of
// them at 4096 x 64 (one lane alone walked nlist * d / 2 dependent steps: 262144
// keys, one of them zero, 11.9 ms).
template <int KT>
__device__ __attribute__((noinline)) int assign_one(const uint16_t* __restrict__ row, int d,
                                                    const float* __restrict__ centroids,
                                                    int nlist, int cosine) {
    const int lane = threadIdx.x & 63;
    float best = -__builtin_inff();
    int arg = 0;
    for (int l0 = 0; l0 < nlist; l0 += 64) {
        const int l = l0 + lane;
        const float* c = centroids + (int64_t)(l < nlist ? l : 0) * d;
        float a0 = 0.0f, a1 = 0.0f, cn = 0.0f, xn = 0.0f;
        for (int t = 0; t < d; t += 8) {             // d is a multiple of 8
            const u32x4 w = *(const u32x4*)(row + t);
            float cv[8];
            __builtin_memcpy(cv, c + t, 32);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x0 = elem_f32<KT>(w[j] & 0xFFFFu), x1 = elem_f32<KT>(w[j] >> 16);
                a0 = __builtin_fmaf(x0, cv[2 * j], a0);
                a1 = __builtin_fmaf(x1, cv[2 * j + 1], a1);
                cn = __builtin_fmaf(cv[2 * j], cv[2 * j], cn);
                cn = __builtin_fmaf(cv[2 * j + 1], cv[2 * j + 1], cn);
                xn = __builtin_fmaf(x0, x0, xn);
                xn = __builtin_fmaf(x1, x1, xn);
            }
        }
        const float inv_x = (xn > 0.0f) ? 1.0f / __builtin_sqrtf(xn) : 0.0f;
        float s = a0 + a1;
        if (cosine) s = (s * ((cn > 0.0f) ? 1.0f / __builtin_sqrtf(cn) : 0.0f)) * inv_x;
        if (l < nlist && s > best) {
            best = s;
            arg = l;
        }
        if (cosine && inv_x == 0.0f && __ballot(best == 0.0f)) break;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        take_better(best, arg, __shfl_xor(best, off, 64), __shfl_xor(arg, off, 64));
    return arg;
}

// out_list of the keys that `mask`'s lanes hold (a lane's key is row `i` of the
// store), a wave at a time for each.
template <int KT>
__device__ __forceinline__ void assign_rest(uint64_t mask, int64_t i,
                                            const uint16_t* __restrict__ keys, int64_t ld, int d,
                                            const float* __restrict__ centroids, int nlist,
                                            int cosine, int32_t* __restrict__ out_list) {
    while (mask) {
        const int src = __builtin_ctzll(mask);
        mask &= mask - 1;
        const int64_t key = __shfl(i, src, 64);
        const int l = assign_one<KT>(keys + key * ld, d, centroids, nlist, cosine);
        if ((int)(threadIdx.x & 63) == src) out_list[key] = l;
    }
}

// out_list[i] = argmax_l sim(key i, centroid l); ties to the lower l.
//
// Bound: the matrix cores and, beside them, the vector ALUs that prepare the
// centroids.  Operands are bfloat16, whose exponents are those of fp32, so that
// a value is the exact sum of its leading 8 bits, the next 8 and the rest: an
// fp32 centroid (normalised first under cosine) goes in as three parts, an fp16
// key as two, a bf16 key as it is.  Nothing is scaled and no bit of either side
// is left out; the products are exact and summed in the fp32 accumulators, the
// small parts first.  (Two fp16 parts of a scaled centroid leave up to 2^-23 of
// an element, and of one below 2^-17 of its row's largest only 2^-39 of that
// largest.)  A lane keeps the best score of its own four rows of every
// 16-centroid tile and the tile it came from (strictly greater, in ascending
// order), five instructions per four scores; at the end the lanes (and waves)
// merge per key, and four lanes settle which of the winning four rows it was,
// one row each, in fp32.
//
// Two ways to share the centroids:
//   assign_stage: a wave has its own T tiles of 16 keys; the block's waves
//     prepare the centroids together, kTileC of them per stage, into LDS in
//     A-fragment order (conflict-free 16-byte reads), double-buffered with one
//     barrier a stage.  One half of the waves prepares the next stage before
//     its products and the other half after them, so that on every SIMD one
//     wave's preparation runs beside the other's products.
//   assign_split: the waves of a block hold the same T tiles of keys, and deal
//     out the centroids, 16 at a time, each preparing its tile in registers:
//     more preparation per key, but no barrier, and 16 T keys fill a block.
//
// 4096 centroids, 64 dims, cosine: 262144 bf16 keys 2340 us with one thread per
// key on the VALU, 338 us staged (1.22 PFLOP/s of products; a large torch matrix
// product reaches 1.2 to 1.4), 561 split; 16384 keys 1614, 136 (two key tiles a
// wave) and 42 us.  fp16 keys, twice the products: 262144 587 us staged, 16384
// 53 us split.

// The sum over the G consecutive lanes of a group (G 8, 16 or 32).
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x),
                                                                 CTRL, 0xF, 0xF, false));
}
template <int G>
__device__ __forceinline__ float group_sum(float x) {
    x += dpp<0xB1>(x);                             // quad xor 1
    x += dpp<0x4E>(x);                             // quad xor 2
    x += dpp<0x141>(x);                            // half-row mirror
    if constexpr (G >= 16) x += dpp<0x140>(x);     // row mirror
    if constexpr (G >= 32) x += __shfl_xor(x, 16, 64);
    return x;
}
// x as the exact sum of three bfloat16 values (the upper halves of part[0 .. 2]):
// its leading 8 bits, the next 8, and the rest.  An infinite x is its first part.
__device__ __forceinline__ void three_parts(float x, uint32_t (&part)[3]) {
#pragma clang fp contract(off)
    asm volatile("" : "+v"(x));    // one rounded number, not the product it may come from
    part[0] = __builtin_bit_cast(uint32_t, x) & 0xFFFF0000u;
    const float r = __builtin_fabsf(x) == __builtin_inff()
                        ? 0.0f
                        : x - __builtin_bit_cast(float, part[0]);
    part[1] = __builtin_bit_cast(uint32_t, r) & 0xFFFF0000u;
    part[2] = __builtin_bit_cast(uint32_t, r - __builtin_bit_cast(float, part[1]));
}

// The upper halves of two words, that of b on top.
__device__ __forceinline__ uint32_t upper_halves(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

__device__ __forceinline__ f32x4 mfma(const u32x4& a, const u32x4& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The first part of an fp16 key's element (11 bits): its leading 8 bits, or the
// bfloat16 below where these are all of it, so that no part of a number is 0
// (which an infinite centroid element would turn into NaN).
__device__ __forceinline__ uint32_t key_part(float x) {
    const uint32_t b = __builtin_bit_cast(uint32_t, x);
    return x == 0.0f ? 0u : (b - 1u) & 0xFFFF0000u;
}

constexpr int kParts = 3;                          // of a centroid
// Parts of a key: 8 + 3 bits of an fp16 one.
template <int KT>
constexpr int kKeyParts = KT == DT_F16 ? 2 : 1;

// Keys base + 16 t + col as B fragments (k = 8 grp + 32 ks .. + 7); rows past n
// re-read row n - 1.  Bit t of the result: the products serve the key, whose
// squared norm is an ordinary number (no sum of its products overflows or
// vanishes where the definition's does not), or which is zero (every score is 0
// or NaN) or holds a NaN (every score is).
template <int KT, int KS, int T>
__device__ __forceinline__ uint32_t load_keys(const uint16_t* __restrict__ keys, int64_t base,
                                              int64_t n, int d, int64_t ld,
                                              u32x4 (&kf)[T][KS][kKeyParts<KT>]) {
    const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
    uint32_t served = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int64_t i = base + 16 * t + col;
        const uint16_t* row = keys + (i < n ? i : n - 1) * ld;
        u32x4 kw[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int e = 8 * grp + 32 * ks;
            kw[ks] = *(const u32x4*)(row + (e < d ? e : 0));
        }
        float xn = 0.0f, big = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (8 * grp + 32 * ks >= d) kw[ks] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t w = kw[ks][j];
                const float x0 = elem_f32<KT>(w & 0xFFFFu), x1 = elem_f32<KT>(w >> 16);
                xn = __builtin_fmaf(x0, x0, xn);
                xn = __builtin_fmaf(x1, x1, xn);
                big = __builtin_fmaxf(big, __builtin_fmaxf(__builtin_fabsf(x0), __builtin_fabsf(x1)));
                if constexpr (KT == DT_F16) {
                    const uint32_t b0 = key_part(x0), b1 = key_part(x1);
                    kf[t][ks][0][j] = upper_halves(b0, b1);
                    kf[t][ks][kKeyParts<KT> - 1][j] = upper_halves(
                        __builtin_bit_cast(uint32_t, x0 - __builtin_bit_cast(float, b0)),
                        __builtin_bit_cast(uint32_t, x1 - __builtin_bit_cast(float, b1)));
                } else {
                    kf[t][ks][0][j] = w;
                }
            }
        }
        xn += __shfl_xor(xn, 16, 64);
        xn += __shfl_xor(xn, 32, 64);
        big = __builtin_fmaxf(big, __shfl_xor(big, 16, 64));
        big = __builtin_fmaxf(big, __shfl_xor(big, 32, 64));
        served |= ((xn > 0x1p-100f && xn < 0x1p100f) || big == 0.0f || xn != xn) ? 1u << t : 0u;
        if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // registers: four tiles' loads
    }
    return served;
}

// The products of one centroid tile (first row l0, its parts in `a`) with T key
// tiles.
template <int KT, int KS, int T>
__device__ __forceinline__ void tile_products(int l0, const u32x4 (&a)[kParts][KS],
                                              const u32x4 (&kf)[T][KS][kKeyParts<KT>],
                                              float (&best)[T], int (&row0)[T]) {
    constexpr int KP = kKeyParts<KT>;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        // Parts p of the centroid and u of the key: a product's size falls with
        // p + u.
#pragma unroll
        for (int o = kParts + KP - 2; o >= 0; --o)
#pragma unroll
            for (int p = kParts - 1; p >= 0; --p)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if (o - p >= 0 && o - p < KP) acc = mfma(a[p][ks], kf[t][ks][o - p], acc);
        const float m = __builtin_fmaxf(__builtin_fmaxf(acc[0], acc[1]),
                                        __builtin_fmaxf(acc[2], acc[3]));
        const bool up = m > best[t];
        best[t] = up ? m : best[t];
        row0[t] = up ? l0 : row0[t];
        // Taken here: put off, the comparisons' masks would be kept (and
        // spilled) instead.
        asm volatile("" : "+v"(row0[t]));
        if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // registers: four sums
    }
}

// The best group of four rows of each key over the four lanes that hold it.
__device__ __forceinline__ void merge_lanes(float& b, int& r) {
#pragma unroll
    for (int off = 16; off < 64; off <<= 1)
        take_better(b, r, __shfl_xor(b, off, 64), __shfl_xor(r, off, 64));
}

// Which of rows r .. r + 3 is the key's best: this lane's row l of them in
// fp32, merged over the four lanes at distances step and 2 step.
template <int KT, bool COS>
__device__ __forceinline__ int settle(const uint16_t* __restrict__ row, int d,
                                      const float* __restrict__ centroids, int nlist, int l,
                                      int step) {
    const float* c = centroids + (int64_t)(l < nlist ? l : 0) * d;
    float a0 = 0.0f, a1 = 0.0f, c0 = 0.0f, c1 = 0.0f;
    for (int e = 0; e < d; e += 8) {
        const u32x4 w = *(const u32x4*)(row + e);
        float cv[8];
        __builtin_memcpy(cv, c + e, 32);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a0 = __builtin_fmaf(elem_f32<KT>(w[j] & 0xFFFFu), cv[2 * j], a0);
            a1 = __builtin_fmaf(elem_f32<KT>(w[j] >> 16), cv[2 * j + 1], a1);
            c0 = __builtin_fmaf(cv[2 * j], cv[2 * j], c0);
            c1 = __builtin_fmaf(cv[2 * j + 1], cv[2 * j + 1], c1);
        }
    }
    float s = a0 + a1;
    const float cn = c0 + c1;
    if constexpr (COS) s = s * ((cn > 0.0f) ? 1.0f / __builtin_sqrtf(cn) : 0.0f);
    // No number among the scores: the first list, as nothing beats it.
    s = (l < nlist && s == s) ? s : -__builtin_inff();
    take_better(s, l, __shfl_xor(s, step, 64), __shfl_xor(l, step, 64));
    take_better(s, l, __shfl_xor(s, 2 * step, 64), __shfl_xor(l, 2 * step, 64));
    return l;
}

template <int KT, int KD, int T, bool COS>
__global__ __launch_bounds__(512) void assign_stage_kernel(
    const uint16_t* __restrict__ keys, int64_t n, int d, int64_t ld,
    const float* __restrict__ centroids, int nlist, int32_t* __restrict__ out_list) {
    constexpr int W = 8;
    constexpr int KS = KD / 32;                    // 32-dim steps
    constexpr int kTileC = KD <= 64 ? 64 : 32;     // centroids per stage
    constexpr int CT = kTileC / 16;                // centroid tiles per stage
    constexpr int LPC = KD / 4;                    // threads per centroid (4 dims each)
    constexpr int CPP = 64 * W / 2 / LPC;          // centroids per pass of half the waves
    constexpr int NP = kTileC / 2 / CPP;           // passes over half a stage
    static_assert(LPC <= 64 && 2 * NP * CPP == kTileC, "staging shape");
    __shared__ u32x4 s_a[2][CT][kParts][KS][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool early = wv < W / 2;                 // waves w and w + 4 share a SIMD
    const int col = lane & 15, grp = lane >> 4;
    const int64_t base = ((int64_t)blockIdx.x * W + wv) * (16 * T);

    // Staging: this thread's 4 dims of rows sr + p * CPP of a stage (dims >= d
    // are zero; loads on clamped addresses).
    const int st = tid & (64 * W / 2 - 1);
    const int sr = (early ? 0 : kTileC / 2) + st / LPC, sd = 4 * (st % LPC);
    float4 raw[NP];
    auto request = [&](int l0) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int l = l0 + sr + p * CPP;
            const bool in = l < nlist && sd < d;
            __builtin_memcpy(&raw[p], centroids + (in ? (int64_t)l * d + sd : 0), 16);
        }
    };
    auto stage = [&](int l0, int buf) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int r = sr + p * CPP;
            const bool in = sd < d;
            float x[4] = {in ? raw[p].x : 0.0f, in ? raw[p].y : 0.0f, in ? raw[p].z : 0.0f,
                          in ? raw[p].w : 0.0f};
            if constexpr (COS) {
                float cn = 0.0f;
#pragma unroll
                for (int t = 0; t < 4; ++t) cn = __builtin_fmaf(x[t], x[t], cn);
                cn = group_sum<LPC>(cn);
                const float mul = (cn > 0.0f) ? 1.0f / __builtin_sqrtf(cn) : 0.0f;
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = x[t] * mul;
            }
            uint32_t part[4][kParts];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                // Rows past the last centroid score NaN: never the best.
                three_parts(l0 + r < nlist ? x[t] : __builtin_nanf(""), part[t]);
            // A[row r % 16][k = sd % 32 ..]: lane 16 * ((sd % 32) / 8) + r % 16.
            const int al = 16 * ((sd & 31) >> 3) + (r & 15);
            const int half = (sd >> 2) & 1;
#pragma unroll
            for (int q = 0; q < kParts; ++q)
                ((u32x2*)&s_a[buf][r >> 4][q][sd >> 5][al])[half] =
                    u32x2{upper_halves(part[0][q], part[1][q]), upper_halves(part[2][q], part[3][q])};
        }
    };

    request(0);
    u32x4 kf[T][KS][kKeyParts<KT>];
    float best[T];
    int row0[T];                                   // first row of the best's 16-row tile
    const uint32_t plain = load_keys<KT, KS, T>(keys, base, n, d, ld, kf);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        best[t] = -__builtin_inff();
        row0[t] = 0;
    }
    stage(0, 0);
    if (early) request(kTileC);
    __syncthreads();
    int buf = 0;
    for (int l0 = 0; l0 < nlist; l0 += kTileC) {
        const bool more = l0 + kTileC < nlist;
        if (early) {
            if (more) stage(l0 + kTileC, buf ^ 1);
            request(l0 + 2 * kTileC);
        } else {
            request(l0 + kTileC);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            u32x4 a[kParts][KS];
#pragma unroll
            for (int p = 0; p < kParts; ++p)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) a[p][ks] = s_a[buf][c][p][ks][lane];
            tile_products<KT, KS, T>(l0 + 16 * c, a, kf, best, row0);
        }
        if (!early && more) stage(l0 + kTileC, buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
    for (int t = 0; t < T; ++t) {
        float b = best[0];
        int r = row0[0];
#pragma unroll
        for (int u = 1; u < T; ++u) {              // t is uniform: scalar selects
            b = t == u ? best[u] : b;
            r = t == u ? row0[u] : r;
        }
        r += 4 * grp;
        merge_lanes(b, r);
        const int64_t i = base + 16 * t + col;
        const uint16_t* row = keys + (i < n ? i : n - 1) * ld;
        const int l = settle<KT, COS>(row, d, centroids, nlist, r + grp, 16);
        const bool mine = grp == 0 && i < n, served = (plain >> t) & 1u;
        if (mine && served) out_list[i] = l;
        assign_rest<KT>(__ballot(mine && !served), i, keys, ld, d, centroids, nlist, COS, out_list);
    }
}

template <int KT, int KD, int T, bool COS>
__global__ __launch_bounds__(512) void assign_split_kernel(
    const uint16_t* __restrict__ keys, int64_t n, int d, int64_t ld,
    const float* __restrict__ centroids, int nlist, int32_t* __restrict__ out_list) {
    constexpr int W = 8;
    constexpr int KS = KD / 32;                    // 32-dim steps
    __shared__ float s_best[W][16 * T];
    __shared__ int s_row0[W][16 * T];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int64_t base = (int64_t)blockIdx.x * (16 * T);
    const int ntiles = (nlist + 15) / 16;

    // This lane's part of a centroid tile: row tile * 16 + col, dims 8 grp + 32
    // ks .. + 7 (rows past the last re-read it, dims >= d read dim 0).
    float raw[KS][8];
    auto request = [&](int tile) {
        int l = tile * 16 + col;
        l = l < nlist ? l : nlist - 1;
        const float* c = centroids + (int64_t)l * d;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int e = 8 * grp + 32 * ks;
            __builtin_memcpy(raw[ks], c + (e < d ? e : 0), 32);
        }
    };
    request(wv);
    u32x4 kf[T][KS][kKeyParts<KT>];
    float best[T];
    int row0[T];
    const uint32_t plain = load_keys<KT, KS, T>(keys, base, n, d, ld, kf);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        best[t] = -__builtin_inff();
        row0[t] = 0;
    }
    for (int tile = wv; tile < ntiles; tile += W) {
        // Normalise, and split.  Rows past the last centroid become NaN: their
        // scores are never the best.
        const bool real = tile * 16 + col < nlist;
        float mul = 1.0f;
        if constexpr (COS) {
            float cn = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                float a = 0.0f;
#pragma unroll
                for (int j = 0; j < 8; ++j) a = __builtin_fmaf(raw[ks][j], raw[ks][j], a);
                cn += 8 * grp + 32 * ks < d ? a : 0.0f;
            }
            cn += __shfl_xor(cn, 16, 64);
            cn += __shfl_xor(cn, 32, 64);
            mul = (cn > 0.0f) ? 1.0f / __builtin_sqrtf(cn) : 0.0f;
        }
        u32x4 a[kParts][KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bool in = 8 * grp + 32 * ks < d;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t part[2][kParts];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float v = in ? raw[ks][2 * j + h] : 0.0f;
                    if constexpr (COS) v = v * mul;
                    three_parts(real ? v : __builtin_nanf(""), part[h]);
                }
#pragma unroll
                for (int q = 0; q < kParts; ++q) a[q][ks][j] = upper_halves(part[0][q], part[1][q]);
            }
        }
        if (tile + W < ntiles) request(tile + W);
        tile_products<KT, KS, T>(tile * 16, a, kf, best, row0);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        int r = row0[t] + 4 * grp;
        merge_lanes(best[t], r);
        if (grp == 0) {
            s_best[wv][16 * t + col] = best[t];
            // The sign marks a key that the products do not serve.
            s_row0[wv][16 * t + col] = (plain >> t) & 1u ? r : -1;
        }
    }
    __syncthreads();
    // Four lanes per key: the best group of all waves, then one row each (whole
    // waves: 64 T keys' lanes).
    for (int u = tid; u < 64 * T; u += 64 * W) {
        const int key = u >> 2;
        const int64_t i = base + key;
        float b = s_best[0][key];
        int r = s_row0[0][key];
        const bool served = r >= 0;
#pragma unroll
        for (int w = 1; w < W; ++w) take_better(b, r, s_best[w][key], s_row0[w][key]);
        const uint16_t* row = keys + (i < n ? i : n - 1) * ld;
        const int l = settle<KT, COS>(row, d, centroids, nlist, (served ? r : 0) + (u & 3), 1);
        const bool mine = (u & 3) == 0 && i < n;
        if (mine && served) out_list[i] = l;
        assign_rest<KT>(__ballot(mine && !served), i, keys, ld, d, centroids, nlist, COS, out_list);
    }
}

// ---------------------------------------------------------------- encoding
constexpr int kEncThreads = 256;
constexpr int kEncGroup = 8;     // entries per comparison with the best so far

// Squared distance of a residual slice to a codebook entry, in dimension
// order; DS dims, or dsub <= kMaxDsub of them when DS = 0.
template <int DS>
__device__ __forceinline__ float slice_dist(const float* rs, const float* __restrict__ cb,
                                            int dsub) {
    float dist = 0.0f;
#pragma unroll
    for (int t = 0; t < (DS ? DS : kMaxDsub); ++t) {
        if (DS || t < dsub) {
            const float df = rs[t] - cb[t];
            dist = __builtin_fmaf(df, df, dist);
        }
    }
    return dist;
}

// Codes of key i: nearest codebook entry (squared L2, ties to the lower
// entry) to each slice of the residual key - centroid[list]; codes j0 ..
// j0 + jn - 1 of 256 keys per block, one thread per key.
//
// Bound: the vector ALUs, 2 DS instructions per (slice, entry) for the
// distance itself.  Every lane compares with the same entry at the same time,
// so the codebook comes through scalar loads and enters the subtractions as a
// scalar operand: no LDS and no vector register for it.  Eight distances are
// reduced to their minimum before one comparison with the best so far, and the
// entry inside the winning group is found once per slice, from the same
// arithmetic (10 instead of 24 selection instructions per eight entries).
// The slice length is a template parameter (with a run-time length the loop
// was 16 predicated steps for each entry, from LDS): 262144 keys of 64
// dims, 16 slices, 256 entries: 2303 -> 240 us, 0.9 of the VALUs' issue rate.
template <int KT, int DS>
__global__ __launch_bounds__(kEncThreads) void pq_encode_kernel(
    const uint16_t* __restrict__ keys, int64_t n, int d, int64_t ld,
    const float* __restrict__ centroids, const int32_t* __restrict__ list_ids,
    const float* __restrict__ codebooks, int m, int ksub, int nlist, int jn, int words,
    uint8_t* __restrict__ codes) {
    constexpr int R = DS ? DS : kMaxDsub;
    const int64_t i = (int64_t)blockIdx.x * kEncThreads + threadIdx.x;
    const int j0 = blockIdx.y * jn;
    const int j1 = j0 + jn < m ? j0 + jn : m;
    const int dsub = DS ? DS : d / m;
    const int64_t ic = i < n ? i : n - 1;
    const int32_t li = list_ids[ic];
    const bool known = li >= 0 && li < nlist;      // no such list: code 0 throughout
    const float* c = centroids + (int64_t)(known ? li : 0) * d;
    const uint16_t* row = keys + ic * ld;
    uint32_t word = 0;
    for (int j = j0; j < j1; ++j) {
        float rs[R];
#pragma unroll
        for (int t = 0; t < R; ++t)
            rs[t] = (DS || t < dsub) ? elem_f32<KT>(row[j * dsub + t]) - c[j * dsub + t] : 0.0f;
        const float* cb = codebooks + (int64_t)j * ksub * dsub;
        float bd = __builtin_inff();
        int be = 0;
        int e = 0;
        for (; e + kEncGroup <= ksub; e += kEncGroup) {
            float g = slice_dist<DS>(rs, cb + (int64_t)e * dsub, dsub);
#pragma unroll
            for (int u = 1; u < kEncGroup; ++u)    // a NaN distance is no minimum
                g = __builtin_fminf(g, slice_dist<DS>(rs, cb + (int64_t)(e + u) * dsub, dsub));
            const bool up = g < bd;
            bd = up ? g : bd;
            be = up ? e : be;
        }
        for (; e < ksub; ++e) {
            const float g = slice_dist<DS>(rs, cb + (int64_t)e * dsub, dsub);
            const bool up = g < bd;
            bd = up ? g : bd;
            be = up ? e : be;
        }
        // The first entry from be on at that distance (the same bits).
        int code = 0;
        if (bd < __builtin_inff()) {
            code = be;
            while (code < ksub - 1 &&
                   !(slice_dist<DS>(rs, cb + (int64_t)code * dsub, dsub) == bd))
                ++code;
        }
        if (!known) code = 0;
        if (words) {
            word |= (uint32_t)code << (8 * (j & 3));
            if ((j & 3) == 3) {
                if (i < n) *(uint32_t*)(codes + i * m + (j & ~3)) = word;
                word = 0;
            }
        } else if (i < n) {
            codes[i * m + j] = (uint8_t)code;
        }
    }
}

template <int KT, int KD, int T, bool STAGE>
hipError_t assign_shape(const void* keys, int64_t n, int d, int64_t ld, const float* centroids,
                        int nlist, int cosine, int32_t* out_list, hipStream_t stream) {
    const int64_t per = (int64_t)16 * T * (STAGE ? 8 : 1);
    const dim3 grid((unsigned)((n + per - 1) / per)), block(512);
    const uint16_t* k = (const uint16_t*)keys;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, stream, k, n, d, ld, centroids, nlist, out_list);
        return hipGetLastError();
    };
    if constexpr (STAGE)
        return cosine ? go(assign_stage_kernel<KT, KD, T, true>)
                      : go(assign_stage_kernel<KT, KD, T, false>);
    else
        return cosine ? go(assign_split_kernel<KT, KD, T, true>)
                      : go(assign_split_kernel<KT, KD, T, false>);
}

// The shape with the least time, from its rounds of one block per compute unit,
// in tenths of a round of the split shape with 4 tiles (which has to be ahead by a
// twentieth: it loses by more where the centroids are few).  Where the registers
// leave room for a second block on a unit, its round costs less than the first.
// Measured (us at 4096 centroids; split a round, then 1, 2, 3 and 4 rounds of two
// tiles and 1 and 2 of four):
//   bf16  d  32   20 | 81 112 160 218 | 113 170      64   35 | 137 210 326 425 | 190 298
//        128   69 | 264 410 630 823 | 397 781
//   fp16  32   25 | 96 150 220 303 | 150 245      64   49 | 174 285 445 593 | 276 557
//        128   90 | 355 710 1065 1422 | 530 1070
// 70000 keys, against blocks by the shapes' former costs: 64 dims bf16 189 -> 175,
// fp16 276 -> 243; 165000: fp16 556 -> 439, 128 dims bf16 782 -> 625.  Fewer
// centroids scale all alike down to about a thousand; below, two tiles gain (256 x
// 64 dims fp16, 100000 keys: 38 against 44).
template <int KT, int KD>
hipError_t assign_dim(const void* keys, int64_t n, int d, int64_t ld, const float* centroids,
                      int nlist, int cosine, int32_t* out_list, hipStream_t stream) {
    const int64_t cus = device_cus();
    auto rounds = [&](int64_t per) { return (n + per * cus - 1) / (per * cus); };
    constexpr int kFrags = kKeyParts<KT> * (KD / 32);    // of a key tile
    const int64_t split4 = 10 * rounds(64);
    const int64_t r2 = rounds(256), r4 = rounds(512);
    const int64_t stage2 = kFrags > 4 ? 39 * r2 : r2 == 1 ? 39 : r2 / 2 * 59 + r2 % 2 * 32;
    const int64_t stage4 = KT == DT_BF16 && kFrags <= 2 ? r4 / 2 * 90 + r4 % 2 * 57 : 57 * r4;
    if (21 * split4 <= 20 * stage2 && 21 * split4 <= 20 * stage4)
        return assign_shape<KT, KD, 4, false>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
    if (stage2 < stage4)
        return assign_shape<KT, KD, 2, true>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
    return assign_shape<KT, KD, 4, true>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
}

template <int KT>
hipError_t assign_type(const void* keys, int64_t n, int d, int64_t ld, const float* centroids,
                       int nlist, int cosine, int32_t* out_list, hipStream_t stream) {
    if (d <= 32) return assign_dim<KT, 32>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
    if (d <= 64) return assign_dim<KT, 64>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
    return assign_dim<KT, 128>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
}

template <int KT, int DS>
hipError_t encode_dsub(const void* keys, int64_t n, int d, int64_t ld, const float* centroids,
                       int nlist, const int32_t* list_ids, const float* codebooks, int m, int ksub,
                       uint8_t* codes, hipStream_t stream) {
    // All slices of a key in one block once that gives every SIMD four waves;
    // fewer keys spread their slices over more blocks.
    const int64_t blocks = (n + kEncThreads - 1) / kEncThreads;
    const int64_t want = (int64_t)device_cus() * 4;
    int64_t parts = (want + blocks - 1) / blocks;
    if (parts > m) parts = m;
    int jn = (int)((m + parts - 1) / parts);
    if (jn >= 3 && m % 4 == 0) jn = (jn + 3) / 4 * 4;
    // Four codes a store where words are aligned and blocks hold whole words.
    const int words = m % 4 == 0 && jn % 4 == 0 && ((uintptr_t)codes & 3) == 0;
    hipLaunchKernelGGL((pq_encode_kernel<KT, DS>),
                       dim3((unsigned)blocks, (unsigned)((m + jn - 1) / jn)), dim3(kEncThreads), 0,
                       stream, (const uint16_t*)keys, n, d, ld, centroids, list_ids, codebooks, m,
                       ksub, nlist, jn, words, codes);
    return hipGetLastError();
}

template <int KT>
hipError_t encode_type(const void* keys, int64_t n, int d, int64_t ld, const float* centroids,
                       int nlist, const int32_t* list_ids, const float* codebooks, int m, int ksub,
                       uint8_t* codes, hipStream_t stream) {
    switch (d / m) {
        case 2:
            return encode_dsub<KT, 2>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m, ksub, codes, stream);
        case 4:
            return encode_dsub<KT, 4>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m, ksub, codes, stream);
        case 8:
            return encode_dsub<KT, 8>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m, ksub, codes, stream);
        case 16:
            return encode_dsub<KT, 16>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m, ksub, codes, stream);
        default:
            return encode_dsub<KT, 0>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m, ksub, codes, stream);
    }
}

}  // namespace

hipError_t launch_ivf_assign(const void* keys, int key_dtype, int64_t n, int d, int64_t ld,
                             const float* centroids, int nlist, int cosine, int32_t* out_list,
                             hipStream_t stream) {
    return key_dtype == DT_BF16
               ? assign_type<DT_BF16>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream)
               : assign_type<DT_F16>(keys, n, d, ld, centroids, nlist, cosine, out_list, stream);
}

hipError_t launch_pq_encode(const void* keys, int key_dtype, int64_t n, int d, int64_t ld,
                            const float* centroids, int nlist, const int32_t* list_ids,
                            const float* codebooks, int m, int ksub, uint8_t* codes,
                            hipStream_t stream) {
    return key_dtype == DT_BF16
               ? encode_type<DT_BF16>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m,
                                      ksub, codes, stream)
               : encode_type<DT_F16>(keys, n, d, ld, centroids, nlist, list_ids, codebooks, m,
                                     ksub, codes, stream);
}

}  // namespace sense
