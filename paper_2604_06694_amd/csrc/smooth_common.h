// What the two smoothing translation units share: pooling on load, complex arithmetic, LDS padding, which lengths and
// masks go where.
#pragma once

#include "common.h"

namespace audiokv {
namespace {

constexpr int kMaxPow2L = 32768;          // 128 KiB of fp32 in LDS
__host__ __device__ inline bool pow2_length(int L) { return L >= 4 && L <= kMaxPow2L && (L & (L - 1)) == 0; }

// Pooled value at position j of one head's sequence x[0..L) (global or LDS).
__device__ __forceinline__ float pooled_at(const float* x, int L, int j, int kernel, int mode) {
    const int half = kernel >> 1;
    if (mode == AUDIOKV_POOL_AVG) {
        float acc = 0.f;
        for (int t = -half; t <= half; ++t) {
            const int p = j + t;
            acc += (p >= 0 && p < L) ? x[p] : 0.f;       // zero padding
        }
        return acc * (1.0f / (float)kernel);              // divisor is always the kernel size (one rounded reciprocal)
    }
    float acc = -INFINITY;
    for (int t = -half; t <= half; ++t) {
        const int p = j + t;
        if (p >= 0 && p < L) acc = fmaxf(acc, x[p]);
    }
    return acc;
}

// Pooled values at positions j0 and j0 + 1 of a sequence held in LDS, kernel size K known at compile time. Same
// taps, padding, order of operations and reciprocal as pooled_at, so both give the same bits.
template <int K>
__device__ __forceinline__ void pooled_pair_lds(const float* x, int L, int j0, int mode, float& o0, float& o1) {
    const float fill = mode == AUDIOKV_POOL_AVG ? 0.f : -INFINITY;
    float w[K + 1];
    if (j0 - K / 2 >= 0 && j0 + 1 + K / 2 < L) {     // every tap inside the sequence: all but the edge threads
#pragma unroll
        for (int u = 0; u <= K; ++u) w[u] = x[j0 - K / 2 + u];
    } else {
#pragma unroll
        for (int u = 0; u <= K; ++u) {
            const int p = j0 - K / 2 + u;
            const float v = x[min(max(p, 0), L - 1)];
            w[u] = (p >= 0 && p < L) ? v : fill;
        }
    }
    if (mode == AUDIOKV_POOL_AVG) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int u = 0; u < K; ++u) { a0 += w[u]; a1 += w[u + 1]; }
        o0 = a0 * (1.0f / (float)K);
        o1 = a1 * (1.0f / (float)K);
    } else {
        float a0 = -INFINITY, a1 = -INFINITY;
#pragma unroll
        for (int u = 0; u < K; ++u) { a0 = fmaxf(a0, w[u]); a1 = fmaxf(a1, w[u + 1]); }
        o0 = a0;
        o1 = a1;
    }
}

// Pooled values at positions j0 and j0 + 1 of x[0..L) (global memory or LDS), kernels of 3 to 9 (wider ones are pooled by a
// launch of their own): all taps at once, independent loads. The bits of pooled_at.
__device__ __forceinline__ void pooled_pair(const float* x, int L, int j0, int kernel, int mode, float& o0, float& o1) {
    switch (kernel) {
        case 3:  pooled_pair_lds<3>(x, L, j0, mode, o0, o1); break;
        case 5:  pooled_pair_lds<5>(x, L, j0, mode, o0, o1); break;
        case 7:  pooled_pair_lds<7>(x, L, j0, mode, o0, o1); break;
        default: pooled_pair_lds<9>(x, L, j0, mode, o0, o1); break;
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));    // any head start: heads are L floats apart

// Pooled values around samples 4 .. 11 of a window of 16. Same taps, order of additions and reciprocal as pooled_at
// (which is what makes the fused path equal the staged one): POOL = 7, the usual size, spelled out; POOL = 9 for any
// size up to 9, where the taps outside the kernel are replaced by the padding's neutral value.
template <int POOL>
__device__ __forceinline__ void pooled_window(const float (&w)[16], int kernel, int mode, float (&o)[8]) {
    const int half = POOL == 7 ? 3 : kernel >> 1;
    if (mode == AUDIOKV_POOL_AVG) {
        const float inv = POOL == 7 ? 1.0f / 7.0f : 1.0f / (float)kernel;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float a = 0.f;
#pragma unroll
            for (int u = -(POOL / 2); u <= POOL / 2; ++u) a += POOL == 7 || (u < 0 ? -u : u) <= half ? w[4 + e + u] : 0.f;
            o[e] = a * inv;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float a = -INFINITY;
#pragma unroll
            for (int u = -(POOL / 2); u <= POOL / 2; ++u)
                a = fmaxf(a, POOL == 7 || (u < 0 ? -u : u) <= half ? w[4 + e + u] : -INFINITY);
            o[e] = a;
        }
    }
}
// N consecutive floats from `at` (any alignment)
template <int N>
__device__ __forceinline__ void window_load(const float* __restrict__ at, float (&w)[N]) {
#pragma unroll
    for (int u = 0; u < N / 4; ++u) {
        const f32x4 a = *reinterpret_cast<const f32x4u*>(at + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * u + e] = a[e];
    }
}

struct cf { float re, im; };
__device__ __forceinline__ cf cmul(cf a, cf b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__host__ __device__ __forceinline__ cf cadd(cf a, cf b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cf csub(cf a, cf b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cf cconj(cf a) { return {a.re, -a.im}; }

// LDS slot of complex element i. One spare slot per 16 elements: a thread's 16-point group at stride 1 or 4 would
// otherwise sit in a single bank.
__host__ __device__ __forceinline__ int pad(int i) { return i + (i >> 4); }
__host__ __device__ constexpr size_t padded_len(size_t n) { return n + (n >> 4) + 1; }

// Masks for which the filter needs no transform at all, and for which a transform would only add rounding noise to
// what is exactly a plateau or exactly the input (the selection that follows breaks ties by index, so the noise
// would decide instead): 2 = every bin is kept with weight 1 (Eq. 19 returns s itself), 1 = only the DC bin
// survives (Eq. 19 returns the mean of s at every position), 0 = anything else.
__host__ __device__ inline int degenerate_mask(int L, int kstar, int T) {
    if (kstar >= (L >> 1)) return 2;
    if (kstar + T == 0) return 1;
    return 0;
}

}  // namespace
}  // namespace audiokv
