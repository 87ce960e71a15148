// What the selection of a head (select_body.h) is made of, and the selection for the smoothing of short heads. select.hip describes the
// method.
#pragma once

#include "common.h"

namespace audiokv {

// What a smoothing launch needs to select as well.
struct SelectJob {
    const int32_t* budgets = nullptr;
    const int32_t* cu_b = nullptr;
    int32_t* indices = nullptr;
    bool done = false;                // set by the launch that did
};

namespace {

// float -> uint32 whose unsigned order is the float order; -0.0 and +0.0 map to one key
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// its inverse
__device__ __forceinline__ float key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}

// Workgroup barrier that orders LDS traffic only: nothing is exchanged through memory, and the stores on their way (the window's
// indices, scores combined from chunks) are no reason to wait.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Largest value over the lanes of a full wave, in lane 63 (the sum likewise)
#define AUDIOKV_DPP_F(x, ctrl, rows, none) \
    __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(x), ctrl, rows, 0xf, false))
#define AUDIOKV_WAVE_FOLD(op, x, none)                      \
    do {                                                    \
        x = op(x, AUDIOKV_DPP_F(x, 0x111, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x112, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x114, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x118, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x142, 0xa, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x143, 0xc, none));      \
    } while (0)
// the same over the first N lanes, a power of two up to 16: in lane N - 1
#define AUDIOKV_ROW_FOLD(op, x, none, N)                    \
    do {                                                    \
        x = op(x, AUDIOKV_DPP_F(x, 0x111, 0xf, none));      \
        if (N > 2) x = op(x, AUDIOKV_DPP_F(x, 0x112, 0xf, none)); \
        if (N > 4) x = op(x, AUDIOKV_DPP_F(x, 0x114, 0xf, none)); \
        if (N > 8) x = op(x, AUDIOKV_DPP_F(x, 0x118, 0xf, none)); \
    } while (0)
__device__ __forceinline__ float plus(float a, float b) { return a + b; }
__device__ __forceinline__ float wave_sum63(float x) { AUDIOKV_WAVE_FOLD(plus, x, 0.f); return x; }
__device__ __forceinline__ float wave_max63(float x) { AUDIOKV_WAVE_FOLD(fmaxf, x, -INFINITY); return x; }
template <int N> __device__ __forceinline__ float row_sum(float x) { AUDIOKV_ROW_FOLD(plus, x, 0.f, N); return x; }
template <int N> __device__ __forceinline__ float row_max(float x) { AUDIOKV_ROW_FOLD(fmaxf, x, -INFINITY, N); return x; }
__device__ __forceinline__ float lane_float(float x, int lane) {           // uniform lane
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
#undef AUDIOKV_ROW_FOLD
#undef AUDIOKV_WAVE_FOLD
#undef AUDIOKV_DPP_F

constexpr int kDigitBits = 11, kBins = 1 << kDigitBits;   // bins of one histogram round
constexpr int kLast = 64;            // candidates that one wave ranks against each other

// Inclusive sum over the first N lanes, a power of two up to 16
template <int N>
__device__ __forceinline__ int row_incl(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    if (N > 2) x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    if (N > 4) x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    if (N > 8) x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    return x;
}

// Largest value over the lanes of a full wave, in lane 63.
__device__ __forceinline__ uint32_t wave_max63(uint32_t x) {
#define AUDIOKV_MAX_STEP(ctrl, rows) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, rows, 0xf, false))
    AUDIOKV_MAX_STEP(0x111, 0xf);
    AUDIOKV_MAX_STEP(0x112, 0xf);
    AUDIOKV_MAX_STEP(0x114, 0xf);
    AUDIOKV_MAX_STEP(0x118, 0xf);
    AUDIOKV_MAX_STEP(0x142, 0xa);
    AUDIOKV_MAX_STEP(0x143, 0xc);
#undef AUDIOKV_MAX_STEP
    return x;
}

// The selection of one head by its workgroup, for kernels that have its scores at hand.
template <int EPT, int NT, class Scores>
__device__ __forceinline__ void select_head(const Geom& g, int head, int L, const int32_t* __restrict__ budgets,
                                            const int32_t* __restrict__ cu_b, int32_t* __restrict__ indices, Scores scores)
{
    constexpr bool always = false;
#include "select_body.h"
}

}  // namespace
}  // namespace audiokv
