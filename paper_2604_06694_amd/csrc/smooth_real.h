// One workgroup per head for power-of-two lengths from 1024 to 32768 (smooth_real.hip).
#pragma once

#include "common.h"

namespace audiokv {

constexpr int kRealMinL = 1024;
__host__ __device__ inline bool real_length(int L) { return L >= kRealMinL && L <= 32768 && (L & (L - 1)) == 0; }

// every head whose length is in `lengths` (the sum of different lengths of the above); heads of other lengths are left alone. The
// cutoff leaves a mask that needs a transform, or is to be found from the spectrum.
hipError_t launch_smooth_real(unsigned lengths, const Geom& g, const float* in, bool pool_on_load, const int32_t* cu_seqlens, double cutoff_frac,
                              float alpha, float* out, int32_t* kstar_out, bool cutoffs_only, hipStream_t s);

// Pooling (kernel 7), smoothing with a fixed cutoff and selection of a call whose heads all have L tokens, 1024 to 16384.
struct SelectJob;
constexpr int kFusedMaxL = 16384;
hipError_t launch_smooth_select(int L, const Geom& g, const float* in, const int32_t* cu_seqlens, double cutoff_frac, float alpha, float* out,
                                const SelectJob& job, hipStream_t s);

}  // namespace audiokv
