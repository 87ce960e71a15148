// The convolution path of the spectral smoothing: how smooth.hip hands it work.
#pragma once

#include "conv_filter.h"

namespace audiokv {

// Chunks of 2^10 .. 2^13 points, at most 16 per head: lengths up to 131072.
constexpr int kConvMaxPool = 9;           // pooling kernels that the convolution's loads apply
constexpr int kConvMinLogC = 10, kConvMaxLogC = 13, kConvMaxLogR = 4;

// log2 of the transform of a head of L samples cut into chunks of 2^log_c points
__host__ __device__ inline int conv_log_points(int L, int log_c) {
    int lg = log_c;
    while ((1 << lg) < L) ++lg;
    return lg;
}

// One run of the path over the items of a call that it owns.
struct ConvCall {
    bool any = false;
    ConvFilterJob job{};
    int log_c = 0;
    int max_r = 1;            // chunks of the longest head
    size_t points = 0;        // points of the longest transform: stride of `part` (per head) and `spec` (per item)
    void* part = nullptr;     // complex results of the chunks (unused when max_r = 1)
    void* spec = nullptr;     // the filters' bins, or null: every workgroup transforms its own share of the filter
};

// taps and, if c.spec is set, the filters' bins
hipError_t launch_conv_filter(const Geom& g, const ConvCall& c, hipStream_t s);
// pool_on_load: `in` lies inside a workspace that extends 16 floats to either side of every head
hipError_t launch_conv(const Geom& g, const ConvCall& c, const float* in, bool pool_on_load, float alpha, float* out, hipStream_t s);

}  // namespace audiokv
