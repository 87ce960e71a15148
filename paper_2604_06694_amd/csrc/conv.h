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
    bool uneven = false;      // other heads have fewer
    size_t points = 0;        // points of the longest transform: stride of `part` (per head) and `spec` (per item)
    void* part = nullptr;     // complex results of the chunks (unused when max_r = 1)
    void* spec = nullptr;     // the filters' bins, or null: every workgroup transforms its own share of the filter
};

// The chunks of a run that are left to be combined by whoever reads the result (conv_join.h): heads of kJoinMaxR chunks of
// 2^kJoinLogC points at most, which is 16384 samples. (Of eight chunks a workgroup would read 256 KB: one layer of 30000 tokens
// 71.9 us with a launch that combines them, 73.5 without.)
constexpr int kJoinLogC = 12, kJoinMaxR = 4;
struct ConvJoin {
    ConvFilterJob job{};
    const float* in = nullptr;          // the samples, for alpha < 1
    int pool_on_load = 0;
    float alpha = 1.f;
    const void* part = nullptr;         // null: nothing is left
    size_t part_stride = 0;             // complex values per head
    float* out = nullptr;               // where the result goes
};

// taps and, if c.spec is set, the filters' bins
hipError_t launch_conv_filter(const Geom& g, const ConvCall& c, hipStream_t s);
// pool_on_load: `in` lies inside a workspace that extends 16 floats to either side of every head
// join: if given and the chunks are of that kind, they are left uncombined
hipError_t launch_conv(const Geom& g, const ConvCall& c, const float* in, bool pool_on_load, float alpha, float* out, hipStream_t s,
                       ConvJoin* join = nullptr);

// Pooling (kernel 7), smoothing and selection of a call whose heads are all of one chunk of up to 4096 points
struct SelectJob;
hipError_t launch_conv_select(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, const SelectJob& sel, hipStream_t s);

}  // namespace audiokv
