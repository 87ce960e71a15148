// The low-pass filter of the spectral smoothing as a sequence of taps, evaluated in float64. A header of its own
// because its evaluation depends on the lengths and the cutoff only and rides along in whatever launch is at hand.
#pragma once

#include "common.h"

namespace audiokv {

// Taps h[0..L) of an item of L tokens, written once per distinct length of a call (by the first item that has it).
struct ConvFilterJob {
    float* h;                 // taps of item i start at h + i * item_stride; null: no such job
    int64_t item_stride;      // at least L; 8 floats past the last taps are there to be read
    const int32_t* cu_seqlens;
    int n_items;
    double cutoff_frac;
    int taper_bins;
    int max_length;           // of the items that have taps
    // workgroups of `threads`, a tap and its mirror image per thread (in a call of very many items more)
    int blocks_per_item(int threads) const { return blocks_per_part((max_length / 2 + threads) / threads, n_items, threads); }
};

struct SmoothFilters {
    bool long_work = false;
    ConvFilterJob taps{};     // taps.h: the only preparation is these taps (null: none, or more than that)
};

#if defined(__HIPCC__)
namespace {

// sin(pi n x) / sin(pi x), x = p / (2 q) with |x| < 3/4
__device__ __forceinline__ double sine_ratio(long long p, long long q, int n) {
#pragma clang fp contract(off)
    if (p == 0) return (double)n;
    const double x = (double)p / (double)(2 * q);
    return sinpi((double)n * x) / sinpi(x);
}

// One tap of the circular filter whose frequency response is the mask (Eqs. 17-18): h[n] = (1/L) sum over all L bins
// of mask * cos(2 pi k n / L). The bins up to k* add up to a ratio of sines with an exactly reduced angle. The
// taper's weights are (1 + cos(pi j / (T+1))) / 2, so its bins are three geometric series; a Nyquist bin counts once.
// Compiled into several sources whose settings differ: nothing is contracted, so that the taps are the same bits wherever
// they are evaluated.
// 0 <= n <= L/2
__device__ __forceinline__ float low_pass_tap(int n, int L, int kstar, int T) {
#pragma clang fp contract(off)
    // (2 k* + 1) n mod 2 L, 0 <= n <= L/2: in float64, where all of it is exact (a 64-bit integer remainder takes as long as a
    // sine), from a quotient that may be off by one
    const double all = (double)(2 * kstar + 1) * (double)n, turn = 2.0 * (double)L;
    double r = fma(-floor(all / turn), turn, all);
    r = r < 0.0 ? r + turn : r >= turn ? r - turn : r;
    double v = n == 0 ? (double)(2 * kstar + 1) : sinpi(r / (double)L) / sinpi((double)n / (double)L);
    const int half = L >> 1, J = min(T, half - kstar);
    if (J > 0) {
        const double phi = 2.0 * (double)((long long)kstar * n % L) / (double)L;        // angle of bin k*, in units of pi
        const long long t1 = (long long)T + 1;
        // sum_{j=1..J} cos(phi + a j) = cos(phi + a (J+1)/2) sin(a J/2) / sin(a/2)
        auto series = [&](long long p, long long q) {                                   // a = pi * p / q
            return cospi(phi + (double)p / (double)q * (0.5 * (double)(J + 1))) * sine_ratio(p, q, J);
        };
        v += series(2LL * n, L) + 0.5 * (series(2LL * n * t1 + L, L * t1) + series(2LL * n * t1 - L, L * t1));
        if (2 * (kstar + J) == L) v -= 0.5 * (1.0 + cospi((double)J / (double)t1)) * ((n & 1) ? -1.0 : 1.0);
    }
    return (float)(v / (double)L);
}

__device__ __forceinline__ int conv_kstar(double cutoff_frac, int L) { return (int)floor(cutoff_frac * (double)(L >> 1)); }
// whether the convolution path smooths an item of length L: not a power of two (smooth.hip has a faster transform for
// those), and a mask that needs a transform at all
__device__ __forceinline__ bool conv_item(const ConvFilterJob& job, int L) {
    if (L >= 4 && L <= 32768 && (L & (L - 1)) == 0) return false;
    const int kstar = conv_kstar(job.cutoff_frac, L);
    return kstar < (L >> 1) && kstar + job.taper_bins > 0;
}

// the first item with the same length owns its taps (and its spectrum)
__device__ __forceinline__ int conv_owner(const int32_t* __restrict__ cu_seq, int item, int L) {
    for (int i = 0; i < item; ++i)
        if (cu_seq[i + 1] - cu_seq[i] == L) return i;
    return item;
}

// workgroup `block` of per_item * n_items, of `threads` threads each
__device__ __forceinline__ void conv_filter_block(const ConvFilterJob& job, int block, int per_item, int threads) {
    const int item = block / per_item, part = block - item * per_item;
    const int L = job.cu_seqlens[item + 1] - job.cu_seqlens[item];
    if (!conv_item(job, L) || conv_owner(job.cu_seqlens, item, L) != item) return;
    const int kstar = conv_kstar(job.cutoff_frac, L);
    float* h = job.h + item * job.item_stride;
    for (int n = part * threads + (int)threadIdx.x; n <= L >> 1; n += per_item * threads) {
        const float v = low_pass_tap(n, L, kstar, job.taper_bins);
        h[n] = v;
        if (n > 0) h[L - n] = v;                    // h is even
    }
}

}  // namespace
#endif

}  // namespace audiokv
