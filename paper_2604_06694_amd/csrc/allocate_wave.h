// Budget allocation of a pool of up to 128 heads by one wave (allocate.hip describes the method). A header of its own because
// a pool this small rides along in whatever launch is at hand.
#pragma once

#include "common.h"

#if defined(__HIPCC__)
namespace audiokv {
namespace {

// float64 operations that round one by one, whatever the including file's contraction setting is
__device__ __forceinline__ double add_rn(double a, double b) {
#pragma clang fp contract(off)
    return a + b;
}
__device__ __forceinline__ double sub_rn(double a, double b) {
#pragma clang fp contract(off)
    return a - b;
}
__device__ __forceinline__ double mul_rn(double a, double b) {
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ double div_rn(double a, double b) {
#pragma clang fp contract(off)
    return a / b;
}

__device__ __forceinline__ int n_keep_dev(double ratio, int L) {
    return (int)floor(add_rn(mul_rn(ratio, (double)L), 0.5));
}

// Whether the weights' sum defines shares: without one (all weights zero, a NaN, an infinity) the heads share equally. A share
// that is NaN would not compare with the others, and the hand-out of the remainder below would never end.
__device__ __forceinline__ bool has_shares(double sum) { return sum > 0.0 && sum < (double)INFINITY; }

__device__ __forceinline__ double lane_double(double v, int lane) {       // uniform lane
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane), hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ long long wave_sum_ll(long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// What a workgroup of allocate.hip does for larger pools, here for at most 64 PER heads by one wave, head 64 j + l in register j
// of lane l: no LDS and no barrier, the chains (the weight sum in head order, the ranks) run over lane reads. Same operations in
// the same order, hence the same bits. What this is for is latency: a launch that allocated four heads 6.2 -> 3.8 us.
// The chains grow with the heads: a call on 112 of them takes 22 us here and 24 by 256 threads (weights that cap in several
// rounds 33 and 41), on 128 25 and 26; beyond, the threads have it. Beside the sweeps, on the helper stream, it takes 65 us.
template <int PER>
__device__ __forceinline__ void allocate_wave(
    const int seg, const float* __restrict__ weights, int n_segments, int n, int weight_group, int window,
    const int32_t* __restrict__ cu_seq, double ratio, double beta,
    int32_t* __restrict__ budgets, int32_t* __restrict__ cu_budgets)
{
    const int lane = threadIdx.x & 63;
    const int L = cu_seq[seg + 1] - cu_seq[seg];
    const int nk = n_keep_dev(ratio, L);
    const int r = (int)floor(mul_rn(beta, (double)(nk - window)));
    const int f = window + r;                       // w + r of Eq. 1
    const long long Bs = (long long)n * (nk - f);   // budget shared out by weight
    const int cap = L - f;                          // no head keeps more than L tokens

    double S[PER], x[PER], frac[PER];
    int e[PER];
    bool live[PER], capped[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int h = 64 * j + lane;
        live[j] = h < n;
        capped[j] = false;
        const float* w = weights + ((size_t)seg * n + min(h, n - 1)) * weight_group;
        S[j] = 0.0;
        for (int q = 0; q < weight_group; ++q) S[j] = add_rn(S[j], (double)w[q]);
        x[j] = 0.0;
    }
    // proportional shares with the cap: heads over the cap are fixed at it and the rest is shared again among the others
    for (;;) {
        int ncap = 0;
        double tot = 0.0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            ncap += __builtin_popcountll(__builtin_amdgcn_ballot_w64(live[j] && capped[j]));
            const double add = capped[j] ? 0.0 : S[j];       // (+0.0 leaves the sum as it is, bit for bit)
            const int m = min(64, n - 64 * j);
            for (int l = 0; l < m; ++l) tot = add_rn(tot, lane_double(add, l));
        }
        const double T = (double)(Bs - (long long)ncap * cap);
        bool over = false;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (live[j] && !capped[j]) {
                x[j] = has_shares(tot) ? div_rn(mul_rn(T, S[j]), tot) : div_rn(T, (double)(n - ncap));
                over = over || x[j] > (double)cap;
            }
        if (__builtin_amdgcn_ballot_w64(over) == 0) break;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (live[j] && !capped[j] && x[j] > (double)cap) { capped[j] = true; x[j] = (double)cap; }
    }
    // floors and fractional parts
    long long sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const double fl = floor(x[j]);
        e[j] = !live[j] ? 0 : capped[j] ? cap : (int)fl;
        frac[j] = capped[j] ? 0.0 : sub_rn(x[j], fl);
        sum += e[j];
    }
    long long left = Bs - wave_sum_ll(sum);
    // largest remainder, rounds as in allocate_pool
    while (left != 0) {
        const bool give = left > 0;
        const long long want = give ? left : -left;
        bool el[PER];
        double key[PER];
        int rank[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            el[j] = live[j] && !capped[j] && (give ? e[j] < cap : e[j] > 0);
            key[j] = el[j] ? frac[j] : (give ? -1.0 : 2.0);
            rank[j] = 0;
        }
#pragma unroll
        for (int j2 = 0; j2 < PER; ++j2) {
            const int m = min(64, n - 64 * j2);
            for (int l = 0; l < m; ++l) {
                const double o = lane_double(key[j2], l);
                const int oh = 64 * j2 + l;
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    const int h = 64 * j + lane;
                    const bool ahead = give ? (o > frac[j] || (o == frac[j] && oh < h)) : (o < frac[j] || (o == frac[j] && oh > h));
                    rank[j] += ahead ? 1 : 0;
                }
            }
        }
        int granted = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const bool got = el[j] && rank[j] < want;
            if (got) e[j] += give ? 1 : -1;
            granted += __builtin_popcountll(__builtin_amdgcn_ballot_w64(got));
        }
        if (granted == 0) break;                    // cannot happen for valid input (n_keep <= L)
        left = give ? left - granted : left + granted;
    }
    // budgets and their exclusive scan; the scan base is the total of the pools before this one
    long long run = 0;
    for (int s2 = lane; s2 < seg; s2 += 64) run += (long long)n * n_keep_dev(ratio, cu_seq[s2 + 1] - cu_seq[s2]);
    run = wave_sum_ll(run);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int b = live[j] ? f + e[j] : 0;
        long long incl = b;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (live[j]) {
            budgets[(size_t)seg * n + 64 * j + lane] = b;
            cu_budgets[(size_t)seg * n + 64 * j + lane] = (int32_t)(run + incl - b);
        }
        run += __shfl(incl, 63, 64);
    }
    if (lane == 0 && seg == n_segments - 1) cu_budgets[(size_t)n_segments * n] = (int32_t)run;
}

// pool `seg` by the calling wave (pools of up to kAllocateWaveHeads heads)
__device__ __forceinline__ void allocate_small(
    const int seg, const float* __restrict__ weights, int n_segments, int n, int weight_group, int window,
    const int32_t* __restrict__ cu_seq, double ratio, double beta,
    int32_t* __restrict__ budgets, int32_t* __restrict__ cu_budgets)
{
    if (n <= 64) allocate_wave<1>(seg, weights, n_segments, n, weight_group, window, cu_seq, ratio, beta, budgets, cu_budgets);
    else allocate_wave<kAllocateWaveHeads / 64>(seg, weights, n_segments, n, weight_group, window, cu_seq, ratio, beta, budgets, cu_budgets);
}

}  // namespace
}  // namespace audiokv
#endif
