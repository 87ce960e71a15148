// Spectral Score Smoothing of power-of-two lengths, 1024 .. 32768 samples, one workgroup per head (paper Sec. 3.3, Eqs.
// 13-20).
//
// The real sequence is viewed as N = L/2 complex points, transformed in registers and LDS (fft_regs.h), turned into the
// real spectrum bin by bin, masked, turned back and transformed back. A bin k needs its partner N - k; the spectrum goes
// to LDS once for that, every thread reads the partners of its own eight bins and forms its own results (both threads of
// a pair do the pair's arithmetic, and bins whose pair is masked altogether are skipped).
//
// What bounds it is latency: a pass is an LDS round trip of eight points per thread, a radix-8 butterfly and a barrier.
// Three radix-2 stages per pass with the twiddles of the whole transform held in registers (looked up per pass at
// N = 16384, where a thread has sixteen points) take about half the vector instructions of the four stages per
// pass with two complex multiplications per butterfly of smooth_pow2_kernel, which keeps the shorter heads (as fast
// there) and 32768 samples with an energy-adaptive cutoff (52 us for 112 heads there, 54 here). Pool + smooth
// inside evict, before -> now: 4 heads of 2048 12.0 -> 8.0 us, 112 heads of 8192 23 -> 13.2, of 32768 55 -> 42; smooth calls:
// 112 heads of 16384 21.2 -> 13.6 us, with an energy-adaptive cutoff 4 heads of 8192 19.3 -> 13.5. Error against 64 bits
// (2-norm, relative, mean of 36 sequences), smooth_pow2_kernel -> this: 2048 1.21e-7 -> 0.99e-7, 8192 1.24e-7 -> 1.05e-7, 32768
// 1.17e-7 -> 1.14e-7 (1.26e-7 with roots from a float32 polynomial, 1.18e-7 with float32 products of two table entries).
#include <algorithm>
#include <atomic>

#include "fft_regs.h"
#include "select_head.h"
#include "smooth_real.h"

namespace audiokv {
namespace {

// N = 16384: 1024 threads with two groups of eight points each
template <int LOGC> constexpr int kRealGroups = LOGC == 14 ? 2 : 1;
template <int LOGC> constexpr int kRealThreads = (1 << LOGC) / (8 * kRealGroups<LOGC>);

template <int LOGC>
struct RealLds {
    static constexpr bool kTable = LOGC <= 13;               // the whole root table fits beside the points, otherwise a quarter
    cf z[padded_len((size_t)1 << LOGC)];                     // also: raw samples, bin energies
    cf roots[padded_len((size_t)1 << (kTable ? LOGC - 1 : LOGC - 3))];
    double part[32];                                         // partial sums of the energy search, one per wave
    int cross_wave, kstar;
};

// a value of a lane that the DPP control names, 0 where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_scan(double v) {      // inclusive, over a full wave, without LDS
    v = dpp_add<0x111, 0xf>(v);                              // row_shr 1, 2, 4, 8: prefixes within 16 lanes
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);                              // row_bcast 15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);                           // row_bcast 31 into rows 2 and 3
}

// Adaptive cutoff (Eqs. 14-16): the smallest k >= first with sum_{first<=i<=k} e[i] >= rho * sum_{first<=i<n_bins} e[i].
// Bin energies fp32, sums float64: every thread adds a run of PER consecutive bins, all requested at once, the runs' totals are
// scanned, and the thread whose run crosses the target walks it again. Uniform result. (Runs read one bin after the other and a
// scan by LDS permutes: smooth calls on four heads of 8192 13.2 -> 12.6 us, of 2048 10.0 -> 9.1. Runs kept in registers for the second
// walk cost all threads what one reads in a moment.)
template <int T, int PER, class Lds>
__device__ __forceinline__ int energy_search(const float* e, int n_bins, int first, double rho, Lds& m) {
    constexpr int kWaves = (T + 63) / 64;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int k0 = t * PER;                                  // (the last threads may have no bins)
    const auto counts = [&](int u) { return k0 + u >= first && k0 + u < n_bins; };
    double mine = 0.0;
    {
        float run[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) run[u] = e[min(k0 + u, n_bins - 1)];
#pragma unroll
        for (int u = 0; u < PER; ++u) mine += counts(u) ? (double)run[u] : 0.0;
    }
    double incl = wave_scan(mine);
    if (lane == 63) m.part[wave] = incl;
    if (t == 0) { m.cross_wave = T; m.kstar = min(first, n_bins - 1); }
    __syncthreads();
    double total = 0.0, before = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w == wave) before = total;
        total += m.part[w];
    }
    incl += before;
    const double target = rho * total;
    if (target > 0.0 && counts(0) | counts(PER - 1) && incl >= target) atomicMin(&m.cross_wave, t);
    __syncthreads();
    if (t == m.cross_wave) {
        double acc = incl - mine;
        int ks = min(k0 + PER, n_bins) - 1;                  // (rounding between the two summation orders)
        float run[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) run[u] = e[min(k0 + u, n_bins - 1)];
        bool found = false;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (counts(u)) acc += (double)run[u];
            if (counts(u) && !found && acc >= target) { ks = k0 + u; found = true; }
        }
        m.kstar = ks;
    }
    __syncthreads();
    // (the total is added up in another order than the prefixes: at rho = 1 all of them may stay an ulp below it)
    return target > 0.0 && m.cross_wave == T ? n_bins - 1 : m.kstar;
}

// weight of bin k (Eqs. 17-18)
__device__ __forceinline__ float bin_weight(int k, int kstar, int T) {
    if (k <= kstar) return 1.f;
    if (k > kstar + T) return 0.f;
    return 0.5f * (1.f + cis_pi((float)(k - kstar) / (float)(T + 1)).re);
}

// POOL: 0 none, 7 the usual size, 1 any size up to 9. KEEP: the result is left in LDS as well, from smem on, for whoever passes the
// next barrier.
template <int LOGC, int POOL, bool ENERGY, bool KEEP = false>
__device__ __forceinline__ void smooth_real_head(
    const Geom& g, const float* __restrict__ src, double cutoff_frac, float alpha, float* __restrict__ dst,
    int32_t* __restrict__ kstar_out, int cutoffs_only, unsigned char* smem)
{
    constexpr int VT = kRealGroups<LOGC>;
    using F = Fft<LOGC, VT>;
    constexpr int N = 1 << LOGC, L = 2 * N, T = F::THREADS;
    RealLds<LOGC>& m = *reinterpret_cast<RealLds<LOGC>*>(smem);
    const int head = blockIdx.x;
    int t = threadIdx.x;

    // ---- samples 2 n, 2 n + 1 of the points n of the first layout ----
    cf v[VT][8];
    if constexpr (POOL != 0) {
        // one coalesced read of the raw scores into LDS, pooled from there
        float* raw = reinterpret_cast<float*>(m.z);
        float x[L / T];
#pragma unroll
        for (int u = 0; u < L / T; ++u) x[u] = src[t + u * T];
#pragma unroll
        for (int u = 0; u < L / T; ++u) raw[t + u * T] = x[u];
    } else {
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int n = t + vt * T + (N / 8) * q;
                v[vt][q] = {src[2 * n], src[2 * n + 1]};
            }
    }
    if constexpr (RealLds<LOGC>::kTable) F::fill_table(m.roots, t);
    else F::fill_every_fourth(m.roots, t);
    __syncthreads();
    if constexpr (POOL != 0) {
        const float* raw = reinterpret_cast<const float*>(m.z);
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int n = t + vt * T + (N / 8) * q;
                if constexpr (POOL == 7) pooled_pair_lds<7>(raw, L, 2 * n, g.pool_mode, v[vt][q].re, v[vt][q].im);
                else pooled_pair(raw, L, 2 * n, g.pool_kernel, g.pool_mode, v[vt][q].re, v[vt][q].im);
            }
        __syncthreads();
    }
    auto transforms = [&](const auto& tw) {
        F::forward(v, m.z, tw, t);

        // ---- real spectrum, mask, and back ----
        // X_k = E + w^k O with E, O the transforms of the even and odd samples, both read off Z[k] and conj(Z[N-k])
        F::put_last(m.z, v, t);
        __syncthreads();
        const int Tb = g.taper_bins;
        const int first = g.cutoff_mode == AUDIOKV_CUTOFF_ENERGY_NO_DC ? 1 : 0;
        int kstar = (int)floor(cutoff_frac * (double)N);     // N = floor(L/2) = bins - 1
        const cf z0 = m.z[0];
        auto partner = [&](int k) { return cconj(m.z[pad(F::slot_of((N - k) & (N - 1)))]); };
        auto even_odd = [&](cf A, cf B, cf& E, cf& O) {
            E = {0.5f * (A.re + B.re), 0.5f * (A.im + B.im)};
            const cf d = csub(A, B);
            O = {0.5f * d.im, -0.5f * d.re};                 // -i (A - B) / 2
        };
        static_assert(!ENERGY || VT == 1, "sixteen points and sixteen partners per thread do not fit 128 registers");
        cf other[VT][8];                                     // (filled where the energies need every bin)
        typename F::BinRoots roots_of_bins(t);
        if constexpr (ENERGY) {
            float en[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = F::bin_of(8 * t + e);
                other[0][e] = partner(k);
                cf E, O;
                even_odd(v[0][e], other[0][e], E, O);
                const cf X = cadd(E, mul(roots_of_bins(e), O));
                en[e] = fmaf(X.re, X.re, X.im * X.im);
                if (k == 0) { const float x = z0.re + z0.im; en[e] = x * x; }
            }
            __syncthreads();                                 // all partners are read
            float* ek = reinterpret_cast<float*>(m.z);
#pragma unroll
            for (int e = 0; e < 8; ++e) ek[F::bin_of(8 * t + e)] = en[e];
            if (t == 0) { const float x = z0.re - z0.im; ek[N] = x * x; }
            __syncthreads();
            kstar = energy_search<T, N / T + 1>(ek, N + 1, first, cutoff_frac, m);
            __syncthreads();
#if defined(__HIP_DEVICE_COMPILE__)
            // (what the energies were made of is formed again below: kept across the search it takes 40 registers)
            asm volatile("" : "+v"(roots_of_bins.base.re), "+v"(roots_of_bins.base.im), "+v"(t));
#pragma unroll
            for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(other[0][e].re), "+v"(other[0][e].im));
#endif
        }
        if constexpr (!KEEP) {                               // (with KEEP other waves count on every barrier to the end)
            if (kstar_out && t == 0) kstar_out[head] = kstar;
            if (cutoffs_only) return;
            if (degenerate_mask(L, kstar, Tb) == 2) {
                // every bin kept: the samples themselves (a fixed cutoff that says so never gets here)
                for (int n = t; n < L; n += T) dst[n] = POOL ? pooled_at(src, L, n, g.pool_kernel, g.pool_mode) : src[n];
                return;
            }
        }
        const int ktop = kstar + Tb;                         // last bin with a non-zero weight
        // bin k and its pair N - k, weighted and merged into what the backward transform takes in the slot of k
        auto merged = [&](bool dc, cf A, auto B, auto root, auto weight, auto weight_n) -> cf {
            if (dc) {                                        // the DC bin, always kept, with the Nyquist bin folded in
                const float X0 = z0.re + z0.im, XN = (z0.re - z0.im) * weight_n();
                return {0.5f * (X0 + XN), 0.5f * (X0 - XN)};
            }
            cf E, O;
            even_odd(A, B(), E, O);
            const cf Wk = root();
            const float wk = weight(), wn = weight_n();
            const cf WO = mul(Wk, O), X = cadd(E, WO), Y = csub(E, WO);          // bin k; conjugate of bin N - k
            const cf Xk = {X.re * wk, X.im * wk}, Xn = {Y.re * wn, Y.im * wn};
            const cf E2 = {0.5f * (Xk.re + Xn.re), 0.5f * (Xk.im + Xn.im)};
            const cf O2 = mul({0.5f * (Xk.re - Xn.re), 0.5f * (Xk.im - Xn.im)}, cconj(Wk));
            return {E2.re - O2.im, E2.im + O2.re};
        };
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) {
            if constexpr (ENERGY && LOGC <= 12) {
                // All bins are at hand and many are kept: four at a time without branches, the weights of a hard mask without the
                // taper's arithmetic (calls on four heads of 2048 9.19 -> 8.56 us, of 8192 12.3 -> 11.9, 112 of 8192 12.8 -> 12.3).
                // With a fixed cutoff most pairs are skipped, and the registers cost a workgroup per CU (320 heads of 8192 11.3 ->
                // 15.9).
                constexpr int U = 4;
#pragma unroll
                for (int e0 = 0; e0 < 8; e0 += U) {
                    float wk[U], wn[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = F::bin_of(8 * t + e0 + u);
                        wk[u] = k <= kstar ? 1.f : 0.f;
                        wn[u] = N - k <= kstar ? 1.f : 0.f;
                    }
                    if (Tb > 0)                              // (uniform)
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int k = F::bin_of(8 * t + e0 + u);
                            wk[u] = bin_weight(k, kstar, Tb);
                            wn[u] = bin_weight(N - k, kstar, Tb);
                        }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int e = e0 + u, k = F::bin_of(8 * t + e);
                        const cf o = merged(e == 0 && k == 0, v[0][e], [&] { return other[0][e]; }, [&] { return roots_of_bins(e); }, [&] { return wk[u]; },
                                            [&] { return wn[u]; });
                        // (nothing of a pair that is masked altogether: not even the NaN of an infinity times zero)
                        const bool none = k > ktop && N - k > ktop;
                        v[0][e] = {none ? 0.f : o.re, none ? 0.f : o.im};
                    }
                }
            } else {
                const typename F::BinRoots root = ENERGY ? roots_of_bins : typename F::BinRoots(t + vt * T);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int k = F::bin_of(8 * (t + vt * T) + e);
                    cf o = {0.f, 0.f};
                    if (k <= ktop || N - k <= ktop)
                        o = merged(k == 0, v[vt][e], [&] { return ENERGY ? other[vt][e] : partner(k); }, [&] { return root(e); },
                                   [&] { return bin_weight(k, kstar, Tb); }, [&] { return bin_weight(N - k, kstar, Tb); });
                    v[vt][e] = o;
                }
            }
        }
        __syncthreads();                                     // all partners are read: the slots are free
        F::backward(v, m.z, tw, t);

        // residual mix (Eq. 20); 1/N completes the inverse transform
        const float inv = 1.0f / (float)N;
        float* kept = reinterpret_cast<float*>(m.z);
        if constexpr (KEEP) __syncthreads();                 // all points are read
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int n = t + vt * T + (N / 8) * q;
                float o0 = v[vt][q].re * inv, o1 = v[vt][q].im * inv;
                if (alpha != 1.f) {
                    float a0, a1;
                    if constexpr (POOL != 0) {
                        a0 = pooled_at(src, L, 2 * n, g.pool_kernel, g.pool_mode);
                        a1 = pooled_at(src, L, 2 * n + 1, g.pool_kernel, g.pool_mode);
                    } else {
                        a0 = src[2 * n]; a1 = src[2 * n + 1];
                    }
                    o0 = mix(a0, o0, alpha);
                    o1 = mix(a1, o1, alpha);
                }
                dst[2 * n] = o0;
                dst[2 * n + 1] = o1;
                if constexpr (KEEP) { kept[2 * n] = o0; kept[2 * n + 1] = o1; }
            }
    };
    if constexpr (RealLds<LOGC>::kTable) {
        typename F::Twiddles tw;
        F::init(tw, m.roots, t);
        transforms(tw);
    } else {
        transforms(typename F::EveryFourth(m.roots, t));
    }
}

// length and place of the head of a workgroup
__device__ __forceinline__ int head_span(const Geom& g, const int32_t* __restrict__ cu_seq, int head, size_t& off) {
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tok0 = cu_seq[item], L = cu_seq[item + 1] - tok0;
    off = (size_t)tok0 * g.H_kv + (size_t)h * L;
    return L;
}

// ENERGY: the cutoff is energy-adaptive. As a branch in one kernel its bins and partners cost the fixed cutoff registers too: with
// 16384 samples it spilled, with 8192 a CU held one workgroup instead of two. Smooth calls, in one kernel and apart: fixed cutoff 192
// heads of 16384 15.4 and 14.3 us, 320 of 8192 15.0 and 11.3; energy-adaptive 320 of 8192 25.3 and 18.4, 192 of 16384 23.0 and 21.6.
// (N = 16384 is not built with an energy-adaptive cutoff: sixteen points and sixteen partners per thread do not fit 128 registers)
template <int LOGC, int POOL, bool ENERGY>
__global__ __launch_bounds__(kRealThreads<LOGC>) void smooth_real_kernel(
    Geom g, const float* __restrict__ in, const int32_t* __restrict__ cu_seq, double cutoff_frac, float alpha,
    float* __restrict__ out, int32_t* __restrict__ kstar_out, int cutoffs_only)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    size_t off;
    if (head_span(g, cu_seq, blockIdx.x, off) != 2 << LOGC) return;      // another launch's head
    smooth_real_head<LOGC, POOL, ENERGY>(g, in + off, cutoff_frac, alpha, out + off, kstar_out, cutoffs_only, smem);
}

// The barriers of smooth_real_head with a fixed cutoff, pooled on load and kept: filling, pooling, the spectrum's exchange (two) and the
// result, and those of the transforms (tests/test_fused_barriers.py counts them in the built kernels).
template <int LOGC> constexpr int kRealBarriers = 5 + 2 * Fft<LOGC, kRealGroups<LOGC>>::BARRIERS;

// Smoothing and selection of a head in one workgroup: the scores go from one to the other through LDS. In place of two launches, of
// which the second waits for the first to drain, starts and reads the scores again (evict, two launches and one: four heads of 1024
// 23.3 and 21.8 us, 2048 25.0 and 23.6, 8192 34.7 and 32.9, 16384 50.6 and 48.9; 112 heads of 2048 90.3 and 87.1, of 8192 with a decoding
// step 280 and 276). The waves that the transform does not need pass its barriers.
template <int LOGC> constexpr int kFusedThreads = LOGC <= 10 ? 512 : 1024;
template <int LOGC> constexpr int kFusedTokens = LOGC <= 11 ? 4 : 1 << (LOGC - 9);      // per thread
template <int LOGC>
__global__ __launch_bounds__(kFusedThreads<LOGC>) void smooth_select_kernel(
    Geom g, const float* __restrict__ in, const int32_t* __restrict__ cu_seq, double cutoff_frac, float alpha, float* __restrict__ out,
    SelectJob job)
{
    constexpr int NT = kFusedThreads<LOGC>, EPT = kFusedTokens<LOGC>, L = 2 << LOGC;
    static_assert(EPT * NT >= L, "a head's tokens");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    size_t off;
    if (head_span(g, cu_seq, blockIdx.x, off) != L) return;              // (uniform; the launch has heads of this length only)
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) < kRealThreads<LOGC> / 64)
        smooth_real_head<LOGC, 7, false, true>(g, in + off, cutoff_frac, alpha, out + off, nullptr, 0, smem);
    else
#pragma unroll 1
        for (int i = 0; i < kRealBarriers<LOGC>; ++i) __syncthreads();
    __syncthreads();
    const float* kept = reinterpret_cast<const float*>(smem);
    select_head<EPT, NT>(g, blockIdx.x, L, job.budgets, job.cu_b, job.indices, [&](float (&x)[EPT], int n_cand) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int n = (int)threadIdx.x + e * NT;
            x[e] = n < n_cand ? kept[n] : 0.f;
        }
    });
}

// A call of several lengths: all heads in one launch, as many threads as the longest takes. The waves that a shorter head does
// not need end at once (a barrier waits for the waves that are left). One launch per length instead would add up the times of
// what runs side by side here: one call of four heads each of 1024, 2048, .. 16384 samples took 40.1 us, 13.5 in one launch (longest alone 13.8).
template <int POOL, bool ENERGY>
__global__ __launch_bounds__(1024) void smooth_mixed_kernel(
    Geom g, const float* __restrict__ in, const int32_t* __restrict__ cu_seq, double cutoff_frac, float alpha,
    float* __restrict__ out, int32_t* __restrict__ kstar_out, int cutoffs_only, unsigned lengths)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    size_t off;
    const int L = head_span(g, cu_seq, blockIdx.x, off);
    if ((L & (L - 1)) != 0 || !(lengths & (unsigned)L)) return;          // uniform
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#define AUDIOKV_MIXED(LOGC)                                                                                               \
    case 2 << LOGC:                                                                                                      \
        if (wave < kRealThreads<LOGC> / 64)                                                                               \
            smooth_real_head<LOGC, POOL, ENERGY>(g, in + off, cutoff_frac, alpha, out + off, kstar_out, cutoffs_only, smem); \
        break
    switch (L) {
        AUDIOKV_MIXED(9);
        AUDIOKV_MIXED(10);
        AUDIOKV_MIXED(11);
        AUDIOKV_MIXED(12);
        AUDIOKV_MIXED(13);
        case 2 << 14:
            if constexpr (!ENERGY)
                smooth_real_head<14, POOL, false>(g, in + off, cutoff_frac, alpha, out + off, kstar_out, cutoffs_only, smem);
            break;
    }
#undef AUDIOKV_MIXED
}

size_t real_lds(int L) {
    switch (L) {
        case 1024:  return sizeof(RealLds<9>);
        case 2048:  return sizeof(RealLds<10>);
        case 4096:  return sizeof(RealLds<11>);
        case 8192:  return sizeof(RealLds<12>);
        case 16384: return sizeof(RealLds<13>);
        default:    return sizeof(RealLds<14>);
    }
}

template <int POOL, bool ENERGY>
hipError_t launch_mixed(unsigned lengths, const Geom& g, const float* in, const int32_t* cu_seqlens, double cutoff_frac, float alpha,
                        float* out, int32_t* kstar_out, bool cutoffs_only, hipStream_t s) {
    const int longest = 1 << (31 - __builtin_clz(lengths));
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(smooth_mixed_kernel<POOL, ENERGY>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(RealLds<14>));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((smooth_mixed_kernel<POOL, ENERGY>), dim3((unsigned)(g.n_items * g.H_kv)), dim3(std::min(longest / 16, 1024)),
                       real_lds(longest), s, g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only ? 1 : 0, lengths);
    return hipGetLastError();
}

template <int LOGC, int POOL, bool ENERGY>
hipError_t launch(const Geom& g, const float* in, const int32_t* cu_seqlens, double cutoff_frac, float alpha, float* out,
                  int32_t* kstar_out, bool cutoffs_only, hipStream_t s) {
    constexpr int T = kRealThreads<LOGC>;
    const int lds = (int)sizeof(RealLds<LOGC>);
    if (lds > 48 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(smooth_real_kernel<LOGC, POOL, ENERGY>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((smooth_real_kernel<LOGC, POOL, ENERGY>), dim3((unsigned)(g.n_items * g.H_kv)), dim3(T), lds, s, g, in, cu_seqlens,
                       cutoff_frac, alpha, out, kstar_out, cutoffs_only ? 1 : 0);
    return hipGetLastError();
}

template <int LOGC, bool ENERGY>
hipError_t launch(const Geom& g, const float* in, bool pool_on_load, const int32_t* cu_seqlens, double cutoff_frac, float alpha,
                  float* out, int32_t* kstar_out, bool cutoffs_only, hipStream_t s) {
    if (!pool_on_load) return launch<LOGC, 0, ENERGY>(g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
    if (g.pool_kernel == 7) return launch<LOGC, 7, ENERGY>(g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
    return launch<LOGC, 1, ENERGY>(g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
}

template <bool ENERGY>
hipError_t launch_lengths(unsigned lengths, const Geom& g, const float* in, bool pool_on_load, const int32_t* cu_seqlens, double cutoff_frac,
                          float alpha, float* out, int32_t* kstar_out, bool cutoffs_only, hipStream_t s) {
    if (ENERGY && lengths >= 32768) return hipErrorInvalidValue;
    if (lengths & (lengths - 1)) {
        if (!pool_on_load) return launch_mixed<0, ENERGY>(lengths, g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        if (g.pool_kernel == 7) return launch_mixed<7, ENERGY>(lengths, g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        return launch_mixed<1, ENERGY>(lengths, g, in, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
    }
    switch (lengths) {
        case 1024:  return launch<9, ENERGY>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        case 2048:  return launch<10, ENERGY>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        case 4096:  return launch<11, ENERGY>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        case 8192:  return launch<12, ENERGY>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        case 16384: return launch<13, ENERGY>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
        case 32768:
            if constexpr (!ENERGY) return launch<14, false>(g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
    }
    return hipErrorInvalidValue;
}

template <int LOGC>
hipError_t launch_fused(const Geom& g, const float* in, const int32_t* cu_seqlens, double cutoff_frac, float alpha, float* out,
                        const SelectJob& job, hipStream_t s) {
    const int lds = (int)sizeof(RealLds<LOGC>);
    if (lds > 24 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(smooth_select_kernel<LOGC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((smooth_select_kernel<LOGC>), dim3((unsigned)(g.n_items * g.H_kv)), dim3(kFusedThreads<LOGC>), lds, s, g, in,
                       cu_seqlens, cutoff_frac, alpha, out, job);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_smooth_select(int L, const Geom& g, const float* in, const int32_t* cu_seqlens, double cutoff_frac, float alpha, float* out,
                                const SelectJob& job, hipStream_t s) {
    switch (L) {
        case 1024:  return launch_fused<9>(g, in, cu_seqlens, cutoff_frac, alpha, out, job, s);
        case 2048:  return launch_fused<10>(g, in, cu_seqlens, cutoff_frac, alpha, out, job, s);
        case 4096:  return launch_fused<11>(g, in, cu_seqlens, cutoff_frac, alpha, out, job, s);
        case 8192:  return launch_fused<12>(g, in, cu_seqlens, cutoff_frac, alpha, out, job, s);
        case 16384: return launch_fused<13>(g, in, cu_seqlens, cutoff_frac, alpha, out, job, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_smooth_real(unsigned lengths, const Geom& g, const float* in, bool pool_on_load, const int32_t* cu_seqlens, double cutoff_frac,
                              float alpha, float* out, int32_t* kstar_out, bool cutoffs_only, hipStream_t s) {
    if (g.cutoff_mode == AUDIOKV_CUTOFF_FRACTION)
        return launch_lengths<false>(lengths, g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
    return launch_lengths<true>(lengths, g, in, pool_on_load, cu_seqlens, cutoff_frac, alpha, out, kstar_out, cutoffs_only, s);
}

}  // namespace audiokv
