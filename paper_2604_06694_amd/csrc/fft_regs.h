// In-place power-of-two transforms with eight points per thread in registers, for the smoothing kernels.
#pragma once

#include <type_traits>

#include "smooth_common.h"

// Every fused multiply-add is written out: the kernels that use this exist in several instantiations (pooling on load or
// not, a filter formed here or there) that have to agree to the last bit, and what the compiler contracts is up to each.
#pragma clang fp contract(off)

namespace audiokv {
namespace {

__host__ __device__ __forceinline__ cf mul(cf a, cf b) {
    return {fmaf(a.re, b.re, -(a.im * b.im)), fmaf(a.re, b.im, a.im * b.re)};
}
// Eq. 20
__device__ __forceinline__ float mix(float s0, float smoothed, float alpha) { return fmaf(alpha, smoothed, (1.f - alpha) * s0); }


// exp(i pi x), |x| <= 2^16: x - k/2 is exact, and on [-1/4, 1/4] the Taylor series of cos and sin in float64 (remainders
// below 4e-13 and, relative, 9.8e-12; a float64 multiply-add issues as fast as a float32 one here). Roots, twists and what splits
// and merges real spectra are float64 values rounded to float32 once, products among them; only a transform that keeps three
// roots per radix-8 butterfly (ALL = false) derives the other four as float32 products.
struct cd { double re, im; };
__host__ __device__ __forceinline__ cd cis_pi_f64(float x) {
    const float k = rintf(2.f * x), r = fmaf(-0.5f, k, x);
    const int q = (int)k;
    const double t = 3.14159265358979324 * (double)r, u = t * t;
    const double c = fma(u, fma(u, fma(u, fma(u, fma(u, fma(u, 1. / 479001600., -1. / 3628800.), 1. / 40320.), -1. / 720.), 1. / 24.), -0.5), 1.);
    const double v = t * fma(u, fma(u, fma(u, fma(u, fma(u, -1. / 39916800., 1. / 362880.), -1. / 5040.), 1. / 120.), -1. / 6.), 1.);
    const double a = q & 1 ? v : c, b = q & 1 ? c : v;                              // quarter turns: swap, then signs
    return {(q + 1) & 2 ? -a : a, q & 2 ? -b : b};
}
__host__ __device__ __forceinline__ cf rounded(cd a) { return {(float)a.re, (float)a.im}; }
__host__ __device__ __forceinline__ cf cis_pi(float x) { return rounded(cis_pi_f64(x)); }
__host__ __device__ __forceinline__ cf mul_rounded(cd a, cd b) {
    return {(float)fma(a.re, b.re, -(a.im * b.im)), (float)fma(a.re, b.im, a.im * b.re)};
}

// exp(-i pi k / n), 0 <= k < n, in constants
constexpr cd unit_root(int k, int n) {
    const double x = 3.14159265358979324 * k / n;
    double c = 0., s = 0., term = 1.;
    for (int j = 0; j < 30; j += 2) {                        // pi^30 / 30! < 4e-18
        c += term;
        s -= term * x / (j + 1);
        term *= -x * x / ((j + 1) * (j + 2));
    }
    return {c, s};
}

// 4- and 8-point DFTs in registers, natural order in and out; S = -1 forwards (exp(-2 pi i / n)), +1 backwards
template <int S>
__device__ __forceinline__ cf mul_i(cf a) { return S < 0 ? cf{a.im, -a.re} : cf{-a.im, a.re}; }     // times S * i
template <int S>
__device__ __forceinline__ void dft4(cf& a, cf& b, cf& c, cf& d) {
    const cf s0 = cadd(a, c), s1 = csub(a, c), s2 = cadd(b, d), s3 = mul_i<S>(csub(b, d));
    a = cadd(s0, s2); b = cadd(s1, s3); c = csub(s0, s2); d = csub(s1, s3);
}
template <int S>
__device__ __forceinline__ void dft8(cf (&v)[8]) {
    constexpr float H = 0.70710678118654752f;
    cf e0 = cadd(v[0], v[4]), e1 = cadd(v[1], v[5]), e2 = cadd(v[2], v[6]), e3 = cadd(v[3], v[7]);
    cf o0 = csub(v[0], v[4]), o1 = csub(v[1], v[5]), o2 = csub(v[2], v[6]), o3 = csub(v[3], v[7]);
    o1 = S < 0 ? cf{H * (o1.re + o1.im), H * (o1.im - o1.re)} : cf{H * (o1.re - o1.im), H * (o1.im + o1.re)};
    o2 = mul_i<S>(o2);
    o3 = S < 0 ? cf{H * (o3.im - o3.re), -H * (o3.re + o3.im)} : cf{-H * (o3.re + o3.im), H * (o3.re - o3.im)};
    dft4<S>(e0, e1, e2, e3);
    dft4<S>(o0, o1, o2, o3);
    v[0] = e0; v[2] = e1; v[4] = e2; v[6] = e3;
    v[1] = o0; v[3] = o1; v[5] = o2; v[7] = o3;
}

// In-place transforms of C = 2^LOGC points by C / (8 VT) threads of VT virtual threads each. Forwards the passes take the
// index bits from the top, three at a time, and leave every group's outputs where its inputs were, so the bins end in a
// digit-reversed order (bin_of, slot_of); backwards the passes mirror it.
//   first layout: virtual thread t holds points t + (C/8) q;  last layout: it holds slots 8 t + e  (e, q = 0..7)
// Virtual threads of thread x: x, x + THREADS.
// ALL: the seven roots of every radix-8 butterfly in registers, all of them rounded once, instead of three that the others are
// products of.
template <int LOGC, int VT = 1, bool ALL = false>
struct Fft {
    static constexpr int C = 1 << LOGC, THREADS = C / (8 * VT);
    static constexpr int P8 = LOGC / 3;                       // radix-8 passes
    static constexpr int REM = LOGC - 3 * P8;                 // bits left for a pass of radix 2 or 4 on the last layout
    static constexpr int TW = REM ? P8 : P8 - 1;              // passes with twiddles
    static constexpr int BARRIERS = P8 - (REM ? 0 : 1);       // of forward, and of backward
    __host__ __device__ static constexpr int low_bit(int p) { return LOGC - 3 * (p + 1); }

    struct W3 { cf w1, w2, w4; };
    struct W7 { cf w1, w2, w4, w3, w5, w6, w7; };
    using W = std::conditional_t<ALL, W7, W3>;
    // root_{8m}^(j0 {1, 2, 4}) per pass, in registers, from a table of exp(-2 pi i e / C) at pad(e), e < C/2
    struct Twiddles {
        W w[VT][TW];
        __device__ __forceinline__ W operator()(int p, int vt) const { return w[vt][p]; }
    };
    // The same looked up where they are used, from a table of every fourth root, exp(-2 pi i 4 j / C) at pad(j). Only the first
    // pass has exponents between them: w + w (root - 1), whose second term is too small for its roundings to matter.
    struct EveryFourth {
        const cf* table; int t; cf m1, m2;
        __host__ __device__ __forceinline__ EveryFourth(const cf* table_, int t_) : table(table_), t(t_) {
            const cd a = cis_pi_f64(-(float)(t & 3) / (float)(C / 2)), b = cis_pi_f64(-(float)(2 * (t & 1)) / (float)(C / 2));
            m1 = rounded({a.re - 1., a.im});
            m2 = rounded({b.re - 1., b.im});
        }
        __host__ __device__ __forceinline__ cf near(int e, cf m) const {
            const cf w = table[pad(e >> 2)], d = mul(w, m);
            return cadd(w, d);
        }
        __host__ __device__ __forceinline__ W3 operator()(int p, int vt) const {
            const int e = exponent(p, t + vt * THREADS);
            if (p == 0) return {near(e, m1), near(2 * e, m2), table[pad(e)]};
            return {table[pad(e >> 2)], table[pad(e >> 1)], table[pad(e)]};
        }
    };
    __host__ __device__ __forceinline__ static int exponent(int p, int t) { return (t & ((1 << low_bit(p)) - 1)) << (3 * p); }   // 4 e < C/2

    __device__ __forceinline__ static int base(int p, int t) {
        const int sb = low_bit(p);
        return ((t >> sb) << (sb + 3)) | (t & ((1 << sb) - 1));
    }
    __host__ __device__ __forceinline__ static constexpr int bin_of(int slot) {
        int k = (slot & ((1 << REM) - 1)) << (3 * P8);
#pragma unroll
        for (int p = 0; p < P8; ++p) k |= ((slot >> low_bit(p)) & 7) << (3 * p);
        return k;
    }
    __device__ __forceinline__ static int slot_of(int bin) {
        int s = bin >> (3 * P8);
#pragma unroll
        for (int p = 0; p < P8; ++p) s |= ((bin >> (3 * p)) & 7) << low_bit(p);
        return s;
    }
    // exp(-2 pi i e / C) at pad(e) for e = t + (C/8) u, u < 4: eighth turns apart
    __host__ __device__ __forceinline__ static void fill_table(cf* table, int t) {
        static_assert(VT == 1, "four entries per thread");
        const cd w = cis_pi_f64(-(float)t / (float)(C / 2));
        const double H = 0.70710678118654752, p = H * (w.re + w.im), q = H * (w.im - w.re);
        table[pad(t)] = rounded(w);
        table[pad(t + C / 8)] = {(float)p, (float)q};
        table[pad(t + C / 4)] = {(float)w.im, (float)-w.re};
        table[pad(t + 3 * C / 8)] = {(float)q, (float)-p};
    }
    // exp(-2 pi i 4 j / C) for j = t, t + C/16: a quarter turn apart
    __host__ __device__ __forceinline__ static void fill_every_fourth(cf* table, int t) {
        static_assert(VT == 2, "two entries per thread");
        const cf w = cis_pi(-(float)t / (float)(C / 8));
        table[pad(t)] = w;
        table[pad(t + C / 16)] = {w.im, -w.re};
    }
    // exp(-i pi k / C) for the bins k of slots 8 t + e: from that of e = 0 and eight constants
    struct BinRoots {
        cd base;
        __host__ __device__ __forceinline__ explicit BinRoots(int t) : base(cis_pi_f64(-(float)bin_of(8 * t) / (float)C)) {}
        __host__ __device__ __forceinline__ cf operator()(int e) const {
            constexpr cd step[8] = {unit_root(bin_of(0), C), unit_root(bin_of(1), C), unit_root(bin_of(2), C), unit_root(bin_of(3), C),
                                    unit_root(bin_of(4), C), unit_root(bin_of(5), C), unit_root(bin_of(6), C), unit_root(bin_of(7), C)};
            return mul_rounded(base, step[e]);
        }
    };
    __host__ __device__ __forceinline__ static void init(Twiddles& tw, const cf* table, int t) {
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int p = 0; p < TW; ++p) {
                const int e = exponent(p, t + vt * THREADS);
                tw.w[vt][p].w1 = table[pad(e)];
                tw.w[vt][p].w2 = table[pad(2 * e)];
                tw.w[vt][p].w4 = table[pad(4 * e)];
                if constexpr (ALL) {
                    auto root = [&](int k) {                 // the second half of the circle: negated
                        const cf r = table[pad(k & (C / 2 - 1))];
                        return k & (C / 2) ? cf{-r.re, -r.im} : r;
                    };
                    tw.w[vt][p].w3 = root(3 * e);
                    tw.w[vt][p].w5 = root(5 * e);
                    tw.w[vt][p].w6 = root(6 * e);
                    tw.w[vt][p].w7 = root(7 * e);
                }
            }
    }
    template <bool CONJ>
    __device__ __forceinline__ static void twist(cf (&v)[8], const W7& w) {
        auto at = [](cf r) { return CONJ ? cconj(r) : r; };
        v[1] = mul(v[1], at(w.w1)); v[2] = mul(v[2], at(w.w2)); v[3] = mul(v[3], at(w.w3)); v[4] = mul(v[4], at(w.w4));
        v[5] = mul(v[5], at(w.w5)); v[6] = mul(v[6], at(w.w6)); v[7] = mul(v[7], at(w.w7));
    }
    template <bool CONJ>
    __device__ __forceinline__ static void twist(cf (&v)[8], const W3& w) {
        const cf w1 = CONJ ? cconj(w.w1) : w.w1, w2 = CONJ ? cconj(w.w2) : w.w2, w4 = CONJ ? cconj(w.w4) : w.w4, w3 = mul(w1, w2);
        v[1] = mul(v[1], w1); v[2] = mul(v[2], w2); v[3] = mul(v[3], w3); v[4] = mul(v[4], w4);
        v[5] = mul(v[5], mul(w1, w4)); v[6] = mul(v[6], mul(w2, w4)); v[7] = mul(v[7], mul(w3, w4));
    }
    template <int S>
    __device__ __forceinline__ static void small_dfts(cf (&v)[8]) {
        if constexpr (REM == 1) {
#pragma unroll
            for (int e = 0; e < 8; e += 2) { const cf a = v[e], b = v[e + 1]; v[e] = cadd(a, b); v[e + 1] = csub(a, b); }
        } else if constexpr (REM == 2) {
            dft4<S>(v[0], v[1], v[2], v[3]);
            dft4<S>(v[4], v[5], v[6], v[7]);
        }
    }
    __device__ __forceinline__ static void put(cf* z, const cf (&v)[8], int b, int sb) {
#pragma unroll
        for (int q = 0; q < 8; ++q) z[pad(b + (q << sb))] = v[q];
    }
    __device__ __forceinline__ static void get(const cf* z, cf (&v)[8], int b, int sb) {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = z[pad(b + (q << sb))];
    }
    __device__ __forceinline__ static void put_last(cf* z, const cf (&v)[VT][8], int t) {
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) put(z, v[vt], 8 * (t + vt * THREADS), 0);
    }
    // first layout in, last layout out; every thread's own first-layout slots are free
    template <class TWID>
    __device__ __forceinline__ static void forward(cf (&v)[VT][8], cf* z, const TWID& tw, int t) {
#pragma unroll
        for (int p = 0; p < P8; ++p) {
            const int sb = low_bit(p);
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                const int b = base(p, t + vt * THREADS);
                if (p) get(z, v[vt], b, sb);
                dft8<-1>(v[vt]);
                if (p < TW) twist<false>(v[vt], tw(p, vt));
                if (p + 1 < P8 || REM) put(z, v[vt], b, sb);
            }
            if (p + 1 < P8 || REM) __syncthreads();
        }
        if (REM)
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) { get(z, v[vt], 8 * (t + vt * THREADS), 0); small_dfts<-1>(v[vt]); }
    }
    // last layout in (every thread's own last-layout slots are free), first layout out, unnormalised
    template <class TWID>
    __device__ __forceinline__ static void backward(cf (&v)[VT][8], cf* z, const TWID& tw, int t) {
        if (REM) {
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) { small_dfts<1>(v[vt]); put(z, v[vt], 8 * (t + vt * THREADS), 0); }
            __syncthreads();
        }
#pragma unroll
        for (int p = P8 - 1; p >= 0; --p) {
            const int sb = low_bit(p);
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                const int b = base(p, t + vt * THREADS);
                if (p + 1 < P8 || REM) get(z, v[vt], b, sb);
                if (p < TW) twist<true>(v[vt], tw(p, vt));
                dft8<1>(v[vt]);
                if (p) put(z, v[vt], b, sb);
            }
            if (p) __syncthreads();
        }
    }
};

}  // namespace
}  // namespace audiokv
