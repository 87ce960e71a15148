// In-place power-of-two transforms with eight points per thread in registers, for the smoothing kernels.
#pragma once

#include "smooth_common.h"

// Every fused multiply-add is written out: the kernels that use this exist in several instantiations (pooling on load or
// not, a filter formed here or there) that have to agree to the last bit, and what the compiler contracts is up to each.
#pragma clang fp contract(off)

namespace audiokv {
namespace {

__device__ __forceinline__ cf mul(cf a, cf b) {
    return {fmaf(a.re, b.re, -(a.im * b.im)), fmaf(a.re, b.im, a.im * b.re)};
}
// Eq. 20
__device__ __forceinline__ float mix(float s0, float smoothed, float alpha) { return fmaf(alpha, smoothed, (1.f - alpha) * s0); }


// exp(i pi x), |x| <= 2^16: x - k/2 is exact, and on [-1/4, 1/4] the Taylor series of cos and sin (remainders below
// 3e-9 and 3e-10)
__device__ __forceinline__ cf cis_pi(float x) {
    const float k = rintf(2.f * x), r = fmaf(-0.5f, k, x), s = r * r;
    const int q = (int)k;
    constexpr float P2 = 9.86960440108935862f, P1 = 3.14159265358979324f;         // pi^2, pi
    const float u = s * P2;
    const float c = fmaf(u, fmaf(u, fmaf(u, fmaf(u, 1.f / 40320.f, -1.f / 720.f), 1.f / 24.f), -0.5f), 1.f);
    const float v = P1 * r * fmaf(u, fmaf(u, fmaf(u, fmaf(u, 1.f / 362880.f, -1.f / 5040.f), 1.f / 120.f), -1.f / 6.f), 1.f);
    const float a = q & 1 ? v : c, b = q & 1 ? c : v;                               // quarter turns: swap, then signs
    return {(q + 1) & 2 ? -a : a, q & 2 ? -b : b};
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
template <int LOGC, int VT = 1>
struct Fft {
    static constexpr int C = 1 << LOGC, THREADS = C / (8 * VT);
    static constexpr int P8 = LOGC / 3;                       // radix-8 passes
    static constexpr int REM = LOGC - 3 * P8;                 // bits left for a pass of radix 2 or 4 on the last layout
    static constexpr int TW = REM ? P8 : P8 - 1;              // passes with twiddles
    static constexpr int low_bit(int p) { return LOGC - 3 * (p + 1); }

    struct W3 { cf w1, w2, w4; };
    // root_{8m}^(j0 {1, 2, 4}) per pass, in registers, from a table of exp(-2 pi i e / C), e < C/2
    struct Twiddles {
        W3 w[VT][TW];
        __device__ __forceinline__ W3 operator()(int p, int vt) const { return w[vt][p]; }
    };
    // the same looked up where they are used, from exp(-2 pi i e / C) = hi[e >> 7] lo[e & 127]
    struct HiLo {
        const cf* lo; const cf* hi; int t;
        __device__ __forceinline__ cf root(int e) const { return mul(hi[e >> 7], lo[e & 127]); }
        __device__ __forceinline__ W3 operator()(int p, int vt) const {
            const int e = exponent(p, t + vt * THREADS);
            return {root(e), root(2 * e), root(4 * e)};
        }
    };
    __device__ __forceinline__ static int exponent(int p, int t) { return (t & ((1 << low_bit(p)) - 1)) << (3 * p); }   // 4 e < C/2

    __device__ __forceinline__ static int base(int p, int t) {
        const int sb = low_bit(p);
        return ((t >> sb) << (sb + 3)) | (t & ((1 << sb) - 1));
    }
    __device__ __forceinline__ static int bin_of(int slot) {
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
    __device__ __forceinline__ static void fill_table(cf* table, int t) {
#pragma unroll 1
        for (int e = t; e < C / 2; e += THREADS) table[e] = cis_pi(-(float)e / (float)(C / 2));
    }
    // lo: 128 entries, hi: C / 256
    __device__ __forceinline__ static void fill_hi_lo(cf* lo, cf* hi, int t) {
#pragma unroll 1
        for (int e = t; e < 128 + C / 256; e += THREADS) {
            const int n = e < 128 ? e : (e - 128) * 128;
            (e < 128 ? lo[e] : hi[e - 128]) = cis_pi(-(float)n / (float)(C / 2));
        }
    }
    __device__ __forceinline__ static void init(Twiddles& tw, const cf* table, int t) {
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int p = 0; p < TW; ++p) {
                const int e = exponent(p, t + vt * THREADS);
                tw.w[vt][p] = {table[e], table[2 * e], table[4 * e]};
            }
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
