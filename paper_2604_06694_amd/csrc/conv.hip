// Spectral Score Smoothing with a fixed cutoff as a convolution (paper Sec. 3.3, Eqs. 17-20), for lengths that are
// not powers of two.
//
// With the mask known in advance, RFFT -> mask -> IRFFT of a sequence of L samples is a circular convolution of length
// L with the mask's taps h (conv_filter.h). The L samples meet taps h[-(L-1)] .. h[L-1], so the circular convolution
// is a window of a linear one with 2L - 1 taps, and that fits a negacyclic convolution of length 2N, N = the power of
// two >= L (products that wrap around fall outside the window, whatever their sign). A real negacyclic convolution of
// length 2N costs one complex transform of N points each way and no untangling of real spectra:
//     z[n] = (x[n] + i x[n+N]) w^n,  w = exp(i pi / 2N):   polynomials mod X^N - i, of which mod X^N + i is the mirror.
// The samples have x[n+N] = 0, and only the real parts of the first L results are wanted:
//     out[n] = Re( w^-n IFFT_N( FFT_N(s w^n) . FFT_N(g w^n) ) ),   g[n] = h[n] - i h[N-n]
// (a chirp-z transform needs two such convolutions of at least L + K points for K kept bins).
//
// A head runs on R workgroups, one per residue of the bins mod R. Workgroup r forms its own C = N / R point input from
// all R C samples, which costs two multiply-adds per sample because the twist and the R-point butterfly merge into
// R constants, transforms it in LDS, multiplies by the filter's bins and transforms back; conv_join_kernel combines
// the R results. Calls whose lengths are shared by few heads transform the filter inside the same workgroups instead
// of in a launch of its own.
//
// What bounds all of this is latency: the chain of LDS exchanges of a transform (a thread keeps eight points, three
// radix-2 stages per exchange) and the gathers, whose loads go without branches around them, four blocks at a time (with
// the edges of the sequence handled in branches the loads waited for each other and a launch took 36 us at any chunk size).
// Pool + smooth of one layer of four heads inside evict, chirp-z path before -> this: L = 13577 41 us in six launches beside
// 50 us of filter preparation on another stream -> 19 us in two (chunks 14, join 5) and nothing beside; a smooth call on 24
// sequences of two heads, 1500 to 30000 samples, 147 -> 41 us (taps 8, chunks 31, join 4); one layer of 30011 alone 78 -> 22,
// 28 layers 144 -> 68. Error against 64 bits (2-norm, relative, mean of 36 sequences): L = 3000 4.4e-7 -> 1.0e-7, 13577 3.5e-7 -> 1.2e-7,
// 30011 3.1e-7 -> 1.3e-7, 100003 4.3e-7 -> 2.1e-7; much of it is the filter's own transform, a gain that differs from length to
// length (60 lengths and cutoffs: mean 3.9e-7 -> 1.3e-7, 1.5e-7 with three roots per butterfly instead of seven).
#include <atomic>

#include "conv_filter.h"
#include "conv.h"
#include "conv_join.h"
#include "fft_regs.h"
#include "select_head.h"

namespace audiokv {
namespace {

// (the 1024 threads of 8192 points have 128 registers each: too few for all roots)
template <int LOGC> using Cfft = Fft<LOGC, 1, (LOGC < 13)>;

// What both transforms of a workgroup start from: points n = 8 t + e + C k of all R blocks k, weighted by the constants
// c[k], summed over k. U blocks' loads are in flight together, none behind a branch: what lies outside the sequence
// is read and masked where the memory around it is known to be there, and clamped where it is not.

// sum_k s[8 t + e + C k] c[k], zero from L on. POOL != 0: samples pooled; they lie inside a workspace that extends at
// least 16 floats to either side of every head. The first U blocks can be requested ahead of everything else (load).
template <int U, int POOL>
struct SampleBlocks {
    static constexpr int LEN = POOL ? 16 : 8, AT = POOL ? 4 : 0;
    float x[U][LEN];
    __device__ __forceinline__ void load(const float* __restrict__ src, const ConvHead& w, int C, int t, int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n0 = (k0 + u) * C + 8 * t;
            // (blocks past the end: from L on. Unpooled, the last block that holds samples: moved to end at L - 1, undone below)
            if (POOL || w.L >= 8) {                          // (uniform)
                window_load(src + (POOL ? min(n0, w.L) - AT : min(n0, w.L - 8)), x[u]);
            } else {
#pragma unroll
                for (int j = 0; j < LEN; ++j) x[u][j] = src[min(j, w.L - 1)];
            }
        }
    }
    __device__ __forceinline__ void add(const ConvHead& w, int C, int kernel, int mode, const cf* __restrict__ c, int t, int k0, cf (&acc)[8]) {
        const float fill = POOL && mode == AUDIOKV_POOL_MAX ? -INFINITY : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n0 = (k0 + u) * C + 8 * t;
            float o[8];
            if constexpr (POOL != 0) {
                // the first and the last window of a head reach beyond it
                if (n0 < AT || n0 + LEN - AT > w.L) {
#pragma unroll
                    for (int j = 0; j < LEN; ++j) x[u][j] = n0 - AT + j >= 0 && n0 - AT + j < w.L ? x[u][j] : fill;
                }
                pooled_window<POOL>(x[u], kernel, mode, o);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = n0 + e < w.L ? o[e] : 0.f;
            } else {
                const int moved = n0 - max(min(n0, w.L - 8), 0);         // 0 except from the last block on
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = n0 + e < w.L || moved > 0 ? x[u][e] : 0.f;
                if (moved > 0) {
#pragma unroll
                    for (int s = 4; s > 0; s >>= 1)
                        if (moved & s) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) o[e] = e + s < 8 ? o[e + s < 8 ? e + s : 0] : 0.f;
                        }
                    if (moved >= 8) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[e] = 0.f;
                    }
                }
            }
            const cf ck = c[(k0 + u) & 15];                  // (blocks past R hold no samples: their constant is unused)
#pragma unroll
            for (int e = 0; e < 8; ++e) { acc[e].re = fmaf(o[e], ck.re, acc[e].re); acc[e].im = fmaf(o[e], ck.im, acc[e].im); }
        }
    }
    // all blocks; LOADED: the first of them are here already
    template <bool LOADED>
    __device__ __forceinline__ void sum(const float* __restrict__ src, const ConvHead& w, int C, int kernel, int mode, const cf* __restrict__ c,
                                        int t, cf (&acc)[8]) {
        if constexpr (LOADED) add(w, C, kernel, mode, c, t, 0, acc);
#pragma unroll 1
        for (int k0 = LOADED ? U : 0; k0 < w.R; k0 += U) {
            load(src, w, C, t, k0);
            add(w, C, kernel, mode, c, t, k0, acc);
        }
    }
};

// sum_k (h[n] - i h[N - n]) c[k], n = 8 t + e + C k; taps from L on are zero, and so is h[N] for n = 0 (a negacyclic
// sequence has no element N). Memory past the taps is there for 8 floats.
template <int U>
struct TapBlocks {
    float a[U][8], b[U][8];                                  // b holds h[low .. low + 7], low = N - n0 - 7, read forwards
    __device__ __forceinline__ void load(const float* __restrict__ h, const ConvHead& w, int C, int t, int k0) {
        const int N = 1 << w.log_n;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n0 = (k0 + u) * C + 8 * t;
            window_load(h + min(n0, w.L), a[u]);
            window_load(h + min(max(N - n0 - 7, 0), w.L), b[u]);
        }
    }
    __device__ __forceinline__ void add(const ConvHead& w, int C, const cf* __restrict__ c, int t, int k0, cf (&acc)[8]) {
        const int N = 1 << w.log_n;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n0 = (k0 + u) * C + 8 * t, low = N - n0 - 7;       // low >= 1, or <= -7 past the last block
            const cf ck = c[(k0 + u) & 15];
#pragma unroll
            for (int e = 0; e < 8; ++e) {                    // (a - i b) c
                const float p = n0 + e < w.L ? a[u][e] : 0.f;
                const float q = low > 0 && low + 7 - e < w.L ? b[u][7 - e] : 0.f;
                acc[e].re = fmaf(p, ck.re, fmaf(q, ck.im, acc[e].re));
                acc[e].im = fmaf(p, ck.im, fmaf(-q, ck.re, acc[e].im));
            }
        }
    }
    template <bool LOADED>
    __device__ __forceinline__ void sum(const float* __restrict__ h, const ConvHead& w, int C, const cf* __restrict__ c, int t, cf (&acc)[8]) {
        if constexpr (LOADED) add(w, C, c, t, 0, acc);
#pragma unroll 1
        for (int k0 = LOADED ? U : 0; k0 < w.R; k0 += U) {
            load(h, w, C, t, k0);
            add(w, C, c, t, k0, acc);
        }
    }
};

// LDS of a workgroup: the padded points, the roots of unity, and the constants of residue r:
//   c[k] = exp(i pi k (1 - 4 r) / 2R), k < R;  step[e] = exp(i pi e (1 - 4 r) / 2N) and
//   back[q] = exp(i pi q (4 r - 1) / 16 R), e, q < 8: factors of the twists of points 8 t + e and t + (C/8) q
template <int LOGC>
struct ConvLds {
    cf z[padded_len((size_t)1 << LOGC)];
    cf table[padded_len((size_t)1 << (LOGC - 1))];
    cf c[16];
    alignas(16) cd step[8], back[8];         // (factors of products: these are rounded, not their factors)
};
template <int LOGC>
__device__ __forceinline__ void fill_constants(ConvLds<LOGC>& m, const ConvHead& w, int r, int t) {
    Cfft<LOGC>::fill_table(m.table, t);
    if (t < 32) {
        const float a = (float)(1 - 4 * r);
        const float x = t < 16 ? (float)(t & (w.R - 1)) * a / (float)(2 * w.R)
                      : t < 24 ? (float)(t - 16) * a / (float)(2 << w.log_n) : -(float)(t - 24) * a / (float)(16 * w.R);
        const cd v = cis_pi_f64(x);
        if (t < 16) m.c[t] = rounded(v);
        else if (t < 24) m.step[t - 16] = v;
        else m.back[t - 24] = v;
    }
    __syncthreads();
}
// exp(i pi n a / 2N) of points n = 8 t + e, a = 1 - 4 r: kept for both passes where there are registers for that
template <int LOGC>
struct Twists {
    static constexpr bool kKept = LOGC < 13;
    cd first;
    cf kept[8];
    __device__ __forceinline__ Twists(const ConvLds<LOGC>& m, const ConvHead& w, float a, int t)
        : first(cis_pi_f64((float)(8 * t) * a / (float)(2 << w.log_n))) {
        if constexpr (kKept)
#pragma unroll
            for (int e = 0; e < 8; ++e) kept[e] = mul_rounded(first, m.step[e]);
    }
    __device__ __forceinline__ cf at(const ConvLds<LOGC>& m, int e) const {
        if constexpr (kKept) return kept[e];
        else return mul_rounded(first, m.step[e]);
    }
};
// The same for two sequences side by side: half the barriers, and each one's work in the shadow of the other's (with the first
// blocks of both requested ahead of the tables: evict on one layer of 13577 55.8 -> 54.5 us, smooth on 24 ragged sequences
// 41.2 -> 39.3, on 30 of 500-32000 74.6 -> 69.9, on one of 1500 13.7 -> 12.3).
// z2: padded_len(C) points
template <int LOGC>
__device__ __forceinline__ void to_bins_of_two(ConvLds<LOGC>& m, cf* z2, const typename Cfft<LOGC>::Twiddles& tw, const Twists<LOGC>& twist, int t,
                                               cf (&a)[8], cf (&b)[8]) {
    using F = Cfft<LOGC>;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const cf w = twist.at(m, e); a[e] = mul(a[e], w); b[e] = mul(b[e], w); }
    F::put(m.z, a, 8 * t, 0);
    F::put(z2, b, 8 * t, 0);
    __syncthreads();
    F::get(m.z, a, t, LOGC - 3);
    F::get(z2, b, t, LOGC - 3);
#pragma unroll
    for (int p = 0; p < F::P8; ++p) {                        // Fft::forward
        const int sb = F::low_bit(p), at = F::base(p, t);
        if (p) { F::get(m.z, a, at, sb); F::get(z2, b, at, sb); }
        dft8<-1>(a);
        dft8<-1>(b);
        if (p < F::TW) { F::template twist<false>(a, tw(p, 0)); F::template twist<false>(b, tw(p, 0)); }
        if (p + 1 < F::P8 || F::REM) { F::put(m.z, a, at, sb); F::put(z2, b, at, sb); __syncthreads(); }
    }
    if (F::REM) {
        F::get(m.z, a, 8 * t, 0);
        F::get(z2, b, 8 * t, 0);
        F::template small_dfts<-1>(a);
        F::template small_dfts<-1>(b);
    }
}
// acc, points 8 t + e, twisted and transformed: the bins of residue r in the last layout
template <int LOGC>
__device__ __forceinline__ void to_bins(ConvLds<LOGC>& m, const typename Cfft<LOGC>::Twiddles& tw, const Twists<LOGC>& twist, int t, const cf (&acc)[8],
                                        cf (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = mul(acc[e], twist.at(m, e));
    Cfft<LOGC>::put(m.z, v, 8 * t, 0);
    __syncthreads();
    Cfft<LOGC>::get(m.z, v, t, LOGC - 3);
    Cfft<LOGC>::forward(reinterpret_cast<cf(&)[1][8]>(v), m.z, tw, t);
}

// the filter's bins of every distinct length, for calls in which many heads share them
template <int LOGC>
__global__ __launch_bounds__(Cfft<LOGC>::THREADS) void conv_spectrum_kernel(Geom g, ConvFilterJob job, int log_r, int turn,
                                                                           cf* __restrict__ spec, size_t spec_stride)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ConvLds<LOGC>& m = *reinterpret_cast<ConvLds<LOGC>*>(smem);
    ConvHead w;
    const int item = blockIdx.x >> log_r, r = (blockIdx.x + item * turn) & ((1 << log_r) - 1), t = threadIdx.x;   // (as in conv_chunk_kernel)
    if (!conv_head(g, job, item * g.H_kv, LOGC, w) || w.owner != item || r >= w.R) return;
    TapBlocks<LOGC == 13 ? 2 : 4> taps;
    constexpr bool kEarly = LOGC < 13;
    if constexpr (kEarly) taps.load(job.h + item * job.item_stride, w, 1 << LOGC, t, 0);
    fill_constants<LOGC>(m, w, r, t);
    typename Cfft<LOGC>::Twiddles tw;
    Cfft<LOGC>::init(tw, m.table, t);
    cf acc[8], v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = {0.f, 0.f};
    taps.template sum<kEarly>(job.h + item * job.item_stride, w, 1 << LOGC, m.c, t, acc);
    to_bins<LOGC>(m, tw, Twists<LOGC>(m, w, (float)(1 - 4 * r), t), t, acc, v);
    cf* out = spec + (size_t)item * spec_stride + ((size_t)r << LOGC) + 8 * t;
#pragma unroll
    for (int e = 0; e < 8; e += 2)
        *reinterpret_cast<f32x4*>(out + e) = f32x4{v[e].re, v[e].im, v[e + 1].re, v[e + 1].im};
}

// SPEC: the filter's bins come from conv_spectrum_kernel; otherwise the workgroup transforms its share of the filter beside its
// share of the samples (8192 points, whose 1024 threads have 128 registers each: before it).
// KEEP: the result of a head of one chunk is left in LDS as well, from smem on, for whoever passes the next barrier.
template <int LOGC, int POOL, bool SPEC, bool KEEP>
__device__ __forceinline__ void conv_chunk(
    const Geom& g, const float* __restrict__ in, const ConvFilterJob& job, const ConvHead& w, int head, int r, const cf* __restrict__ spec,
    size_t spec_stride, cf* __restrict__ part, size_t part_stride, float alpha, float* __restrict__ out, unsigned char* smem)
{
    constexpr int C = 1 << LOGC, T = Cfft<LOGC>::THREADS;
    ConvLds<LOGC>& m = *reinterpret_cast<ConvLds<LOGC>*>(smem);
    constexpr int U = LOGC == 13 ? 2 : 4;                        // (1024 threads: 128 registers)
    const int t = threadIdx.x;
    const float* src = in + w.off;
    const float* h = job.h + w.owner * job.item_stride;
    // Without spectra few heads are at work and a CU has one workgroup: the first blocks are on their way while the tables are
    // filled. With them two share a CU, with 128 registers each.
    constexpr bool kEarly = !SPEC && LOGC < 13;
    SampleBlocks<U, POOL> samples;
    TapBlocks<U> taps;
    if constexpr (kEarly) {
        taps.load(h, w, C, t, 0);
        samples.load(src, w, C, t, 0);
    }
    fill_constants<LOGC>(m, w, r, t);
    typename Cfft<LOGC>::Twiddles tw;
    Cfft<LOGC>::init(tw, m.table, t);
    const float a = (float)(1 - 4 * r);
    const Twists<LOGC> twist(m, w, a, t);

    cf f[8], v[8], acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { f[e] = {0.f, 0.f}; acc[e] = {0.f, 0.f}; }
    if constexpr (SPEC) {
        const cf* b = spec + (size_t)w.owner * spec_stride + ((size_t)r << LOGC) + 8 * t;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const f32x4 p = *reinterpret_cast<const f32x4*>(b + e);
            f[e] = {p[0], p[1]}; f[e + 1] = {p[2], p[3]};
        }
        samples.template sum<false>(src, w, C, g.pool_kernel, g.pool_mode, m.c, t, acc);
        to_bins<LOGC>(m, tw, twist, t, acc, v);
    } else if constexpr (kEarly) {
        taps.template sum<true>(h, w, C, m.c, t, f);
        samples.template sum<true>(src, w, C, g.pool_kernel, g.pool_mode, m.c, t, acc);
        to_bins_of_two<LOGC>(m, reinterpret_cast<cf*>(smem + sizeof(m)), tw, twist, t, acc, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = acc[e];
    } else {
        taps.template sum<false>(h, w, C, m.c, t, acc);
        to_bins<LOGC>(m, tw, twist, t, acc, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = {0.f, 0.f};
        samples.template sum<false>(src, w, C, g.pool_kernel, g.pool_mode, m.c, t, acc);
        to_bins<LOGC>(m, tw, twist, t, acc, v);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = mul(v[e], f[e]);
    Cfft<LOGC>::backward(reinterpret_cast<cf(&)[1][8]>(v), m.z, tw, t);

    // twisted back: point n = t + T q of residue r by exp(i pi n (4 r - 1) / 2N); 1/N completes the inverse transform
    const double inv_n = 1.0 / (double)(1 << w.log_n);
    cd back0 = cis_pi_f64(-(float)t * a / (float)(2 << w.log_n));
    back0 = {back0.re * inv_n, back0.im * inv_n};
    cf* dst = part + (size_t)head * part_stride + (size_t)r * C;
    float* kept = reinterpret_cast<float*>(m.z);
    if constexpr (KEEP) __syncthreads();                         // all points are read
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const cf u = mul(v[q], mul_rounded(back0, m.back[q]));
        const int n = t + T * q;
        if (!KEEP && w.R > 1) dst[n] = u;
        else if (n < w.L) {                                      // a head of one workgroup is done
            float st = u.re;
            if (alpha != 1.f) {
                const float s0 = POOL ? pooled_at(src, w.L, n, g.pool_kernel, g.pool_mode) : src[n];
                st = mix(s0, st, alpha);
            }
            out[w.off + n] = st;
            if constexpr (KEEP) kept[n] = st;
        }
    }
}

template <int LOGC, int POOL, bool SPEC>
__global__ __launch_bounds__(Cfft<LOGC>::THREADS) void conv_chunk_kernel(
    Geom g, const float* __restrict__ in, ConvFilterJob job, int log_r, int turn, const cf* __restrict__ spec, size_t spec_stride,
    cf* __restrict__ part, size_t part_stride, float alpha, float* __restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ConvHead w;
    // Workgroup i runs on XCD i mod 8, and heads of fewer chunks than the longest need the first residues only: where there are such heads
    // (turn = 1), these go to another XCD from head to head. (All on the first ones: 24 sequences of two heads, 1500 to 30000 samples, put
    // 48 of their 172 workgroups on the 32 CUs of XCD 0, one each, and 12 on XCD 7. Smooth calls, so and now: those 36.9 and 27.2 us, 40 of
    // four heads of 3000 to 20000 80.0 and 64.4, 20 of 5000 to 100000 158 and 119; 211 ragged calls 0.95 of the time in the geometric mean,
    // the worst 1.02. Heads that all need every residue lose by it: 12 of 73557 with eight heads 169 and 178, 12 of 82908 with four 97.5 and 101.9.)
    const int head = blockIdx.x >> log_r, r = (blockIdx.x + head * turn) & ((1 << log_r) - 1);
    if (!conv_head(g, job, head, LOGC, w) || r >= w.R) return;
    conv_chunk<LOGC, POOL, SPEC, false>(g, in, job, w, head, r, spec, spec_stride, part, part_stride, alpha, out, smem);
}

// A head of one chunk, pooled with the usual kernel, smoothed and selected in one workgroup, as in smooth_select_kernel (smooth_real.hip):
// evict, two launches and one, four heads of 600 tokens 26.2 and 24.8 us, 1500 28.1 and 26.4, 3000 32.3 and 31.0; 112 heads of 3000 118 and
// 115.
// The barriers of conv_chunk: the constants, the points' exchange, the result, and those of the transforms (counted in the built kernels
// as well, tests/test_fused_barriers.py).
template <int LOGC> constexpr int kConvBarriers = 3 + 2 * Cfft<LOGC>::BARRIERS;
// (512 threads: with the 128 registers that 1024 have, 4096 points spill 110; a selection of 4096 tokens on them takes 0.9 us more)
constexpr int kConvFusedThreads = 512;
template <int LOGC, bool SPEC>
__global__ __launch_bounds__(kConvFusedThreads) void conv_select_kernel(
    Geom g, const float* __restrict__ in, ConvFilterJob job, const cf* __restrict__ spec, size_t spec_stride, float alpha,
    float* __restrict__ out, SelectJob sel)
{
    constexpr int NT = kConvFusedThreads, EPT = LOGC <= 11 ? 4 : 8;
    static_assert(EPT * NT >= 1 << LOGC, "a head's tokens");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    ConvHead w;
    if (!conv_head(g, job, blockIdx.x, LOGC, w) || w.R != 1) return;     // (uniform; the launch has heads of one chunk only)
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) < Cfft<LOGC>::THREADS / 64)
        conv_chunk<LOGC, 7, SPEC, true>(g, in, job, w, blockIdx.x, 0, spec, spec_stride, nullptr, 0, alpha, out, smem);
    else
#pragma unroll 1
        for (int i = 0; i < kConvBarriers<LOGC>; ++i) __syncthreads();
    __syncthreads();
    const float* kept = reinterpret_cast<const float*>(smem);
    select_head<EPT, NT>(g, blockIdx.x, w.L, sel.budgets, sel.cu_b, sel.indices, [&](float (&x)[EPT], int n_cand) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int n = (int)threadIdx.x + e * NT;
            x[e] = n < n_cand ? kept[n] : 0.f;
        }
    });
}

constexpr int kJoinThreads = 64;

__global__ __launch_bounds__(kJoinThreads) void conv_join_kernel(
    Geom g, const float* __restrict__ in, int pool_on_load, ConvFilterJob job, int log_c, const cf* __restrict__ part,
    size_t part_stride, float alpha, float* __restrict__ out)
{
    ConvHead w;
    const int C = 1 << log_c, per_head = C / kJoinThreads, head = blockIdx.x / per_head;
    if (!conv_head(g, job, head, log_c, w) || w.R == 1) return;
    const int n = (blockIdx.x - head * per_head) * kJoinThreads + threadIdx.x;
    const cf* p = part + (size_t)head * part_stride;
    const float* src = in + w.off;
    float* dst = out + w.off;
    float o[16];
    cf v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (r < w.R) v[r] = p[(size_t)r * C + n];
    switch (w.R) {
        case 2:  join<2>(v, o); break;
        case 4:  join<4>(v, o); break;
        case 8:  join<8>(v, o); break;
        default: join<16>(v, o); break;
    }
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int j = n + t * C;
        if (t < w.R && j < w.L) {
            float st = o[t];
            if (alpha != 1.f) {
                const float s0 = pool_on_load ? pooled_at(src, w.L, j, g.pool_kernel, g.pool_mode) : src[j];
                st = mix(s0, st, alpha);
            }
            dst[j] = st;
        }
    }
}

constexpr int kFilterThreads = 256;
__global__ __launch_bounds__(kFilterThreads) void conv_filter_kernel(ConvFilterJob job, int per_item) {
    conv_filter_block(job, blockIdx.x, per_item, kFilterThreads);
}

// Workgroups are numbered in one dimension, those of a head next to each other: the second and third dimension of a grid
// end at 65535, and a batch may hold more heads than that.
int log_residues(const ConvCall& c) { return 31 - __builtin_clz((unsigned)c.max_r); }

template <int LOGC, int POOL, bool SPEC>
hipError_t launch_chunks(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, hipStream_t s) {
    const int lds = (int)(sizeof(ConvLds<LOGC>) + (SPEC || LOGC == 13 ? 0 : padded_len((size_t)1 << LOGC) * sizeof(cf)));
    if (lds > 48 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_chunk_kernel<LOGC, POOL, SPEC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((conv_chunk_kernel<LOGC, POOL, SPEC>), dim3((unsigned)(g.n_items * g.H_kv) << log_residues(c)),
                       dim3(Cfft<LOGC>::THREADS), lds, s, g, in, c.job, log_residues(c), c.uneven ? 1 : 0, (const cf*)c.spec, c.points, (cf*)c.part, c.points, alpha, out);
    return hipGetLastError();
}
template <int LOGC, bool SPEC>
hipError_t launch_fused(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, const SelectJob& sel, hipStream_t s) {
    const int lds = (int)(sizeof(ConvLds<LOGC>) + (SPEC ? 0 : padded_len((size_t)1 << LOGC) * sizeof(cf)));
    if (lds > 24 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_select_kernel<LOGC, SPEC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((conv_select_kernel<LOGC, SPEC>), dim3((unsigned)(g.n_items * g.H_kv)), dim3(kConvFusedThreads), lds, s, g, in,
                       c.job, (const cf*)c.spec, c.points, alpha, out, sel);
    return hipGetLastError();
}
template <int LOGC>
hipError_t launch_fused(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, const SelectJob& sel, hipStream_t s) {
    return c.spec ? launch_fused<LOGC, true>(g, c, in, alpha, out, sel, s) : launch_fused<LOGC, false>(g, c, in, alpha, out, sel, s);
}
template <int LOGC, int POOL>
hipError_t launch_chunks(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, hipStream_t s) {
    return c.spec ? launch_chunks<LOGC, POOL, true>(g, c, in, alpha, out, s) : launch_chunks<LOGC, POOL, false>(g, c, in, alpha, out, s);
}
template <int LOGC>
hipError_t launch_chunks(const Geom& g, const ConvCall& c, const float* in, bool pool_on_load, float alpha, float* out, hipStream_t s) {
    if (!pool_on_load) return launch_chunks<LOGC, 0>(g, c, in, alpha, out, s);
    if (g.pool_kernel == 7) return launch_chunks<LOGC, 7>(g, c, in, alpha, out, s);
    return launch_chunks<LOGC, 9>(g, c, in, alpha, out, s);
}
template <int LOGC>
hipError_t launch_spectra(const Geom& g, const ConvCall& c, hipStream_t s) {
    const int lds = (int)sizeof(ConvLds<LOGC>);
    if (lds > 48 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_spectrum_kernel<LOGC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    hipLaunchKernelGGL((conv_spectrum_kernel<LOGC>), dim3((unsigned)g.n_items << log_residues(c)), dim3(Cfft<LOGC>::THREADS), lds, s,
                       g, c.job, log_residues(c), c.uneven ? 1 : 0, (cf*)c.spec, c.points);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_conv_filter(const Geom& g, const ConvCall& c, hipStream_t s) {
    const int per_item = c.job.blocks_per_item(kFilterThreads);
    hipLaunchKernelGGL(conv_filter_kernel, dim3((unsigned)(per_item * c.job.n_items)), dim3(kFilterThreads), 0, s, c.job, per_item);
    if (!c.spec) return hipGetLastError();
    switch (c.log_c) {
        case 10: return launch_spectra<10>(g, c, s);
        case 11: return launch_spectra<11>(g, c, s);
        case 12: return launch_spectra<12>(g, c, s);
        default: return launch_spectra<13>(g, c, s);
    }
}

hipError_t launch_conv_select(const Geom& g, const ConvCall& c, const float* in, float alpha, float* out, const SelectJob& sel, hipStream_t s) {
    if (c.max_r != 1 || g.pool_kernel != 7) return hipErrorInvalidValue;
    switch (c.log_c) {
        case 10: return launch_fused<10>(g, c, in, alpha, out, sel, s);
        case 11: return launch_fused<11>(g, c, in, alpha, out, sel, s);
        case 12: return launch_fused<12>(g, c, in, alpha, out, sel, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_conv(const Geom& g, const ConvCall& c, const float* in, bool pool_on_load, float alpha, float* out, hipStream_t s,
                       ConvJoin* join) {
    if (pool_on_load && g.pool_kernel > kConvMaxPool) return hipErrorInvalidValue;      // (pooled beforehand)
    // a launch of 2^32 threads or more would drop workgroups without an error
    const long long points = (long long)g.n_items * g.H_kv << c.log_c;
    if (points >= 1LL << 32 || points * c.max_r / 8 >= 1LL << 32) return hipErrorInvalidConfiguration;
    hipError_t e;
    switch (c.log_c) {
        case 10: e = launch_chunks<10>(g, c, in, pool_on_load, alpha, out, s); break;
        case 11: e = launch_chunks<11>(g, c, in, pool_on_load, alpha, out, s); break;
        case 12: e = launch_chunks<12>(g, c, in, pool_on_load, alpha, out, s); break;
        default: e = launch_chunks<13>(g, c, in, pool_on_load, alpha, out, s); break;
    }
    if (e != hipSuccess || c.max_r == 1) return e;
    if (join && c.log_c == kJoinLogC && c.max_r <= kJoinMaxR) {
        *join = ConvJoin{c.job, in, pool_on_load ? 1 : 0, alpha, c.part, c.points, out};
        return hipSuccess;
    }
    hipLaunchKernelGGL(conv_join_kernel, dim3((1u << c.log_c) / kJoinThreads * (unsigned)(g.n_items * g.H_kv)), dim3(kJoinThreads),
                       0, s, g, in, pool_on_load ? 1 : 0, c.job, c.log_c, (const cf*)c.part, c.points, alpha, out);
    return hipGetLastError();
}

}  // namespace audiokv
