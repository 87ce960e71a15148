// What combines the chunks of a convolved head: conv.hip's own launch, or the selection that reads the result.
#pragma once

#include "conv.h"
#include "fft_regs.h"

namespace audiokv {
namespace {

struct ConvHead { int L, log_n, R, owner; size_t off; };

__device__ __forceinline__ bool conv_head(const Geom& g, const ConvFilterJob& job, int head, int log_c, ConvHead& w) {
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tok0 = job.cu_seqlens[item];
    w.L = job.cu_seqlens[item + 1] - tok0;
    if (!conv_item(job, w.L)) return false;
    w.log_n = conv_log_points(w.L, log_c);
    w.R = 1 << (w.log_n - log_c);
    w.owner = conv_owner(job.cu_seqlens, item, w.L);
    w.off = (size_t)tok0 * g.H_kv + (size_t)h * w.L;
    return true;
}

// out[n + C t] = Re sum_r part_r[n] exp(i pi (4 r - 1) t / 2R), t = 0..R-1: an R-point inverse DFT and a rotation
// (v: part_r[n])
template <int R>
__device__ __forceinline__ void join(cf (&v)[16], float* o) {
    if constexpr (R == 2) { const cf a = v[0]; v[0] = cadd(a, v[1]); v[1] = csub(a, v[1]); }
    else if constexpr (R == 4) dft4<1>(v[0], v[1], v[2], v[3]);
    else if constexpr (R == 8) dft8<1>(reinterpret_cast<cf(&)[8]>(v));
    else {
        // sixteen points as two of eight: even and odd residues
        cf e[8], d[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) { e[k] = v[2 * k]; d[k] = v[2 * k + 1]; }
        dft8<1>(e);
        dft8<1>(d);
        constexpr float C1 = 0.92387953251128674f, S1 = 0.38268343236508977f, H = 0.70710678118654752f;
        constexpr cf root[8] = {{1.f, 0.f}, {C1, S1}, {H, H}, {S1, C1}, {0.f, 1.f}, {-S1, C1}, {-H, H}, {-C1, S1}};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const cf x = mul(d[k], root[k]);
            v[k] = cadd(e[k], x);
            v[k + 8] = csub(e[k], x);
        }
    }
    // exp(-i pi t / 2R)
    constexpr cf unit[16] = {{1.f, 0.f}, {0.99518472667219689f, 0.098017140329560602f}, {0.98078528040323045f, 0.19509032201612827f},
                             {0.95694033573220887f, 0.29028467725446237f}, {0.92387953251128676f, 0.38268343236508977f},
                             {0.88192126434835503f, 0.47139673682599764f}, {0.83146961230254524f, 0.55557023301960222f},
                             {0.77301045336273696f, 0.63439328416364549f}, {0.70710678118654752f, 0.70710678118654752f},
                             {0.63439328416364549f, 0.77301045336273696f}, {0.55557023301960222f, 0.83146961230254524f},
                             {0.47139673682599764f, 0.88192126434835503f}, {0.38268343236508977f, 0.92387953251128676f},
                             {0.29028467725446237f, 0.95694033573220887f}, {0.19509032201612827f, 0.98078528040323045f},
                             {0.098017140329560602f, 0.99518472667219689f}};      // cos, sin of pi t / 32
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const cf c = unit[t * (16 / R)];
        o[t] = fmaf(v[t].re, c.re, v[t].im * c.im);
    }
}

}  // namespace
}  // namespace audiokv
