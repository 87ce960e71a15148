// After the eviction path: one decoding step on the compacted cache (paper Sec. 1 / Sec. 4.6: decoding runs on
// the retained tokens only). Every query head attends to the b_h packed rows of its KV head.
//
// Pure streaming: each K and V row is read once, so the bound is HBM. A workgroup takes one chunk of consecutive
// rows of one KV head (rows of a head are contiguous in the packed cache) and all G query heads of its group:
//   1. logits  Q (G x d, padded to 8 or 16 rows, stationary) times the chunk's K rows on the matrix cores
//              (16 keys per MFMA group, 16-byte loads straight from HBM into the B operand), into LDS; each wave
//              keeps the maxima of the logits that it writes;
//   2. weights exp2(logit - chunk maximum), a thread on four query heads of a row, and their sums;
//   3. weights times V on the vector ALUs: a thread owns 8 channels of every (256 / (d/8))-th row, so a wave's
//      load covers whole consecutive rows; fp32 accumulators, reduced over the threads of a channel at the end.
// What a workgroup costs is latency: the first V rows are requested before K, K loads of 128 rows are all in flight
// before the first MFMA (left alone the compiler keeps three), two barriers separate the phases.
// Chunks of a head are combined by a second small kernel (max / sum rescaling in base 2). No atomics.
//
// Budgets differ from head to head and are known on the device only. Chunk c of head g has slot
//     floor(cu_b[g] / R) + g + c        (R rows per chunk)
// and a workgroup finds its head by a binary search for its slot: the slots of a head start one past the last that
// the head before can use (ceil(n / R) <= floor((b + n) / R) - floor(b / R) + 1), so they never meet, and at most one
// slot per head stays empty. No table of chunks has to be written first.
#include "common.h"

namespace audiokv {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
// Rows per workgroup at most: what the weights' LDS buffer (4 bytes per row and padded query head, 32 KiB) holds, four
// workgroups per CU. At least one trip of phase 1 (128 rows).
__host__ __device__ constexpr int max_chunk_rows(int GP) { return GP <= 8 ? 1024 : 512; }
constexpr int kMinLogChunk = 7, kMinChunkRows = 1 << kMinLogChunk;

__device__ __forceinline__ float bf16_lo(unsigned int w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned int w) { return __uint_as_float(w & 0xffff0000u); }

// start of head g's rows, cut so that nothing past total_rows is ever read
__device__ __forceinline__ int head_start(const int32_t* __restrict__ cu_b, int g, int total_rows) {
    return min(cu_b[g], total_rows);
}
__device__ __forceinline__ int first_slot(const int32_t* __restrict__ cu_b, int g, int total_rows, int log_r) {
    return (head_start(cu_b, g, total_rows) >> log_r) + g;
}

// a, b <- sums over lanes 32 apart of a (lower half of the wave) and of b (upper half), in a. (asm: see score_impl.h
// on v_permlane32_swap; the wait states cover the vector writes that produce the operands)
__device__ __forceinline__ float fold32(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
#endif
    return a + b;
}
// the same over lanes 16 apart: even rows of 16 lanes get the sum of a, odd rows that of b
__device__ __forceinline__ float fold16(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
#endif
    return a + b;
}

template <int D, int GP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(GP > 8 ? 2 : D == 256 ? 3 : 4, GP > 8 ? 2 : D == 256 ? 3 : 4)))   // no spills
void decode_partial_kernel(
    Geom g, const __bf16* __restrict__ q, const __bf16* __restrict__ kc, const __bf16* __restrict__ vc,
    const int32_t* __restrict__ cu_b, int n_heads, int total_rows, int log_r,
    float* __restrict__ part,            // [slot][G][D] accumulators
    float* __restrict__ stats)           // [slot][G][2] = (max in base-2 units, sum)
{
    constexpr int VPR = D / 8;                 // 16-byte pieces (lanes) per row
    constexpr int KQ = kThreads / VPR;         // rows in flight per pass of phase 3
    constexpr int KK = D / 32;                 // MFMA k-steps
    constexpr int UN = D == 64 ? 4 : 8;        // V rows in flight per thread
    constexpr int TRIP = 128;                  // rows of one trip of phase 1; phases 2 and 3 go in whole trips, too
    static_assert(TRIP % (KQ * UN) == 0 && kMinChunkRows % TRIP == 0, "a chunk is whole trips of every phase");
    // logits, then weights: [row][query head]; at the end the four waves' accumulators: [wave][query head][channel]
    extern __shared__ __attribute__((aligned(16))) float lg[];
    __shared__ float st_m[4][GP], st_l[4][GP];

    // The last head whose first slot is not past this one. Every round probes 64 heads at equal distances, one per
    // lane: one load latency for up to 64 heads, two up to 4096 (a binary search pays one per doubling).
    const int cid = blockIdx.x;
    int head = 0;
    for (int span = n_heads; span > 1;) {
        const int step = (span + 63) >> 6;
        const int probe = head + (int)(threadIdx.x & 63) * step;
        const bool at_or_before = probe < head + span && first_slot(cu_b, min(probe, n_heads - 1), total_rows, log_r) <= cid;
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(at_or_before));   // a prefix of the lanes
        const int skip = n > 0 ? (n - 1) * step : 0;
        head += skip;
        span = min(step, span - skip);
    }
    head = __builtin_amdgcn_readfirstlane(head);
    const int chunk = cid - first_slot(cu_b, head, total_rows, log_r);
    const int64_t row_b = head_start(cu_b, head, total_rows) + ((int64_t)chunk << log_r);
    const int rows = (int)min((int64_t)1 << log_r, head_start(cu_b, head + 1, total_rows) - row_b);
    if (chunk < 0 || rows <= 0) return;        // uniform: the slot that this head leaves empty
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int G = g.G;
    const __bf16* krow0 = kc + (size_t)row_b * D;
    const __bf16* vrow0 = vc + (size_t)row_b * D;
    const int trips = (rows + TRIP - 1) / TRIP;

    // the first V rows of phase 3 (all of a 128-row chunk at d <= 128) are requested first: one latency for K and V
    const int c8 = tid % VPR, kq = tid / VPR;
    u32x4 vv[UN];
    // Rows past the end carry weight 0, but 0 times an infinity is NaN: they have to read as zeros. A buffer whose size is
    // that of the chunk's rows does that in hardware.
    const auto vbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(vrow0), 0, rows * D * 2, 0x00027000);
    auto load_v = [&](int r0) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
            vv[u] = __builtin_amdgcn_raw_buffer_load_b128(vbuf, ((r0 + kq + u * KQ) * VPR + c8) * 16, 0, 2 /* nontemporal */);
    };
    load_v(0);

    // ---- phase 1: logits in base-2 units ----
    {
        const int qr = lane & 15, kgrp = lane >> 4;             // A operand: query row qr, channels 8*kgrp + 32*kk
        bf16x8 qa[KK];
        const __bf16* qsrc = q + ((size_t)item * g.H_q + (size_t)h * G + min(qr, G - 1)) * D + kgrp * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qa[kk] = *reinterpret_cast<const bf16x8*>(qsrc + kk * 32);   // rows >= G: unused copies
        f32x4 top = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        for (int t = 0; t < trips; ++t) {
            // B operand: key = lane & 15 of two groups of 16 keys (rows past the end are clamped, masked below)
            const int keya = t * TRIP + wave * 16 + qr, keyb = keya + TRIP / 2;
            const __bf16* pa = krow0 + (size_t)min(keya, rows - 1) * D + kgrp * 8;
            const __bf16* pb = krow0 + (size_t)min(keyb, rows - 1) * D + kgrp * 8;
            bf16x8 fa[KK], fb[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                fa[kk] = *reinterpret_cast<const bf16x8*>(pa + kk * 32);
                fb[kk] = *reinterpret_cast<const bf16x8*>(pb + kk * 32);
            }
            __builtin_amdgcn_sched_barrier(0);                  // all loads of the trip before its first MFMA
            f32x4 ca = {0.f, 0.f, 0.f, 0.f}, cb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                ca = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kk], fa[kk], ca, 0, 0, 0);
                cb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kk], fb[kk], cb, 0, 0, 0);
            }
            // result: lane holds key (lane & 15), query rows 4 * (lane >> 4) + i
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ca[i] = keya < rows ? ca[i] * g.c_log2 : -INFINITY;
                cb[i] = keyb < rows ? cb[i] * g.c_log2 : -INFINITY;
                top[i] = fmaxf(top[i], fmaxf(ca[i], cb[i]));
            }
            if (kgrp * 4 < GP) {
                *reinterpret_cast<f32x4*>(&lg[keya * GP + kgrp * 4]) = ca;
                *reinterpret_cast<f32x4*>(&lg[keyb * GP + kgrp * 4]) = cb;
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) top[i] = fmaxf(top[i], __shfl_xor(top[i], o, 64));
        if (qr == 0 && kgrp * 4 < GP)
#pragma unroll
            for (int i = 0; i < 4; ++i) st_m[wave][kgrp * 4 + i] = top[i];
    }
    __syncthreads();

    // ---- phase 2: logits become weights; sums over the chunk ----
    {
        constexpr int QPR = GP / 4;                             // threads per row
        const int qd = tid % QPR, r0 = tid / QPR;
        f32x4 m, l = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            m[i] = fmaxf(fmaxf(st_m[0][qd * 4 + i], st_m[1][qd * 4 + i]), fmaxf(st_m[2][qd * 4 + i], st_m[3][qd * 4 + i]));
        for (int r = r0; r < trips * TRIP; r += kThreads / QPR) {
            f32x4 p = *reinterpret_cast<const f32x4*>(&lg[r * GP + qd * 4]);
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(p[i] - m[i]);
            l += p;
            *reinterpret_cast<f32x4*>(&lg[r * GP + qd * 4]) = p;
        }
#pragma unroll
        for (int o = 32; o >= QPR; o >>= 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) l[i] += __shfl_xor(l[i], o, 64);
        if (lane < QPR)
#pragma unroll
            for (int i = 0; i < 4; ++i) st_l[wave][lane * 4 + i] = l[i];
    }
    __syncthreads();

    // ---- phase 3: weights times V ----
    float acc[GP * 8];                                          // [query head][channel c8 * 8 + i]
#pragma unroll
    for (int e = 0; e < GP * 8; ++e) acc[e] = 0.f;
    for (int r = 0; r < trips * TRIP; r += KQ * UN) {
        if (r) load_v(r);                                       // (the first batch is already on its way)
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            float p[GP];
#pragma unroll
            for (int q4 = 0; q4 < GP / 4; ++q4) {
                const f32x4 t = *reinterpret_cast<const f32x4*>(&lg[(r + kq + u * KQ) * GP + q4 * 4]);
                p[q4 * 4 + 0] = t[0]; p[q4 * 4 + 1] = t[1]; p[q4 * 4 + 2] = t[2]; p[q4 * 4 + 3] = t[3];
            }
            float v[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[2 * i] = bf16_lo(vv[u][i]); v[2 * i + 1] = bf16_hi(vv[u][i]); }
#pragma unroll
            for (int qh = 0; qh < GP; ++qh)
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[qh * 8 + i] = fmaf(p[qh], v[i], acc[qh * 8 + i]);
        }
    }
    // Threads of one wave that share c8, halving the values with the lanes: after a fold over lanes 32 apart the upper
    // half of the wave holds the upper half of the query heads, after one over lanes 16 apart odd rows of 16 lanes
    // the upper half of those.
    constexpr int N32 = GP * 4, N16 = VPR <= 16 ? N32 / 2 : N32;
#pragma unroll
    for (int e = 0; e < N32; ++e) acc[e] = fold32(acc[e], acc[e + N32]);
    int qh0 = (lane >> 5) * (GP / 2);
    if constexpr (VPR <= 16) {
#pragma unroll
        for (int e = 0; e < N16; ++e) acc[e] = fold16(acc[e], acc[e + N16]);
        qh0 += ((lane >> 4) & 1) * (GP / 4);
    }
    if constexpr (VPR == 8) {
#pragma unroll
        for (int e = 0; e < N16; ++e) acc[e] += __shfl_xor(acc[e], 8, 64);
    }
    __syncthreads();                                            // every wave is done with the weights
#pragma unroll
    for (int e = 0; e < N16; e += 4)
        *reinterpret_cast<f32x4*>(&lg[(wave * GP + qh0 + e / 8) * D + c8 * 8 + e % 8]) =
            f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
    __syncthreads();
    float* out = part + (size_t)cid * G * D;
    for (int e = tid; e < G * D; e += kThreads)
        out[e] = ((lg[e] + lg[GP * D + e]) + lg[2 * GP * D + e]) + lg[3 * GP * D + e];
    if (tid < G) {
        stats[((size_t)cid * G + tid) * 2] = fmaxf(fmaxf(st_m[0][tid], st_m[1][tid]), fmaxf(st_m[2][tid], st_m[3][tid]));
        stats[((size_t)cid * G + tid) * 2 + 1] = ((st_l[0][tid] + st_l[1][tid]) + st_l[2][tid]) + st_l[3][tid];
    }
}

// One workgroup per (KV head, query head of its group): combine the chunks. A chain of loads from end to end, so as
// many as possible are in flight: the statistics one chunk per thread, then the accumulators with a thread on four
// channels of every (THREADS / (D/4))-th chunk. Every sum has a fixed order.
// THREADS: 1024 where heads have many chunks (launch_decode).
constexpr int kMergeEarly = 4;            // accumulators per thread requested before the statistics are known
constexpr int kMergeLds = 2048;           // chunks whose weights fit the LDS array (more: recomputed where used)

template <int THREADS>
__global__ __launch_bounds__(THREADS) void decode_merge_kernel(
    Geom g, const int32_t* __restrict__ cu_b, int total_rows, int log_r, const float* __restrict__ part,
    const float* __restrict__ stats, float* __restrict__ out)
{
    const int head = blockIdx.x / g.G, qh = blockIdx.x - head * g.G;
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b0 = head_start(cu_b, head, total_rows), n = head_start(cu_b, head + 1, total_rows) - b0;
    const int c0 = (b0 >> log_r) + head, nc = n > 0 ? (n + (1 << log_r) - 1) >> log_r : 0;
    float* o = out + ((size_t)item * g.H_q + (size_t)h * g.G + qh) * g.D;
    __shared__ float wgt[kMergeLds];
    __shared__ float wave_m[THREADS / 64], wave_l[THREADS / 64];
    __shared__ __attribute__((aligned(16))) f32x4 red[THREADS];

    // The first accumulators are requested together with the statistics: one load latency less (112 heads of 13 chunks 6.3 ->
    // 5.7 us, 64 heads 4.6 -> 4.0).
    const int quads = g.D >> 2, groups = THREADS / quads;  // 256 threads, D = 64, 128, 256: 16, 8, 4 chunks at a time; 1024: 32 and 16
    const int ch4 = tid % quads, grp = tid / quads;
    const f32x4* col = reinterpret_cast<const f32x4*>(part + ((size_t)c0 * g.G + qh) * g.D) + ch4;
    const size_t stride = (size_t)g.G * quads;
    f32x4 early[kMergeEarly];
    if (nc > 0) {
#pragma unroll
        for (int u = 0; u < kMergeEarly; ++u) early[u] = col[(size_t)min(grp + u * groups, nc - 1) * stride];
    }

    const float2* st = reinterpret_cast<const float2*>(stats) + (size_t)c0 * g.G + qh;     // chunk c at st[c * G]
    float m = -INFINITY, l = 0.f;
    for (int c = tid; c < nc; c += THREADS) {
        const float2 s = st[(size_t)c * g.G];
        if (c < kMergeLds) wgt[c] = s.x;
        const float m2 = fmaxf(m, s.x);                          // a chunk holds at least one row: s.x is finite
        l = l * __builtin_amdgcn_exp2f(m - m2) + s.y * __builtin_amdgcn_exp2f(s.x - m2);
        m = m2;
    }
    float M = m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    if (lane == 0) wave_m[wave] = M;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) M = fmaxf(M, wave_m[w]);
    l = m == -INFINITY ? 0.f : l * __builtin_amdgcn_exp2f(m - M);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) wave_l[wave] = l;
    for (int c = tid; c < min(nc, kMergeLds); c += THREADS) wgt[c] = __builtin_amdgcn_exp2f(wgt[c] - M);
    __syncthreads();
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) den += wave_l[w];

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < kMergeEarly; ++u)
        if (grp + u * groups < nc) acc += early[u] * wgt[grp + u * groups];
#pragma unroll 4
    for (int c = grp + kMergeEarly * groups; c < nc; c += groups) {
        const float w = c < kMergeLds ? wgt[c] : __builtin_amdgcn_exp2f(st[(size_t)c * g.G].x - M);
        acc += col[(size_t)c * stride] * w;
    }
    red[tid] = acc;
    __syncthreads();
    if (grp == 0) {
        f32x4 num = acc;
        for (int k = 1; k < groups; ++k) num += red[k * quads + ch4];
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        num = nc > 0 ? num / den : zero;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[ch4 * 4 + i] = num[i];     // `out` need not be aligned beyond its floats
    }
}

}  // namespace

bool decode_supported(int G) { return G >= 1 && G <= 16; }

// Rows per chunk (a power of two): the largest that still gives every CU four workgroups (what its registers hold at
// d <= 128), within what the kernel can hold. Both kernels of a call, d = 128, fixed 1024-row chunks -> this rule:
// 3.3 k rows 36 -> 14 us, 105 k rows 42 -> 20, 367 k rows 59 -> 43 (4.4 TB/s), 1.47 M rows 157 -> 142 (5.3 TB/s);
// with one workgroup per CU instead of four 367 k rows take 47 us and 734 k rows 86 instead of 78.
constexpr int kChunksPerCu = 4;
static int log_chunk_rows(const Geom& g, long long total_rows) {
    int lg = kMinLogChunk;
    while ((2 << lg) <= max_chunk_rows(g.G) && (total_rows >> (lg + 1)) >= 256 * kChunksPerCu) ++lg;
    return lg;
}
// slots of chunks: every head leaves at most one empty
static size_t slot_bound(const Geom& g, long long total_rows) {
    return (size_t)(total_rows >> log_chunk_rows(g, total_rows)) + (size_t)g.n_items * g.H_kv;
}
static size_t stats_bytes(const Geom& g, size_t bound) { return (bound * g.G * 2 * sizeof(float) + 255) & ~(size_t)255; }

// A workspace sized for one cache serves every smaller one. Where the chunks double, the number of slots halves: every call
// beyond the first such line is charged the most that calls below a line need.
size_t decode_workspace_bytes(const Geom& g, long long total_rows) {
    size_t bound = slot_bound(g, total_rows);
    const size_t peak = 2 * 256 * kChunksPerCu - 1 + (size_t)g.n_items * g.H_kv;
    if (log_chunk_rows(g, total_rows) > kMinLogChunk && bound < peak) bound = peak;
    return stats_bytes(g, bound) + bound * g.G * g.D * sizeof(float);
}

hipError_t launch_decode(const Geom& g, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* cu_budgets, long long total_rows, float* out, void* workspace, hipStream_t s)
{
    const int n_heads = g.n_items * g.H_kv;
    const size_t bound = slot_bound(g, total_rows);
    if (total_rows < 0 || bound > (size_t)INT32_MAX || !decode_supported(g.G)) return hipErrorInvalidValue;
    const int log_r = log_chunk_rows(g, total_rows);
    float* stats = static_cast<float*>(workspace);
    float* part = reinterpret_cast<float*>(static_cast<char*>(workspace) + stats_bytes(g, bound));
    const dim3 grid((unsigned)bound);
    const bool wide = g.G > 8;
    const unsigned gp = wide ? 16 : 8;
    const unsigned lds = (unsigned)sizeof(float) * gp * (4u * g.D > (1u << log_r) ? 4u * g.D : (1u << log_r));
#define AUDIOKV_LAUNCH_DECODE(DD, GG)                                                                           \
    hipLaunchKernelGGL((decode_partial_kernel<DD, GG>), grid, dim3(kThreads), lds, s, g, (const __bf16*)q,     \
                       (const __bf16*)k_cache, (const __bf16*)v_cache, cu_budgets, n_heads, (int)total_rows,   \
                       log_r, part, stats)
    switch (g.D) {
        case 64:  if (wide) AUDIOKV_LAUNCH_DECODE(64, 16);  else AUDIOKV_LAUNCH_DECODE(64, 8);  break;
        case 128: if (wide) AUDIOKV_LAUNCH_DECODE(128, 16); else AUDIOKV_LAUNCH_DECODE(128, 8); break;
        case 256: if (wide) AUDIOKV_LAUNCH_DECODE(256, 16); else AUDIOKV_LAUNCH_DECODE(256, 8); break;
        default: return hipErrorInvalidValue;
    }
#undef AUDIOKV_LAUNCH_DECODE
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // 256 threads combine 1024 / D chunks of a head at a time. Where the average head has three such rounds or more, the chain of their
    // loads is the launch: 1024 threads. Calls, d = 256 8 of 2048 to 32768 (5 rounds) 26.8 -> 24.0 us, 28 x 8192 (6) 40.7 -> 39.3; d = 128
    // 1 x 8192 (3) 12.0 -> 11.7, 1 x 32768 (13) 17.1 -> 15.6; with fewer rounds than that 16 x 4096 (1.6) 19.5 and 20.7, 28 x 8192 (1.6)
    // 39.4 and 43.1;
    // d = 64, where a round is sixteen chunks, 1 x 20000 (4) 10.3 and 10.7. More workgroups than two of them per CU hide the chain for one
    // another, and 256 threads leave room for more (49 caches of 16 query heads, 3.6 rounds, 37.9 and 40.8 us, 41 of two heads of eight,
    // d = 256, 3.4 rounds 59.9 and 60.7; with 384 to 512 workgroups 1 % the other way).
    const dim3 merge((unsigned)(n_heads * g.G));
    if (g.D >= 128 && n_heads * g.G <= 512 && (total_rows >> log_r) >= 3LL * (1024 / g.D) * n_heads)
        hipLaunchKernelGGL(decode_merge_kernel<1024>, merge, dim3(1024), 0, s, g, cu_budgets, (int)total_rows, log_r, (const float*)part,
                           (const float*)stats, out);
    else
        hipLaunchKernelGGL(decode_merge_kernel<256>, merge, dim3(256), 0, s, g, cu_budgets, (int)total_rows, log_r, (const float*)part,
                           (const float*)stats, out);
    return hipGetLastError();
}

}  // namespace audiokv
