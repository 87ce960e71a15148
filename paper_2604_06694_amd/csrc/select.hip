// Stage 4: per-head top-k with a forced window tail (paper Sec. 1, Solution 2:
// Top-K selection on the importance scores; window w of Sec. 3.1 Eq. 1).
//
// One workgroup per head, token t + NT e in register e of thread t (coalesced
// loads). A histogram counted in LDS finds the part of the scores' range that
// the threshold lies in: parts of equal width over two standard deviations to
// either side of the mean (to the largest or smallest score if the budget asks
// for a few of the tokens or for nearly all), which the threshold of a share in
// between rarely leaves and where no part holds many tokens, whatever the tails
// are like. The candidates in that part, 64 at most, are ranked against each
// other by every wave for itself, by score and, among equals, by index (ties
// are kept in index order). That gives the threshold as a score T and the
// number of tokens to keep that equal it: a token stays if its score is larger
// than T, or equal to T and the token among the first that many. For a fixed
// register the lanes of a wave hold 64 consecutive tokens, so one lane mask
// gives every (register, wave) chunk its count, a scan over the chunks their
// output offsets, and every kept token computes its own ascending output slot
// from the offset and its rank in the lane mask; equal ones are counted along.
//
// More than 64 candidates in the part, and scores that are not finite: the
// general search. Scores become order-preserving 32-bit keys, and the keys'
// range is divided into 2048 parts, and the part with the threshold again,
// until it holds few or one value only. Both ways compare and count only
// (the mean and the deviation choose where the parts lie, nothing else): the
// result is exact, and the same whichever way it was found.
//
// What bounds it is the chain of one head: the loads of up to 128 KB by one CU,
// five barriers, the adds of the histogram and the stores. Keys of float scores
// that cross zero, as smoothed ones do, leave the bulk of the tokens few parts
// of their range, and the general search alone took a second round for nearly
// every head. Smoothed scores, general search -> this: four heads of 2048 tokens
// 5.1 -> 4.4 us, 13577 12.5 -> 9.1, 32768 20.8 -> 15.5; 112 heads of 8192 10.4 ->
// 9.7, 32768 22.9 -> 18.7; 16 ragged heads 17.0 -> 13.2. Normal scores, which need
// one round either way: four heads of 32768 15.7 -> 13.5. Scores of a few dozen
// values crowd the threshold's part with one value: then that value is the
// threshold, and rounds over the indices of its tokens are not needed. Calls,
// general search with those rounds -> the division with them -> this: four heads
// of 32768 32.8 -> 35.2 -> 22.9 us, of 16385 23.9 -> 28.9 -> 19.4, 800 of 9000 56 ->
// 61 -> 44, 8000 of 500 39 -> 41 -> 39.
// Short heads in large numbers are bound by the instructions of a wave (sums
// over 8 or 16 lanes in three or four steps, reciprocals and roots as one
// instruction: 8000 heads of 500 32.8 -> 30.3 us, general search 31.8).
// Two, four or eight workgroups per head that each find the threshold and write
// a part gained nothing with four heads and lost with 112: every one of them
// has to load the whole head.
#include "common.h"
#include "conv_join.h"
#include "select_head.h"

namespace audiokv {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Block-wide sum; every thread gets the result. `slots` has 2 * kSelWaves ints, `parity` alternates per call.
__device__ __forceinline__ int block_count(int v, int* slots, int parity) {
    v = wave_sum(v);
    int* s = slots + parity * kSelWaves;
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) t += s[w];
    return t;
}

// Block-wide exclusive scan of two counters at once; returns this thread's offsets, totals through pointers.
__device__ __forceinline__ void block_exscan2(int a, int b, int* slots /* 2*kSelWaves */, int& ea, int& eb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int ia = a, ib = b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int ta = __shfl_up(ia, o, 64), tb = __shfl_up(ib, o, 64);
        if (lane >= o) { ia += ta; ib += tb; }
    }
    if (lane == 63) { slots[wave] = ia; slots[kSelWaves + wave] = ib; }
    __syncthreads();
    int pa = 0, pb = 0;
    for (int w = 0; w < wave; ++w) { pa += slots[w]; pb += slots[kSelWaves + w]; }
    ea = pa + ia - a;
    eb = pb + ib - b;
}

constexpr int kCompact = 8;          // undecided keys per thread once the streaming kernel has narrowed the candidates down
// Scores of tokens tid + NT e that a convolution left in chunks: token n + C t from points n of all chunks, and every thread's
// points are those of its own tokens. From n_cand on they are zero here. In place of a launch that combined them: evict on one layer
// of 5000 tokens 40.2 -> 38.8 us, 13577 54.9 -> 52.9, 28 layers of 13577 439 -> 433.
// They go to `smoothed` as well, for every head: nothing in evict reads them there, but what a workspace holds of a call afterwards
// does not depend on who combined the chunks (tests compare it with smooth's result). The stores cost 0.8 us of 53 at 13577 tokens
// and 1.2 of 137 on 40 layers of 12000.
template <int EPT, int NT, int R>
__device__ __forceinline__ void joined_scores(const Geom& g, const ConvJoin& j, const ConvHead& w, int head, int n_cand, float* smoothed,
                                              float (&x)[EPT]) {
    constexpr int C = 1 << kJoinLogC, PER = C / NT;          // points per thread
    const int tid = threadIdx.x;
    const cf* p = reinterpret_cast<const cf*>(j.part) + (size_t)head * j.part_stride;
    cf v[PER][16];
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int r = 0; r < R; ++r) v[i][r] = p[(size_t)r * C + tid + i * NT];
    __builtin_amdgcn_sched_barrier(0);                       // all loads before the first result is worked on
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        float o[16];
        join<R>(v[i], o);
#pragma unroll
        for (int t = 0; t < R; ++t) x[i + PER * t] = o[t];
    }
    if (j.alpha != 1.f) {
        const float* src = j.in + w.off;
#pragma unroll
        for (int e = 0; e < PER * R; ++e) {
            const int n = tid + e * NT;
            if (n < w.L) x[e] = mix(j.pool_on_load ? pooled_at(src, w.L, n, g.pool_kernel, g.pool_mode) : src[n], x[e], j.alpha);
        }
    }
    // (a buffer of the head's size: what lies past its end is not stored. The whole offset goes into the operand that is checked
    // against that size; the scalar one is not.)
    const auto buf = __builtin_amdgcn_make_buffer_rsrc(smoothed, 0, w.L * 4, 0x00027000);
#pragma unroll
    for (int e = 0; e < PER * R; ++e) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(x[e]), buf, (tid + e * NT) * 4, 0, 0);
#pragma unroll
    for (int e = 0; e < EPT; ++e) x[e] = e < PER * R && tid + e * NT < n_cand ? x[e] : 0.f;
}

// EPT, NT: tokens per thread, threads; the head must have at most EPT * NT candidates. JOIN: some heads' scores are left in chunks.
template <int EPT, int NT, bool JOIN>
__global__ __launch_bounds__(NT) void select_kernel(
    Geom g, const float* __restrict__ all_scores, const int32_t* __restrict__ budgets,
    const int32_t* __restrict__ cu_b, const int32_t* __restrict__ cu_seq, int32_t* __restrict__ indices, ConvJoin chunks, float* smoothed)
{
    const int head = blockIdx.x;
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tok0 = cu_seq[item];
    const int L = cu_seq[item + 1] - tok0;
    const float* head_scores = all_scores + (size_t)tok0 * g.H_kv + (size_t)h * L;
    // (a head that keeps only its window: its smoothed scores are stored all the same)
    constexpr bool always = JOIN;
    const auto scores = [&](float (&x)[EPT], int n_cand) {
        const auto load = [&]() {
            // (a buffer of the candidates' size reads as zero past its end: no clamped addresses, all loads of a thread in flight. As
            // with the stores above, the whole offset is in the operand that is checked.)
            const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(head_scores), 0, n_cand * 4, 0x00027000);
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                x[e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, ((int)threadIdx.x + e * NT) * 4, 0, 0));
        };
        if constexpr (JOIN) {
            constexpr int kMaxR = EPT * NT >> kJoinLogC;
            static_assert(kMaxR == 2 || kMaxR == 4, "the cases below");
            ConvHead w;
            const int R = conv_head(g, chunks.job, head, kJoinLogC, w) ? w.R : 1;     // (a head of one chunk is done)
            if (R == 2) joined_scores<EPT, NT, 2>(g, chunks, w, head, n_cand, smoothed + w.off, x);
            else if (R == 4) joined_scores<EPT, NT, kMaxR>(g, chunks, w, head, n_cand, smoothed + w.off, x);
            else load();
        } else {
            load();
        }
    };
#include "select_body.h"
}

// Heads longer than 32 * 1024 tokens: the keys do not fit the registers of one workgroup, so every counting pass
// streams the scores again (they stay in L2: 4 bytes per token), and the output pass walks the sequence in rounds of
// 32 consecutive tokens per thread. Same threshold, same tie rule, same ascending order; slower per token than the
// register kernel (32 full passes), meant for the rare very long head.
__global__ __launch_bounds__(kSelThreads) void select_stream_kernel(
    Geom g, const float* __restrict__ scores, const int32_t* __restrict__ budgets,
    const int32_t* __restrict__ cu_b, const int32_t* __restrict__ cu_seq, int32_t* __restrict__ indices)
{
    __shared__ int slots[4 * kSelWaves];
    __shared__ uint32_t short_list[kCompact * kSelThreads];
    __shared__ int list_n;
    const int head = blockIdx.x;
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tok0 = cu_seq[item];
    const int L = cu_seq[item + 1] - tok0;
    const float* s = scores + (size_t)tok0 * g.H_kv + (size_t)h * L;
    const int tid = threadIdx.x;

    const int W = min(g.W, L);
    const int n_cand = L - W;
    const int room = cu_b[head + 1] - cu_b[head];
    const int b = min(min(max(budgets[head], W), L), room);
    const int want = max(b - W, 0);
    int32_t* out = indices + cu_b[head];
    for (int w = tid; w < W; w += kSelThreads)
        if (want + w < room) out[want + w] = n_cand + w;
    if (want <= 0) return;

    // the largest T with #(key >= T) >= want, bit by bit; c_up ends as #(key > T): the count of the last trial that
    // failed, which is T + 1 (all lower bits of T are ones from there down)
    uint32_t T = 0;
    int c_lo = n_cand, c_up = 0, parity = 0;
    int bit = 31;
    bool narrow = false;
    for (; bit >= 0; --bit) {
        const uint32_t trial = T | (1u << bit);
        int c = 0;
        for (int j0 = tid; j0 < n_cand; j0 += 16 * kSelThreads) {      // 16 loads in flight: clamped address, masked count
            float f[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) f[u] = s[min(j0 + u * kSelThreads, n_cand - 1)];
#pragma unroll
            for (int u = 0; u < 16; ++u) c += (j0 + u * kSelThreads < n_cand && order_key(f[u]) >= trial) ? 1 : 0;
        }
        const int t = block_count(c, slots, parity);
        parity ^= 1;
        if (t >= want) { T = trial; c_lo = t; } else { c_up = t; }
        // the keys that the remaining bits can still tell apart are those whose upper bits equal T's: once they fit
        // the short list, one more streaming pass collects them and the rest of the search never touches memory
        if (bit > 0 && c_lo - c_up <= kCompact * kSelThreads) { narrow = true; break; }
    }
    if (narrow) {
        const uint32_t hi_part = T >> bit;
        if (tid == 0) list_n = 0;
        __syncthreads();
        for (int j0 = tid; j0 < n_cand; j0 += 16 * kSelThreads) {
            float f[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) f[u] = s[min(j0 + u * kSelThreads, n_cand - 1)];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const uint32_t key = order_key(f[u]);
                const bool mine = j0 + u * kSelThreads < n_cand && (key >> bit) == hi_part;
                // the order of the list does not matter (it is only counted): one LDS add per wave and step
                const unsigned long long m = __builtin_amdgcn_ballot_w64(mine);
                int base = 0;
                if (m) {
                    if ((tid & 63) == 0) base = atomicAdd(&list_n, __builtin_popcountll(m));
                    base = __shfl(base, 0, 64);
                    const int pos = base + __builtin_popcountll(m & ((1ull << (tid & 63)) - 1ull));
                    if (mine && pos < kCompact * kSelThreads) short_list[pos] = key;   // (the counts say it always fits)
                }
            }
        }
        __syncthreads();
        const int n_und = c_lo - c_up;                   // == list_n
        const int c_above = c_up;
        uint32_t ckey[kCompact];
#pragma unroll
        for (int e = 0; e < kCompact; ++e) {
            const int i = tid + e * kSelThreads;
            ckey[e] = i < n_und ? short_list[i] : 0u;
        }
        for (--bit; bit >= 0; --bit) {
            const uint32_t trial = T | (1u << bit);
            int c = 0;
#pragma unroll
            for (int e = 0; e < kCompact; ++e) c += (tid + e * kSelThreads < n_und && ckey[e] >= trial) ? 1 : 0;
            const int t = c_above + block_count(c, slots, parity);
            parity ^= 1;
            if (t >= want) T = trial; else c_up = t;
        }
    }
    const int need_eq = want - c_up;

    int gt_base = 0, eq_base = 0;                    // tokens > T and == T in the rounds before this one
    for (int base = 0; base < n_cand; base += 32 * kSelThreads) {
        const int j0 = base + tid * 32;
        uint32_t mg = 0, me = 0;
        float f[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) f[u] = s[min(j0 + u, n_cand - 1)];
#pragma unroll
        for (int u = 0; u < 32; ++u) {
            const uint32_t key = order_key(f[u]);
            const bool live = j0 + u < n_cand;
            mg |= (live && key > T ? 1u : 0u) << u;
            me |= (live && key == T ? 1u : 0u) << u;
        }
        int gt_before, eq_before;
        block_exscan2(__builtin_popcount(mg), __builtin_popcount(me), slots + 2 * kSelWaves, gt_before, eq_before);
        int gt_round = 0, eq_round = 0;
        for (int w = 0; w < kSelWaves; ++w) { gt_round += slots[2 * kSelWaves + w]; eq_round += slots[3 * kSelWaves + w]; }
        gt_before += gt_base;
        eq_before += eq_base;
        uint32_t m = mg | me;
        while (m) {
            const int bpos = __builtin_ctz(m);
            m &= m - 1;
            if ((mg >> bpos) & 1u) {
                out[gt_before + min(eq_before, need_eq)] = j0 + bpos;
                ++gt_before;
            } else {
                if (eq_before < need_eq) out[gt_before + eq_before] = j0 + bpos;
                ++eq_before;
            }
        }
        gt_base += gt_round;
        eq_base += eq_round;
        __syncthreads();                             // the scan slots are rewritten by the next round
    }
}

}  // namespace

bool select_supported(int L) { return L >= 1; }
bool select_joins(int max_L) { return max_L <= kJoinMaxR << kJoinLogC; }

hipError_t launch_select(const Geom& g, const float* scores, const int32_t* budgets, const int32_t* cu_budgets,
                         const int32_t* cu_seqlens, int max_L, int32_t* indices, hipStream_t s, const ConvJoin* join)
{
    const int n_heads = g.n_items * g.H_kv;
#define AUDIOKV_LAUNCH_SELECT(E, NT, J)                                                                 \
    do {                                                                                                \
        hipLaunchKernelGGL((select_kernel<E, NT, J>), dim3(n_heads), dim3(NT), 0, s, g, scores, budgets, \
                           cu_budgets, cu_seqlens, indices, join ? *join : ConvJoin{}, join ? join->out : nullptr); \
    } while (0)
    if (join) {
        // (a head in chunks has more than 4096 tokens)
        if (max_L <= 8192) AUDIOKV_LAUNCH_SELECT(8, 1024, true);
        else if (select_joins(max_L)) AUDIOKV_LAUNCH_SELECT(16, 1024, true);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // Four tokens per thread while the head lasts: fewer waves make the barriers cheaper (512 threads against 1024 at
    // 2048 tokens 4.2 us against 4.9), more tokens per thread make every pass longer (256 threads of eight 5.6 us, 512 of
    // eight at 4096 tokens 5.8 us against 4.9, 512 of sixteen at 8192 tokens 8.2 us against 7.1).
    if (max_L <= 2048) AUDIOKV_LAUNCH_SELECT(4, 512, false);
    else if (max_L <= 4096) AUDIOKV_LAUNCH_SELECT(4, 1024, false);
    else if (max_L <= 8192) AUDIOKV_LAUNCH_SELECT(8, 1024, false);
    else if (max_L <= 16384) AUDIOKV_LAUNCH_SELECT(16, 1024, false);
    else if (max_L <= 32768) AUDIOKV_LAUNCH_SELECT(32, 1024, false);
    else   // longer heads than the registers and the LDS staging of one workgroup hold
        hipLaunchKernelGGL(select_stream_kernel, dim3(n_heads), dim3(kSelThreads), 0, s, g, scores, budgets, cu_budgets,
                           cu_seqlens, indices);
#undef AUDIOKV_LAUNCH_SELECT
    return hipGetLastError();
}

}  // namespace audiokv
