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

namespace audiokv {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

// float -> uint32 whose unsigned order is the float order; -0.0 and +0.0 map to one key
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// its inverse
__device__ __forceinline__ float key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}

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

// Workgroup barrier that orders LDS traffic only: nothing is exchanged through memory, and the stores on their way (the window's
// indices, scores combined from chunks) are no reason to wait.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Largest value over the lanes of a full wave, in lane 63 (the sum likewise)
#define AUDIOKV_DPP_F(x, ctrl, rows, none) \
    __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(x), ctrl, rows, 0xf, false))
#define AUDIOKV_WAVE_FOLD(op, x, none)                      \
    do {                                                    \
        x = op(x, AUDIOKV_DPP_F(x, 0x111, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x112, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x114, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x118, 0xf, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x142, 0xa, none));      \
        x = op(x, AUDIOKV_DPP_F(x, 0x143, 0xc, none));      \
    } while (0)
// the same over the first N lanes, a power of two up to 16: in lane N - 1
#define AUDIOKV_ROW_FOLD(op, x, none, N)                    \
    do {                                                    \
        x = op(x, AUDIOKV_DPP_F(x, 0x111, 0xf, none));      \
        if (N > 2) x = op(x, AUDIOKV_DPP_F(x, 0x112, 0xf, none)); \
        if (N > 4) x = op(x, AUDIOKV_DPP_F(x, 0x114, 0xf, none)); \
        if (N > 8) x = op(x, AUDIOKV_DPP_F(x, 0x118, 0xf, none)); \
    } while (0)
__device__ __forceinline__ float plus(float a, float b) { return a + b; }
__device__ __forceinline__ float wave_sum63(float x) { AUDIOKV_WAVE_FOLD(plus, x, 0.f); return x; }
__device__ __forceinline__ float wave_max63(float x) { AUDIOKV_WAVE_FOLD(fmaxf, x, -INFINITY); return x; }
template <int N> __device__ __forceinline__ float row_sum(float x) { AUDIOKV_ROW_FOLD(plus, x, 0.f, N); return x; }
template <int N> __device__ __forceinline__ float row_max(float x) { AUDIOKV_ROW_FOLD(fmaxf, x, -INFINITY, N); return x; }
__device__ __forceinline__ float lane_float(float x, int lane) {           // uniform lane
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
#undef AUDIOKV_ROW_FOLD
#undef AUDIOKV_WAVE_FOLD
#undef AUDIOKV_DPP_F

constexpr int kCompact = 8;          // undecided keys per thread once the streaming kernel has narrowed the candidates down
constexpr int kDigitBits = 11, kBins = 1 << kDigitBits;   // bins of one histogram round
constexpr int kLast = 64;            // candidates that one wave ranks against each other

// Inclusive sum over the first N lanes, a power of two up to 16
template <int N>
__device__ __forceinline__ int row_incl(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    if (N > 2) x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    if (N > 4) x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    if (N > 8) x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    return x;
}

// Largest value over the lanes of a full wave, in lane 63.
__device__ __forceinline__ uint32_t wave_max63(uint32_t x) {
#define AUDIOKV_MAX_STEP(ctrl, rows) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, rows, 0xf, false))
    AUDIOKV_MAX_STEP(0x111, 0xf);
    AUDIOKV_MAX_STEP(0x112, 0xf);
    AUDIOKV_MAX_STEP(0x114, 0xf);
    AUDIOKV_MAX_STEP(0x118, 0xf);
    AUDIOKV_MAX_STEP(0x142, 0xa);
    AUDIOKV_MAX_STEP(0x143, 0xc);
#undef AUDIOKV_MAX_STEP
    return x;
}

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
    Geom g, const float* __restrict__ scores, const int32_t* __restrict__ budgets,
    const int32_t* __restrict__ cu_b, const int32_t* __restrict__ cu_seq, int32_t* __restrict__ indices, ConvJoin chunks, float* smoothed)
{
    constexpr int NW = NT / 64;
    constexpr int kFine = EPT * NT <= 2048 ? 2048 : EPT * NT <= 16384 ? 4096 : 8192;    // parts of the first division
    constexpr int kFinePer = kFine / NT;             // parts per thread in the scan
    constexpr int kPer = kBins / NT;                 // the same in the general search
    constexpr int kChunks = EPT * NW;                // chunks of 64 consecutive tokens, in token order
    constexpr int kChunkPer = (kChunks + 63) / 64;   // chunks per lane in their scan
    static_assert(kFinePer % 2 == 0 && kFine >= kBins, "the histograms share their memory");
    __shared__ __attribute__((aligned(16))) int hist[kFine];
    __shared__ __attribute__((aligned(16))) int chunk_n[kChunkPer * 64];
    __shared__ __attribute__((aligned(16))) unsigned long long last[kLast];
    __shared__ int upto_thread[NT];                  // inclusive counts within a wave
    __shared__ float part[4 * NW];                   // per wave: sums, or extremes
    __shared__ uint32_t extreme[2 * NW];             // per wave: largest key, largest complement of a key
    __shared__ int wave_n[NW];
    __shared__ int pick[3];
    __shared__ int last_n;
    const int head = blockIdx.x;
    const int item = head / g.H_kv, h = head - item * g.H_kv;
    const int tok0 = cu_seq[item];
    const int L = cu_seq[item + 1] - tok0;
    const float* s = scores + (size_t)tok0 * g.H_kv + (size_t)h * L;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wave_at = wave * 64;

    const int W = min(g.W, L);
    const int n_cand = L - W;
    // never write past this head's slice of the output, whatever the caller's budgets say
    const int room = cu_b[head + 1] - cu_b[head];
    const int b = min(min(max(budgets[head], W), L), room);
    const int want = max(b - W, 0);                  // how many candidates to keep
    int32_t* out = indices + cu_b[head];

    // the forced window tail: highest indices, so they close the ascending list
    for (int w = tid; w < W; w += NT)
        if (want + w < room) out[want + w] = n_cand + w;
    if (!JOIN && want <= 0) return;
    if (n_cand > EPT * NT) return;                   // launcher never allows this

    // (a buffer of the candidates' size reads as zero past its end: no clamped addresses, all loads of a thread in flight. As with
    // the stores above, the whole offset is in the operand that is checked.)
    // A value that the compiler is to take for another one from here on: lane masks of comparisons with it are formed again
    // where they are needed again, instead of 32 pairs of scalar registers being kept (and spilled).
    auto renewed = [](auto& v) {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+s"(v));
#endif
    };
    int n_live = n_cand;
    const auto live = [&](int e) { return tid < n_live - e * NT; };
    const auto full = [&](int e) { return (e + 1) * NT <= n_cand; };            // uniform
    const auto any = [&](int e) { return e * NT + wave_at < n_cand; };          // uniform over the wave
    const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(s), 0, n_cand * 4, 0x00027000);
    float x[EPT];
    const auto load = [&]() {
#pragma unroll
        for (int e = 0; e < EPT; ++e) x[e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, (tid + e * NT) * 4, 0, 0));
    };
    if constexpr (JOIN) {
        constexpr int kMaxR = EPT * NT >> kJoinLogC;
        static_assert(kMaxR == 2 || kMaxR == 4, "the cases below");
        ConvHead w;
        const int R = conv_head(g, chunks.job, head, kJoinLogC, w) ? w.R : 1;     // (a head of one chunk is done)
        if (R == 2) joined_scores<EPT, NT, 2>(g, chunks, w, head, n_cand, smoothed + w.off, x);
        else if (R == 4) joined_scores<EPT, NT, kMaxR>(g, chunks, w, head, n_cand, smoothed + w.off, x);
        else load();
        if (want <= 0) return;                       // (its smoothed scores are stored all the same)
    } else {
        load();
    }
#pragma unroll
    for (int u = 0; u < kFine / NT; u += 2) *reinterpret_cast<int2*>(&hist[u * NT + 2 * tid]) = make_int2(0, 0);
    if (tid == 0) last_n = 0;

    // Mean and deviation. (Sums of scores and squares: where the deviation is so small beside the mean that they cancel, the
    // parts come out too wide or too narrow and the search takes longer.)
    const bool few = 12 * (long long)want < n_cand, most = 12 * (long long)(n_cand - want) < n_cand;   // (uniform) below a twelfth, above eleven
    float s1 = 0.f, s2 = 0.f, end = -INFINITY;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        s1 += x[e];
        s2 = fmaf(x[e], x[e], s2);
    }
    if (few || most) {
        const float sign = few ? 1.f : -1.f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) end = fmaxf(end, live(e) ? sign * x[e] : -INFINITY);
        end = wave_max63(end);
    }
    s1 = wave_sum63(s1);
    s2 = wave_sum63(s2);
    if (lane == 63) { part[wave] = s1; part[NW + wave] = s2; part[2 * NW + wave] = end; }
    lds_barrier();
    float hi, inv;
    {
        const auto of_wave = [&](int which, float none) { return lane < NW ? part[which * NW + (lane < NW ? lane : 0)] : none; };
        const float n_inv = __builtin_amdgcn_rcpf((float)n_cand), mean = lane_float(row_sum<NW>(of_wave(0, 0.f)), NW - 1) * n_inv;
        const float dev = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-mean, mean, lane_float(row_sum<NW>(of_wave(1, 0.f)), NW - 1) * n_inv), 0.f));
        hi = fmaf(2.f, dev, mean);
        float lo = fmaf(-2.f, dev, mean);
        if (few || most) {
            const float top = lane_float(row_max<NW>(of_wave(2, -INFINITY)), NW - 1);
            if (few) hi = fmaxf(hi, top);
            else lo = fminf(lo, -top);
        }
        inv = (float)kFine * __builtin_amdgcn_rcpf(hi - lo);
        if (!(inv > 0.f && fabsf(hi) * inv < INFINITY)) inv = 0.f;       // no number, no end, or no width: the general search
    }
    // part of a score: falls as the score rises, rounded and cut off alike for all
    const float at0 = hi * inv;
    const auto fine = [&](int e) { return (int)__builtin_amdgcn_fmed3f(fmaf(x[e], -inv, at0), 0.f, (float)(kFine - 1)); };

    // a token past the end is below everything
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (!full(e)) x[e] = live(e) ? x[e] : -INFINITY;

    renewed(n_live);
    int rank = want, inside = n_cand;
    // Adds to one part take their turns, which a long head with many equal scores would wait for: a wave that finds a quarter
    // of the lanes of a register in one part counts that part from lane masks and adds it once (half zeros at 32768 tokens
    // 30 -> 20 us, all equal but one 64 -> 39). Heads of up to eight registers finish sooner without. Registers past the end look
    // crowded but hold no candidates (left in: half zeros at 18000 tokens 22 us instead of 17, random scores 16.2 instead of 14.5).
    auto add_all = [&](auto part_of, auto counts) {
        int crowded = -1, many = 15;
        if constexpr (EPT >= 16) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = (int)part_of(u * (EPT / 4));
                const int one = __builtin_amdgcn_readlane(p, 21 * u);
                const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(counts(u * (EPT / 4)) && p == one));
                if (n > many) { many = n; crowded = one; }
            }
        }
        if (crowded < 0) {
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (any(e) && counts(e)) atomicAdd(&hist[part_of(e)], 1);
        } else {
            int n = 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int p = (int)part_of(e);
                n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(counts(e) && p == crowded));
                if (counts(e) && p != crowded) atomicAdd(&hist[p], 1);
            }
            if (lane == 0 && n) atomicAdd(&hist[crowded], n);
        }
    };
    // The part at which the running count reaches `rank`: every wave looks for the wave, then the thread, then the part. The rank
    // in it and what it holds follow.
    auto locate = [&]() -> int {
        lds_barrier();
        int sum = 0;
#pragma unroll
        for (int u = 0; u < kFinePer; u += 2) {
            const int2 n = *reinterpret_cast<const int2*>(&hist[tid * kFinePer + u]);
            sum += n.x + n.y;
        }
        const int incl = wave_incl(sum);
        upto_thread[tid] = incl;
        if (lane == 63) wave_n[wave] = incl;
        lds_barrier();
        int before = 0;
        auto first_at = [&](int upto) {              // `upto` rises with the lanes and reaches rank
            const int l = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto >= rank) | (1ull << 63));
            before = l > 0 ? __builtin_amdgcn_readlane(upto, l > 0 ? l - 1 : 0) : before;
            return l;
        };
        const int w = first_at(row_incl<NW>(lane < NW ? wave_n[lane < NW ? lane : 0] : 0)) & (NW - 1);
        const int t = w * 64 + first_at(before + upto_thread[w * 64 + lane]);
        const int n_at = lane < kFinePer ? hist[t * kFinePer + (lane < kFinePer ? lane : 0)] : 0;
        const int u = first_at(before + row_incl<kFinePer>(n_at)) & (kFinePer - 1);
        inside = __builtin_amdgcn_readlane(n_at, u);
        rank -= before;
        return t * kFinePer + u;
    };
    const bool divided = n_cand > kLast && inv > 0.f;
    int bin = 0, bin2 = -1;
    // a part divided in the same way
    const auto finer = [&](int e) { return (int)__builtin_amdgcn_fmed3f((fmaf(x[e], -inv, at0) - (float)bin) * (float)kFine, 0.f, (float)(kFine - 1)); };
    const auto in_part = [&](int e) { return fine(e) == bin && (bin2 < 0 || finer(e) == bin2); };
    if (divided) {
        // (tokens past the end of a wave's last register count in the last part: no harm, the part ends with them)
        add_all(fine, any);
        bin = locate();
        // Too many, in a part with two ends: once more, unless the parts beside it are empty (a few values that many share)
        if (inside > kLast && bin > 0 && bin < kFine - 1 && hist[max(bin - 1, 0)] + hist[min(bin + 1, kFine - 1)] > 0) {
            lds_barrier();                         // (the counts are read)
#pragma unroll
            for (int u = 0; u < kFine / NT; u += 2) *reinterpret_cast<int2*>(&hist[u * NT + 2 * tid]) = make_int2(0, 0);
            lds_barrier();
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (fine(e) == bin) atomicAdd(&hist[finer(e)], 1);
            bin2 = locate();
        }
    }

    // The 64 candidates at most that are left: every wave ranks them by (score falling, index), one per lane, against all. No
    // two are equal, so exactly one is number `rank`.
    // (rank: afterwards among those that share its score; more: some of them come after it)
    auto rank_last = [&](uint32_t& at, bool& more) {
        lds_barrier();
        const int n_last = min(last_n, kLast);
        const unsigned long long mine = last[min(lane, n_last - 1)];
        int upto = 0;
#pragma unroll 4
        for (int i = 0; i < n_last; ++i) upto += last[i] <= mine ? 1 : 0;
        const int winner = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto == rank) | (1ull << 63));
        at = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), winner);
        more = __builtin_amdgcn_ballot_w64((uint32_t)(mine >> 32) == at && upto > rank) != 0;
        rank -= __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n_last && (uint32_t)(mine >> 32) < at));
    };
    auto put_last = [&](uint32_t order, int e) {
        const int pos = atomicAdd(&last_n, 1);
        if (pos < kLast) last[pos] = ((unsigned long long)order << 32) | (uint32_t)(tid + e * NT);
    };

    // For a fixed register e, wave w holds the 64 consecutive tokens of chunk e * NW + w. Counts of the chunks (lane e has that of
    // register e), scanned: every wave scans all the chunks for itself, kChunkPer per lane, and has those ahead of its own in
    // lane (e * NW + wave) / kChunkPer.
    auto scan_chunks = [&](int my_n) {
        if (lane < EPT) chunk_n[lane * NW + wave] = my_n;
        if (kChunks < 64 && tid >= kChunks && tid < 64) chunk_n[tid] = 0;
        lds_barrier();
        int sum = 0, ahead = 0;                      // a lane's chunks; those before the one of this wave
#pragma unroll
        for (int u = 0; u < kChunkPer; ++u) {
            const int c = chunk_n[lane * kChunkPer + u];
            if (u < (wave & (kChunkPer - 1))) ahead += c;
            sum += c;
        }
        return ahead + (wave_incl(sum) - sum);
    };
    const auto lanes_before = [&](unsigned long long m, int from) {
        return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)from));
    };

    // Writes the tokens that are larger than the threshold, and the first `rank` of those equal to it. Both are counted per
    // chunk, in two halves of a number (32768 tokens at most).
    auto write_first = [&](uint32_t threshold, auto larger, auto equal) {
        int my_n = 0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            if (EPT <= 4 && !any(e)) continue;       // (four registers are what the shortest heads have: most of them empty)
            const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(larger(e, threshold))) |
                          __builtin_popcountll(__builtin_amdgcn_ballot_w64(equal(e, threshold))) << 16;
            asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(my_n) : "s"(c), "n"(e));
        }
        const int ahead = scan_chunks(my_n);
        renewed(threshold);
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            if (EPT <= 4 && !any(e)) continue;
            const uint32_t at = (uint32_t)__builtin_amdgcn_readlane(ahead, (e * NW + wave) / kChunkPer);
            const int equal_before = (int)(at >> 16), first = (int)(at & 0xffffu) + min(equal_before, rank);
            const bool same = equal(e, threshold);
            const bool k = larger(e, threshold) || (same && lanes_before(__builtin_amdgcn_ballot_w64(same), equal_before) < rank);
            const int pos = lanes_before(__builtin_amdgcn_ballot_w64(k), first);
            if (k && pos < want) out[pos] = tid + e * NT;
        }
    };

    uint32_t T;                                      // the threshold's order key
    if (divided && inside <= kLast) {
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (in_part(e) && live(e)) put_last(~order_key(x[e]), e);
        bool more;
        rank_last(T, more);
        T = ~T;
        if (!more) {                                 // (uniform) all that share the threshold's score stay
            uint32_t least = __float_as_uint(key_value(T));
            int my_n = 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(x[e] >= __uint_as_float(least)));
                asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(my_n) : "s"(c), "n"(e));
            }
            const int ahead = scan_chunks(my_n);
            renewed(least);
            // every kept token writes itself to its slot: the slots of a wave's tokens are consecutive, so each store
            // instruction writes one run of the output
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const bool k = x[e] >= __uint_as_float(least);
                const int pos = lanes_before(__builtin_amdgcn_ballot_w64(k), __builtin_amdgcn_readlane(ahead, (e * NW + wave) / kChunkPer));
                if (k && pos < want) out[pos] = tid + e * NT;
            }
            return;
        }
    } else {
        // ---- the general search, among what is in the part found so far (or all candidates) ----
        // From here on a key is its distance below the largest one, and what is no candidate is further than all (keys are at
        // least 1, which only the lowest NaN would not be, so no distance is 0xffffffff). Shorter distances come first.
        lds_barrier();                                 // (the parts' counts are read)
        renewed(n_live);
        uint32_t key[EPT];
        uint32_t big = 0, small = 0;                     // (the complement of the smallest)
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const bool c = live(e) && (!divided || in_part(e));
            key[e] = c ? max(order_key(x[e]), 1u) : 0u;
            big = max(big, key[e]);
            small = max(small, c ? ~key[e] : 0u);
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) hist[tid + u * NT] = 0;
        big = wave_max63(big);
        small = wave_max63(small);
        if (lane == 63) { extreme[wave] = big; extreme[NW + wave] = small; }
        lds_barrier();
        {
            const uint32_t a = extreme[lane & (NW - 1)], c = extreme[NW + (lane & (NW - 1))];
            big = (uint32_t)__builtin_amdgcn_readlane((int)wave_max63(a), 63);
            small = ~(uint32_t)__builtin_amdgcn_readlane((int)wave_max63(c), 63);
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) key[e] = key[e] ? big - key[e] : 0xffffffffu;
        auto cand = [&](int e) { return key[e] != 0xffffffffu; };

        // The bracket: candidates with distances in [d0, d0 + lim]. It holds `inside` candidates, the threshold (number `rank` of
        // them in order, from 1) among them.
        int nb = 32 - __builtin_clz((big - small) | 1u);   // distances have at most nb bits
        uint32_t d0 = 0, lim = 0xffffffffu >> (32 - nb);
        // One add per candidate, but candidates that may all be equal: the lanes that share the first one's bin as one number.
        auto add_shared = [&](int bin) {
            const int b0 = __builtin_amdgcn_readfirstlane(bin);
            const unsigned long long m = __builtin_amdgcn_ballot_w64(bin == b0);
            if (bin != b0) atomicAdd(&hist[bin], 1);
            else if (lane == __builtin_ctzll(m)) atomicAdd(&hist[bin], __builtin_popcountll(m));
        };

        // After the bins of a round are counted: the first bin at which the running count reaches `rank`.
        auto settle = [&]() -> int {
            lds_barrier();
            int n[kPer], sum = 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u) { n[u] = hist[tid * kPer + u]; sum += n[u]; }
#pragma unroll
            for (int u = 0; u < kPer; ++u) hist[tid * kPer + u] = 0;      // for the next round
            int incl = wave_incl(sum);
            if (lane == 63) wave_n[wave] = incl;
            lds_barrier();
            const int wn = lane < NW ? wave_n[lane < NW ? lane : 0] : 0;
            const int before = wave == 0 ? 0 : __builtin_amdgcn_readlane(row_incl<NW>(wn), wave - 1);
            int c = before + incl - sum;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                if (c < rank && rank <= c + n[u]) { pick[0] = tid * kPer + u; pick[1] = c; pick[2] = n[u]; }   // exactly one bin
                c += n[u];
            }
            lds_barrier();
            rank -= pick[1];
            inside = pick[2];
            return pick[0];
        };

        // Rounds over the bits of the distance, eleven at a time. The first one counts every candidate, later ones, rare, those
        // that are left.
        if (inside > kLast && big != small) {
            int sh = max(nb - kDigitBits, 0);
            add_all([&](int e) { return key[e] >> sh; }, cand);
            d0 = (uint32_t)settle() << sh;
            nb = sh;
            lim = (1u << nb) - 1u;
            while (inside > kLast && nb > 0) {           // uniform
                sh = max(nb - kDigitBits, 0);
#pragma unroll
                for (int e = 0; e < EPT; ++e)
                    if (key[e] - d0 <= lim && cand(e)) add_shared((int)((key[e] - d0) >> sh));
                d0 += (uint32_t)settle() << sh;
                nb = sh;
                lim = (1u << nb) - 1u;
            }
        }
        if (inside > kLast || big == small) {          // all that are left share the threshold's score
            T = big - d0;
        } else {
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (key[e] - d0 <= lim && cand(e)) put_last(key[e], e);
            bool more;
            rank_last(T, more);
            T = big - T;
        }
    }

    if (divided) {                                 // (all scores are finite)
        write_first(__float_as_uint(key_value(T)), [&](int e, uint32_t v) { return x[e] > __uint_as_float(v); },
                    [&](int e, uint32_t v) { return x[e] == __uint_as_float(v); });
    } else {
        const auto order = [&](int e) { return live(e) ? max(order_key(x[e]), 1u) : 0u; };
        write_first(T, [&](int e, uint32_t v) { return order(e) > v; }, [&](int e, uint32_t v) { return order(e) == v; });
    }
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
