// Stage 4: per-head top-k with a forced window tail (paper Sec. 1, Solution 2:
// Top-K selection on the importance scores; window w of Sec. 3.1 Eq. 1).
//
// One workgroup per head. Scores become order-preserving 32-bit keys held in
// registers (token t + NT e in register e of thread t: coalesced loads). The
// extremes of the keys give their range; a histogram of 2048 equal parts of the
// range, counted in LDS, gives the part that the threshold lies in. If it holds
// more than 64 candidates, it is divided in the same way again, and once its
// keys are all equal, by token index (ties are kept in index order, so key and
// index together order the candidates strictly). The last candidates, 64 at
// most, are ranked against each other by every wave for itself, which gives the
// threshold as a key T and an index X: a token stays if its key is larger than
// T, or equal to T and its index at most X. For a fixed register the lanes of a
// wave hold 64 consecutive tokens, so one lane mask gives every (register, wave)
// chunk its count, a scan over the chunks their output offsets, and every kept
// token computes its own ascending output slot from the offset and its rank in
// the lane mask. Integer-only (counts and integer adds in any order): bit-exact.
//
// What bounds it is the chain of one head: the loads of up to 128 KB by one CU
// and six barriers. Rounds of 2048 parts over the range that is there take the
// place of one counting pass per bit (short heads) and of pivots from a sample
// (long ones). Four heads of 2048 tokens 10.6 -> 4.2 us, 8192 12.7 -> 6.3, 16384
// 14.5 -> 9.0, 32768 21.9 -> 15.2; 112 heads of 16384 17.6 -> 10.9. Two, four or
// eight workgroups per head that each find the threshold and write a part gain
// nothing with four heads (14.8 us at 32768, 8.4 at 16384) and lose with 112
// (11.7 and more): every one of them has to load the whole head.
#include "common.h"

namespace audiokv {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

// float -> uint32 whose unsigned order is the float order; -0.0 and +0.0 map to one key
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
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

constexpr int kCompact = 8;          // undecided keys per thread once the streaming kernel has narrowed the candidates down
constexpr int kDigitBits = 11, kBins = 1 << kDigitBits;   // bins of one histogram round
constexpr int kLast = 64;            // candidates that one wave ranks against each other

// Inclusive sum over the lanes of a full wave, in six data-parallel-primitive steps (no LDS).
__device__ __forceinline__ int wave_incl(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8: prefixes within 16 lanes
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast 31 into rows 2 and 3
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

template <int EPT, int NT>   // tokens per thread, threads; the head must have at most EPT * NT candidates
__global__ __launch_bounds__(NT) void select_kernel(
    Geom g, const float* __restrict__ scores, const int32_t* __restrict__ budgets,
    const int32_t* __restrict__ cu_b, const int32_t* __restrict__ cu_seq, int32_t* __restrict__ indices)
{
    constexpr int NW = NT / 64;
    constexpr int kPer = kBins / NT;                 // bins per thread in the scan
    constexpr int kChunks = EPT * NW;                // chunks of 64 consecutive tokens, in token order
    constexpr int kChunkPer = (kChunks + 63) / 64;   // chunks per lane in their scan
    __shared__ __attribute__((aligned(16))) int hist[kBins];
    __shared__ __attribute__((aligned(16))) int chunk_n[kChunkPer * 64];
    __shared__ __attribute__((aligned(16))) unsigned long long last[kLast];
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
    const int lane = tid & 63, wave = tid >> 6;

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
    if (want <= 0) return;
    if (n_cand > EPT * NT) return;                   // launcher never allows this

    // Thread t holds tokens t, t + NT, t + 2 NT, ...: the loads are coalesced straight into registers, and for a fixed
    // register the lanes of a wave hold 64 consecutive tokens. Past the end a thread loads the last candidate again (clamped address instead of a branch around the load: all loads of a thread are in
    // flight together), which leaves the extremes what they are.
    auto live = [&](int e) { return tid < n_cand - e * NT; };
    uint32_t key[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) key[e] = max(order_key(s[min(tid + e * NT, n_cand - 1)]), 1u);
#pragma unroll
    for (int u = 0; u < kPer; ++u) hist[tid + u * NT] = 0;
    if (tid == 0) last_n = 0;
    uint32_t big = key[0], small = key[0];
#pragma unroll
    for (int e = 1; e < EPT; ++e) { big = max(big, key[e]); small = min(small, key[e]); }
    big = wave_max63(big);
    small = wave_max63(~small);
    if (lane == 63) { extreme[wave] = big; extreme[NW + wave] = small; }
    __syncthreads();
    {
        const uint32_t a = extreme[lane & (NW - 1)], c = extreme[NW + (lane & (NW - 1))];
        big = (uint32_t)__builtin_amdgcn_readlane((int)wave_max63(a), 63);
        small = ~(uint32_t)__builtin_amdgcn_readlane((int)wave_max63(c), 63);
    }

    // From here on a key is its distance below the largest one, and what is no candidate is further than all (keys are
    // at least 1, which only the lowest NaN would not be, so no distance is 0xffffffff). The order: shorter distances first, of equal ones the smaller index.
#pragma unroll
    for (int e = 0; e < EPT; ++e) key[e] = live(e) ? big - key[e] : 0xffffffffu;

    // The bracket: candidates with distances in [d0, d0 + lim] and indices in [i0, i0 + ilim]. It holds `inside`
    // candidates, the threshold (number `rank` of them in order, from 1) among them.
    int nb = 32 - __builtin_clz((big - small) | 1u);   // distances have at most nb bits
    uint32_t d0 = 0, lim = 0xffffffffu >> (32 - nb);
    uint32_t i0 = 0, ilim = (uint32_t)n_cand - 1u;
    int inside = n_cand, rank = want;
    auto in_indices = [&](int e) { return (uint32_t)(tid + e * NT) - i0 <= ilim; };
    // One add per candidate, but candidates that may all be equal: the lanes that share the first one's bin as one number.
    auto add_shared = [&](int bin) {
        const int b0 = __builtin_amdgcn_readfirstlane(bin);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(bin == b0);
        if (bin != b0) atomicAdd(&hist[bin], 1);
        else if (lane == __builtin_ctzll(m)) atomicAdd(&hist[bin], __builtin_popcountll(m));
    };

    // After the bins of a round are counted: the first bin at which the running count reaches `rank`.
    auto settle = [&]() -> int {
        __syncthreads();
        int n[kPer], sum = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) { n[u] = hist[tid * kPer + u]; sum += n[u]; }
#pragma unroll
        for (int u = 0; u < kPer; ++u) hist[tid * kPer + u] = 0;      // for the next round
        int incl = wave_incl(sum);
        if (lane == 63) wave_n[wave] = incl;
        __syncthreads();
        const int wn = lane < NW ? wave_n[lane < NW ? lane : 0] : 0;
        const int before = wave == 0 ? 0 : __builtin_amdgcn_readlane(wave_incl(wn), wave - 1);
        int c = before + incl - sum;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (c < rank && rank <= c + n[u]) { pick[0] = tid * kPer + u; pick[1] = c; pick[2] = n[u]; }   // exactly one bin
            c += n[u];
        }
        __syncthreads();
        rank -= pick[1];
        inside = pick[2];
        return pick[0];
    };

    // Rounds over the bits of the distance, eleven at a time. The first one counts every candidate, later ones, rare, those
    // that are left.
    if (inside > kLast && big != small) {
        int sh = max(nb - kDigitBits, 0);
        // Adds to one bin take their turns, which a long head with many equal scores would wait for: a wave that finds a
        // quarter of the lanes of a register in one bin counts that bin from lane masks and adds it once (half zeros at
        // 32768 tokens 30 -> 20 us, all equal but one 64 -> 39). Heads of up to eight registers finish sooner without. Registers
        // past the end look crowded but hold no candidates (left in: half zeros at 18000 tokens 22 us instead of 17, random
        // scores 16.2 instead of 14.5).
        int crowded = -1, many = 15;
        if constexpr (EPT >= 16) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int bin = (int)(key[u * (EPT / 4)] >> sh);
                const int one = __builtin_amdgcn_readlane(bin, 21 * u);
                const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(live(u * (EPT / 4)) && bin == one));
                if (n > many) { many = n; crowded = one; }
            }
        }
        if (crowded < 0) {
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (live(e)) atomicAdd(&hist[key[e] >> sh], 1);
        } else {
            int n = 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int bin = (int)(key[e] >> sh);
                n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(live(e) && bin == crowded));
                if (live(e) && bin != crowded) atomicAdd(&hist[bin], 1);
            }
            if (lane == 0 && n) atomicAdd(&hist[crowded], n);
        }
        d0 = (uint32_t)settle() << sh;
        nb = sh;
        lim = (1u << nb) - 1u;
        while (inside > kLast && nb > 0) {           // uniform
            sh = max(nb - kDigitBits, 0);
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (key[e] - d0 <= lim && live(e)) add_shared((int)((key[e] - d0) >> sh));
            d0 += (uint32_t)settle() << sh;
            nb = sh;
            lim = (1u << nb) - 1u;
        }
    } else if (big == small) {
        lim = 0;
    }
    // More than 64 candidates tie with the threshold: the same rounds over the bits of their indices.
    if (inside > kLast) {
        nb = 32 - __builtin_clz((uint32_t)n_cand);
        while (inside > kLast) {                     // a bracket of one index holds one candidate: ends
            const int sh = max(nb - kDigitBits, 0);
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (key[e] == d0 && in_indices(e)) add_shared((int)(((uint32_t)(tid + e * NT) - i0) >> sh));
            i0 += (uint32_t)settle() << sh;
            nb = sh;
            ilim = min((1u << nb) - 1u, (uint32_t)n_cand - 1u - i0);
        }
    }

    // At most 64 candidates are left: every wave ranks them by (distance, index), one per lane, against all. No two are
    // equal, so exactly one is number `rank`.
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (key[e] - d0 <= lim && in_indices(e)) {
            const int pos = atomicAdd(&last_n, 1);
            if (pos < kLast) last[pos] = ((unsigned long long)key[e] << 32) | (uint32_t)(tid + e * NT);
        }
    __syncthreads();
    const int n_last = min(last_n, kLast);
    const unsigned long long mine = last[min(lane, n_last - 1)];
    int upto = 0;
#pragma unroll 4
    for (int i = 0; i < n_last; ++i) upto += last[i] <= mine ? 1 : 0;
    const int winner = __builtin_ctzll(__builtin_amdgcn_ballot_w64(upto == rank) | (1ull << 63));
    const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), winner);
    const int X = __builtin_amdgcn_readlane((int)(uint32_t)mine, winner);   // at distance T, tokens up to X stay

    // For a fixed register e, wave w holds the 64 consecutive tokens of chunk e * NW + w. Count the chunk's kept tokens
    // from lane masks (lane e collects register e) ...
    auto kept = [&](int e) { return key[e] < T + (tid <= X - e * NT ? 1u : 0u); };
    int my_n = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(kept(e)));
        asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(my_n) : "s"(c), "n"(e));
    }
    if (lane < EPT) chunk_n[lane * NW + wave] = my_n;
    if (kChunks < 64 && tid >= kChunks && tid < 64) chunk_n[tid] = 0;
    __syncthreads();
    // ... every wave scans all the chunks for itself, kChunkPer per lane, and reads off the offsets of its own ...
    int sum = 0, ahead = 0;                          // a lane's chunks; those before the one of this wave
#pragma unroll
    for (int u = 0; u < kChunkPer; ++u) {
        const int c = chunk_n[lane * kChunkPer + u];
        if (u < (wave & (kChunkPer - 1))) ahead += c;
        sum += c;
    }
    ahead += wave_incl(sum) - sum;
    // ... and every kept token writes itself to its slot: the slots of a wave's tokens are consecutive, so each store
    // instruction writes one run of the output.
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const bool k = kept(e);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(k);
        const int base = __builtin_amdgcn_readlane(ahead, (e * NW + wave) / kChunkPer);
        const int pos = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
        if (k && pos < want) out[pos] = tid + e * NT;
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

hipError_t launch_select(const Geom& g, const float* scores, const int32_t* budgets, const int32_t* cu_budgets,
                         const int32_t* cu_seqlens, int max_L, int32_t* indices, hipStream_t s)
{
    const int n_heads = g.n_items * g.H_kv;
#define AUDIOKV_LAUNCH_SELECT(E, NT)                                                                    \
    do {                                                                                                \
        hipLaunchKernelGGL((select_kernel<E, NT>), dim3(n_heads), dim3(NT), 0, s, g, scores, budgets,    \
                           cu_budgets, cu_seqlens, indices);                                            \
    } while (0)
    // Four tokens per thread while the head lasts: fewer waves make the barriers cheaper (512 threads against 1024 at
    // 2048 tokens 4.2 us against 4.9), more tokens per thread make every pass longer (256 threads of eight 5.6 us, 512 of
    // eight at 4096 tokens 5.8 us against 4.9, 512 of sixteen at 8192 tokens 8.2 us against 7.1).
    if (max_L <= 2048) AUDIOKV_LAUNCH_SELECT(4, 512);
    else if (max_L <= 4096) AUDIOKV_LAUNCH_SELECT(4, 1024);
    else if (max_L <= 8192) AUDIOKV_LAUNCH_SELECT(8, 1024);
    else if (max_L <= 16384) AUDIOKV_LAUNCH_SELECT(16, 1024);
    else if (max_L <= 32768) AUDIOKV_LAUNCH_SELECT(32, 1024);
    else   // longer heads than the registers and the LDS staging of one workgroup hold
        hipLaunchKernelGGL(select_stream_kernel, dim3(n_heads), dim3(kSelThreads), 0, s, g, scores, budgets, cu_budgets,
                           cu_seqlens, indices);
#undef AUDIOKV_LAUNCH_SELECT
    return hipGetLastError();
}

}  // namespace audiokv
