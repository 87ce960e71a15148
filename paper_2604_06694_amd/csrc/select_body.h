// The selection of a head, the text of two function bodies: select_kernel (select.hip) and select_head (select_head.h). Text, and no
// function that both call: as a function that is inlined, the same statements became other code in select_kernel (16 tokens per thread
// 6845 instructions, here 7248; most of the difference is in the general search). Calls on 112 heads of 16384 tokens took 9.6 us either
// way in runs that spread by 0.3 %, but 10.3 and 9.5 in one that spread by 7 %: the kernel is what it was before the smoothing selected too.
//
// What it is given: EPT, NT: tokens per thread, threads; the head must have at most EPT * NT candidates. Geom g; head; its length L;
// budgets, cu_b, indices. scores(x, n_cand): the score of token tid + NT e into x[e], zero from n_cand on; called by all threads, and
// also for a head whose budget is its window if the constant `always` is set.
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
    if (!always && want <= 0) return;
    if (n_cand > EPT * NT) return;                   // launcher never allows this

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
    float x[EPT];
    scores(x, n_cand);
    if (want <= 0) return;
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
