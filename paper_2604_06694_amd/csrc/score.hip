// Host-side planning for the score kernels: which (row blocks per wave, row-splitting waves) instantiation
// covers G*W window rows in each of the two sweeps, and into how many key ranges a head is cut.
#include "score_impl.h"

namespace audiokv {

namespace {

struct Plan { int NB, WR, rows_pad, tile_keys, per_cu; };      // per_cu: resident workgroups

// Instantiated (32-row blocks per wave, waves per workgroup) pairs in order of preference per sweep: the first
// that holds the rows is taken (all must exist in score_d*.hip). More than 448 rows take three row tiles per wave in sweep 1;
// they would spill in sweep 2, which also carries the row constants and covers those rows in two launches. 256 rows in
// sweep 1 with three tiles on three waves, the ninth tile padding: 48 items of 16384 535 us for the whole score call, with two
// tiles on four waves, two workgroups per CU 530; 8 x 32768 183 and 179, 1 x 32768 37.2 and 35.1, ragged 8 x 2000-20000 76.7 and 72.1.
struct Combo { int NB, WR; };
const Combo kSweep1_128[] = {{1, 1}, {1, 2}, {1, 4}, {1, 7}, {2, 4}, {2, 7}, {3, 6}};   // d = 64, 128
const Combo kSweep2_128[] = {{1, 1}, {1, 2}, {1, 4}, {1, 7}, {2, 4}, {2, 7}};
const Combo kCombos256[] = {{1, 1}, {1, 2}, {1, 4}, {1, 7}, {1, 8}};                    // d = 256, both sweeps
// 225 to 256 rows of calls that are over before the chip reaches its power limit: one row tile on each of eight waves instead of two
// on each of four, in both sweeps. Twice the waves hide the latencies of a tile and merge the statistics; each key fragment read from
// LDS feeds one product instead of two, which costs power. Score calls at d = 128, two tiles and one: 1 x 2048 15.7 and 14.8 us,
// 1 x 13577 22.6 and 21.3, 2 x 16384 35.2 and 30.4, 4 x 8192 34.4 and 30.8, 8 x 8192 51.5 and 49.7; 8 x 16384 87.5 and 88.8,
// 16 x 8192 88.0 and 90.0, 48 x 16384 521 and 554 (four KV heads each).
constexpr long long kNarrowTileKeys = 3 << 17;     // keys of all heads: between 8 and 16 items of 8192 tokens and four heads

// keys: of all heads of the call (what a row pitch is asked for without: any)
bool make_plan(int rows, int D, int sweep, long long keys, Plan* out) {
    const Combo* cs; int n;
    if (D <= 128 && rows > 224 && rows <= 256 && keys <= kNarrowTileKeys) {
        *out = Plan{1, 8, 256, 32 * AUDIOKV_SCORE_KB, 1};      // nine waves of 128 registers: one workgroup per CU
        return D == 64 || D == 128;
    }
    if (D == 64 || D == 128) { cs = sweep == 1 ? kSweep1_128 : kSweep2_128; n = sweep == 1 ? 7 : 6; }
    else if (D == 256) { cs = kCombos256; n = 5; }
    else return false;
    for (int i = 0; i < n; ++i) {
        const int pad = cs[i].NB * 32 * cs[i].WR;
        if (pad >= rows) {
            // two when the waves are few or hold one row tile each (128 registers), or when the workgroup is four waves of two
            // row tiles without constants (168 registers: three waves per SIMD); one when eight waves take all the registers.
            // At d = 256, four waves and, in sweep 1, seven are resident twice but planned as if they were not: with a tile on its way
            // across barriers one stream of keys per CU is faster than two (128 rows, planned for one and for two: 28 x 8192 98 and
            // 110 us, 4 x 8192 22.2 and 28.4, 8 x 32768 105 and 128, ragged 8 of 2048-32768 41.4 and 49.0, 40 of 1000-4000 51.5 and 55.8).
            const bool two = (cs[i].NB == 1 && D <= 128) || cs[i].WR < 4 || (cs[i].NB == 2 && cs[i].WR == 4 && sweep == 1);
            *out = Plan{cs[i].NB, cs[i].WR, pad, (D == 256) ? 32 : 32 * AUDIOKV_SCORE_KB, two ? 2 : 1};
            return true;
        }
    }
    return false;
}

long long total_keys(int H_kv, int n_items, const int32_t* seqlens_host) {
    long long keys = 0;
    for (int i = 0; i < n_items; ++i) keys += (long long)seqlens_host[i] * H_kv;
    return keys;
}

// What a workgroup costs before its first and after its last tile (query fragments, filling the ring, the row
// statistics or constants), in tiles: about 200 keys' worth, fitted to measured launches.
int overhead_tiles(const Plan& p) { return p.tile_keys >= 64 ? 3 : 7; }

// Items of different lengths, as many ranges for every head, so that a head's ranges are as long as the head is (tiles of the head /
// number) and workgroups start as others end. The launch takes about the average load of a slot, plus part of the longest
// workgroup for the ones that start last, plus, when the last round of workgroups fills only part of the
// slots, that round's average workgroup for the slots left idle (all in twice the unit, to keep halves).
// cost: in quarter tiles.
int same_number_for_every_head(const Plan& p, int H_kv, int n_items, const int32_t* seqlens_host, int max_tiles, long long max_parts, long long* cost_out) {
    const int slots = 256 * p.per_cu, overhead = overhead_tiles(p);
    // (every number is tried with every length: quotients rounded up, in float64 and off the whole numbers, so that they are exact. 48
    // lengths took 25 us with integer divisions. Items of as many tiles are counted together where there are more items than such
    // lengths: 281 items of 8 or 9 tiles, score with the log-sum-exp 23.6 and 17.9 us, which the host decides. The arrays have a fixed size: a
    // container could throw, and callers are C.)
    constexpr int kKept = 256;
    double kept[kKept], times[kKept];
    const int tile_shift = __builtin_ctz((unsigned)p.tile_keys);
    const auto tiles = [&](int i) { return (seqlens_host[i] + p.tile_keys - 1) >> tile_shift; };
    const bool counted = max_tiles < kKept && max_tiles < n_items;
    int entries = 0;
    if (counted) {
        int count[kKept] = {};
        for (int i = 0; i < n_items; ++i) ++count[tiles(i)];
        for (int t = 1; t <= max_tiles; ++t)
            if (count[t]) { kept[entries] = t; times[entries++] = count[t]; }
    } else {
        for (int i = 0; i < n_items && i < kKept; ++i) { kept[i] = tiles(i); times[i] = 1.; }
        entries = n_items;
    }
    int best = 1;
    long long best_cost = -1;
    const int ns_max = max_tiles < 64 ? max_tiles : 64;
    for (int ns = 1; ns <= ns_max; ++ns) {
        const long long groups = (long long)n_items * H_kv * ns;   // launched, whether or not they hold tiles
        if (ns > 1 && groups > max_parts) break;
        double sum = 0., most = 0.;
        const double per_range = 1. / ns;
        for (int i = 0; i < entries; ++i) {
            const double t = i < kKept ? kept[i] : tiles(i), n = i < kKept ? times[i] : 1.;
            const double tps = (double)(int)((t + ns - 0.5) * per_range);
            const double used = (double)(int)((t + tps - 0.5) / tps);       // ranges of this head that hold tiles
            sum += n * (t + used * overhead);
            most = tps > most ? tps : most;
        }
        const long long total = (long long)sum * H_kv, load = 2 * ((total + slots - 1) / slots);
        long long cost = load + (long long)most + overhead;
        const long long rem = groups % slots;
        if (groups > slots && rem) cost += 2 * (total / groups) * (slots - rem) / slots;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = ns; }
        // (the load never falls as the number grows)
        else if (load + 1 + overhead >= best_cost) break;
    }
    *cost_out = 2 * best_cost;
    return best;
}

// Which of the two divisions items of different lengths get. Ranges of one size need an item for each lane of a wave and a K that fits the
// memory-side cache (a larger one is streamed faster by ranges that each stay with their head, read backwards by sweep 2). Up to
// 128 heads they are the rule (but for nearly equal lengths); with more, the loads of the XCDs even out by themselves, as many ranges for every head keep a head's queries in
// one L2, and the other division has to promise a fifth less. Score calls, ranges of one size over as many for every head, geometric
// mean and worst: of 803 calls of up to 64 heads 0.92 and 1.15, of 78 of 65 to 128 0.91 and 1.13, of 23 of more that promise it 0.90 and 1.08,
// of 136 that do not 1.04 and 1.34; of 160 of a larger K 1.03 and 1.30. At the lines, as many for every head and ranges of one size: 246 x
// 385-770 tokens of four heads, 256 rows 142 and 172 us, 41 x 212-3402, 128 rows 41 and 34; 32 rows 9 x 23902-24381 (213 MB) 80 and 73,
// 14 x 21207-23328 (321 MB) 106 and 120, 64 rows of eight heads 7 x 11247-22494 (266 MB) 95 and 88, 8 x 24149-26564 (410 MB) 147 and 163.
constexpr int kSizedHeads = 128;
constexpr long long kCacheBytes = 1LL << 28;
enum class Division { same_number, one_size, cheaper };
Division division(int H_kv, int n_items, const int32_t* seqlens_host, int D) {
    long long tokens = 0, longest = 0;
    for (int i = 0; i < n_items; ++i) { tokens += seqlens_host[i]; longest = seqlens_host[i] > longest ? seqlens_host[i] : longest; }
    if (n_items > kCountedItems || tokens * H_kv * D * 2 > kCacheBytes) return Division::same_number;
    // (more than 64 heads of nearly one length leave the XCDs nothing to even out: 64 x 578-636 tokens of two heads, 128 rows 20.8 and
    // 25.9 us, 32 x 832-874 of four 22.7 and 25.8)
    if (n_items * H_kv > 64 && 5 * longest * n_items < 6 * tokens) return Division::same_number;
    return n_items * H_kv <= kSizedHeads ? Division::one_size : Division::cheaper;
}

// max_parts: not more than these where one range for every head is not more than that already.
ScoreRanges plan_ranges(const Plan& p, int H_kv, int n_items, const int32_t* seqlens_host, Division division, long long max_parts = LLONG_MAX) {
    // The heads are cut into key ranges so that the grid fills the 256 CUs evenly: the division minimises the time of
    // the launch in units of a quarter tile, with a fixed prologue cost per workgroup, in whole rounds of workgroups.
    const int overhead = overhead_tiles(p);
    int longest = 1;
    bool uniform = true;             // as many ranges for every head
    for (int i = 0; i < n_items; ++i) {
        if (seqlens_host[i] > longest) longest = seqlens_host[i];
        if (seqlens_host[i] != seqlens_host[0]) uniform = false;
    }
    const int max_tiles = (longest + p.tile_keys - 1) / p.tile_keys;
    // (lengths differ, but a workgroup for every tile of every head, were all as long as the longest, fits the chip at once: to find
    // its item would cost each of them 0.2 us. The same answer for every sweep of a call, whatever its tiling.)
    if (!uniform && max_tiles <= 64 && (long long)n_items * H_kv * max_tiles <= 256) uniform = true;
    ScoreRanges same;
    long long same_cost = 0;
    if (!uniform && division != Division::one_size) {
        same.per_head = same_number_for_every_head(p, H_kv, n_items, seqlens_host, max_tiles, max_parts, &same_cost);
        same.parts = (long long)n_items * H_kv * same.per_head;
        if (division == Division::same_number) return same;
    }
    // One and two compute waves at d <= 128: three workgroups share a CU, which ranges of one size put to use from a tile for each of two on
    // (24 x 5929-6048 tokens, 64 rows at d = 64 with the log-sum-exp at hand 14.5 and 13.1 us, 7 x 12763-14040 of eight heads 67.8
    // and 65.1, planned for two and for three; below that up to 3 % slower).
    long long tokens = 0;
    for (int i = 0; i < n_items; ++i) tokens += seqlens_host[i];
    const int slots = 256 * (!uniform && p.WR < 4 && p.tile_keys >= 64 && tokens * H_kv >= 512LL * p.tile_keys ? 3 : p.per_cu);
    ScoreRanges best;
    long long best_cost = -1;
    const int ns_max = max_tiles < 64 ? max_tiles : 64;
    for (int ns = 1; ns <= ns_max; ++ns) {                  // ranges of a head of the longest item
        const int tiles = (max_tiles + ns - 1) / ns;
        ScoreRanges r;
        r.per_head = ns;
        long long groups = (long long)n_items * ns;         // per KV head, empty ones included
        if (!uniform) {
            r.keys = tiles * p.tile_keys;
            r.per_key = 1. / r.keys;
            groups = 0;
            for (int i = 0; i < n_items; ++i) groups += r.of_length(seqlens_host[i]);
        }
        r.parts = groups * H_kv;
        if (ns > 1 && r.parts > max_parts) continue;
        const long long rounds = (r.parts + slots - 1) / slots;
        // Seven compute waves with a CU to themselves are faster than two sevens that share it (ranges of one size, 224 rows: 8 x 3607-3968
        // tokens of one head in 473 ranges 20.0 us, as this plans them 16.4; 12 x 2351-2587 20.0 and 16.4; 6 x 7092-7802 22.8 and 18.9).
        // Of one to four waves this is not so (32 rows 10 x 586-616 12.2 and 13.5).
        const int quarters = !uniform && p.WR == 7 && p.per_cu == 2 && r.parts <= 256 ? 3 : 4;
        const long long cost = quarters * rounds * (tiles + overhead);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = r; }
    }
    if (!uniform && division == Division::cheaper && 5 * best_cost >= 4 * same_cost) return same;
    return best;
}

}  // namespace

// Sweep 2 cannot hold more than 448 rows without spilling (its row constants come on top of the accumulators), so
// more rows are covered by two launches: the first 448 with the widest tiling, the rest with the smallest that fits;
// the second writes its column sums to a buffer of its own, added to the first afterwards.
constexpr int kSweep2MaxRows = 448;

bool sweep2_is_split(int rows, int D) { return D <= 128 && rows > kSweep2MaxRows; }

int score_padded_rows(int rows, int D) {
    Plan p1, p2;
    if (!make_plan(rows, D, 1, 0, &p1)) return 0;
    if (sweep2_is_split(rows, D)) {
        if (!make_plan(rows - kSweep2MaxRows, D, 2, 0, &p2)) return 0;
        const int pad2 = kSweep2MaxRows + p2.rows_pad;
        return p1.rows_pad > pad2 ? p1.rows_pad : pad2;
    }
    if (!make_plan(rows, D, 2, 0, &p2)) return 0;
    return p1.rows_pad > p2.rows_pad ? p1.rows_pad : p2.rows_pad;
}

bool score_needs_second_raw(int rows, int D) { return sweep2_is_split(rows, D); }

// what sizes the statistics in the workspace
ScoreRanges score_ranges(int H_kv, int n_items, const int32_t* seqlens_host, int rows, int D, long long max_parts) {
    Plan p;
    if (n_items <= 0 || H_kv <= 0 || !make_plan(rows, D, 1, total_keys(H_kv, n_items, seqlens_host), &p)) {
        ScoreRanges none;
        none.parts = (long long)n_items * H_kv;
        return none;
    }
    return plan_ranges(p, H_kv, n_items, seqlens_host, division(H_kv, n_items, seqlens_host, D), max_parts);
}

hipError_t launch_score(const Geom& g, const void* q_win, const void* k, const int32_t* cu_seqlens,
                        const int32_t* seqlens_host, const ScoreRanges& ranges1, float* stats_ws, float* raw_out, hipStream_t s, hipEvent_t between_sweeps,
                        const float* lse, float* raw_second, size_t raw_elems, const AllocateJob* ride_along,
                        const ConvFilterJob* ride_taps)
{
    Plan p1;
    const int rows = g.G * g.W;
    const long long keys = total_keys(g.H_kv, g.n_items, seqlens_host);
    if (!make_plan(rows, g.D, 1, keys, &p1)) return hipErrorInvalidValue;
    const int rows_pad = score_padded_rows(rows, g.D);
    if (rows_pad == 0) return hipErrorInvalidValue;
    // What the memory-side cache (256 MB) holds of K after sweep 1 is its end: where K does not fit, sweep 2 begins there. Score
    // calls, forwards and backwards: 28 x 32768, 448 rows 929 and 915 us, 13 x 32768 452 and 442; 224 rows 30 x 9000 (276 MB) 169 and 165,
    // 48 x 10000 297 and 289; K that fits: 28 x 9000, 256 rows (258 MB) 352 and 356 with the eviction around it.
    const bool backwards = keys * g.D * 2 > kCacheBytes;
    const Division div = ranges1.keys ? Division::one_size : Division::same_number;    // (sweep 2 finds the statistics by that of sweep 1)
    score_detail::SweepArgs args{q_win, k, cu_seqlens, ranges1, rows_pad, 0, stats_ws, ranges1, lse, raw_out, backwards, ride_along, ride_taps};
    auto sweep = [&](int which, const Plan& p, const ScoreRanges& ranges, int row_base, float* raw) -> hipError_t {
        args.ranges = ranges;
        args.row_base = row_base;
        args.raw = raw;
        hipError_t e = hipErrorInvalidValue;
        switch (g.D) {
            case 64:  e = launch_score_d64(which, g, p.NB, p.WR, args, s); break;
            case 128: e = launch_score_d128(which, g, p.NB, p.WR, args, s); break;
            case 256: e = launch_score_d256(which, g, p.NB, p.WR, args, s); break;
        }
        args.alloc = nullptr;                       // they have gone along
        args.taps = nullptr;
        return e;
    };
    hipError_t e = lse ? hipSuccess : sweep(1, p1, ranges1, 0, raw_out);
    if (e != hipSuccess) return e;
    if (between_sweeps) {
        e = hipEventRecord(between_sweeps, s);
        if (e != hipSuccess) return e;
    }
    Plan p2;
    if (!sweep2_is_split(rows, g.D)) {
        if (!make_plan(rows, g.D, 2, keys, &p2)) return hipErrorInvalidValue;
        return sweep(2, p2, plan_ranges(p2, g.H_kv, g.n_items, seqlens_host, div), 0, raw_out);
    }
    if (!raw_second) return hipErrorInvalidValue;
    Plan p2b;
    if (!make_plan(kSweep2MaxRows, g.D, 2, keys, &p2) || !make_plan(rows - kSweep2MaxRows, g.D, 2, keys, &p2b)) return hipErrorInvalidValue;
    e = sweep(2, p2, plan_ranges(p2, g.H_kv, g.n_items, seqlens_host, div), 0, raw_out);
    if (e != hipSuccess) return e;
    e = sweep(2, p2b, plan_ranges(p2b, g.H_kv, g.n_items, seqlens_host, div), kSweep2MaxRows, raw_second);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((raw_elems + 256 * 8 - 1) / (256 * 8));
    hipLaunchKernelGGL(score_detail::score_add_kernel, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, s, raw_out,
                       (const float*)raw_second, raw_elems);
    return hipGetLastError();
}

}  // namespace audiokv
