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
            // At d = 256, four waves and, in sweep 1, seven are resident twice but planned as if they were not: planned with two, 128
            // rows 28 x 8192 take 113.5 us instead of 125.4, but 4 x 8192 29.7 instead of 24.0 and 8 of 2048-32768 56.7 instead of 55.3.
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

int num_splits(const Plan& p, int H_kv, int n_items, const int32_t* seqlens_host) {
    // A head is cut into key ranges so that the grid fills the 256 CUs evenly: the split count minimises the time of
    // the launch in units of one tile, with a fixed prologue cost per workgroup (in tiles).
    const int slots = 256 * p.per_cu;
    // what a workgroup costs before its first and after its last tile (query fragments, filling the ring, the row
    // statistics or constants), in tiles: about 200 keys' worth, fitted to measured launches
    const int overhead = p.tile_keys >= 64 ? 3 : 7;
    int max_tiles = 1;
    bool uniform = true;
    for (int i = 0; i < n_items; ++i) {
        const int t = (seqlens_host[i] + p.tile_keys - 1) / p.tile_keys;
        if (t > max_tiles) max_tiles = t;
        if (seqlens_host[i] != seqlens_host[0]) uniform = false;
    }
    // (for ragged batches, in which every count is tried with every length: quotients rounded up, in float64 and off the whole
    // numbers, so that they are exact. 48 lengths took 25 us with integer divisions. The first lengths' tiles are kept in an array
    // of fixed size: a container could throw, and callers are C.)
    constexpr int kKept = 256;
    double kept[kKept];
    const int tile_shift = __builtin_ctz((unsigned)p.tile_keys);
    const auto tiles = [&](int i) { return (double)((seqlens_host[i] + p.tile_keys - 1) >> tile_shift); };
    if (!uniform)
        for (int i = 0; i < n_items && i < kKept; ++i) kept[i] = tiles(i);
    int best = 1;
    long long best_cost = -1;
    const int ns_max = max_tiles < 64 ? max_tiles : 64;
    for (int ns = 1; ns <= ns_max; ++ns) {
        long long cost;
        if (uniform) {
            // equal workgroups run in whole rounds
            const long long groups = (long long)n_items * H_kv * ns;
            const long long rounds = (groups + slots - 1) / slots;
            cost = rounds * ((max_tiles + ns - 1) / ns + overhead);
        } else {
            // Ragged lengths: a head's ranges are as long as the head is (tiles of the head / ns), and workgroups
            // start as others end. The launch takes about the average load of a slot, plus part of the longest
            // workgroup for the ones that start last, plus, when the last round of workgroups fills only part of the
            // slots, that round's average workgroup for the slots left idle (all in twice the unit, to keep halves).
            const long long groups = (long long)n_items * H_kv * ns;   // launched, whether or not they hold tiles
            double sum = 0., most = 0.;
            const double per_range = 1. / ns;
            for (int i = 0; i < n_items; ++i) {
                const double t = i < kKept ? kept[i] : tiles(i);
                if (!(t > 0.)) continue;
                const double tps = (double)(int)((t + ns - 0.5) * per_range);
                const double used = (double)(int)((t + tps - 0.5) / tps);       // ranges of this head that hold tiles
                sum += t + used * overhead;
                most = tps > most ? tps : most;
            }
            const long long total = (long long)sum * H_kv, longest = most > 0. ? (long long)most + overhead : 0;
            cost = 2 * ((total + slots - 1) / slots) + longest;
            const long long rem = groups % slots;
            if (groups > slots && rem) cost += 2 * (total / groups) * (slots - rem) / slots;
        }
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = ns; }
    }
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

// key ranges per head of sweep 1: what sizes the statistics in the workspace
int score_num_splits(int H_kv, int n_items, const int32_t* seqlens_host, int rows, int D) {
    Plan p;
    if (n_items <= 0 || H_kv <= 0 || !make_plan(rows, D, 1, total_keys(H_kv, n_items, seqlens_host), &p)) return 1;
    return num_splits(p, H_kv, n_items, seqlens_host);
}

hipError_t launch_score(const Geom& g, const void* q_win, const void* k, const int32_t* cu_seqlens,
                        const int32_t* seqlens_host, int ns1, float* stats_ws, float* raw_out, hipStream_t s, hipEvent_t between_sweeps,
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
    const bool backwards = keys * g.D * 2 > (1LL << 28);
    score_detail::SweepArgs args{q_win, k, cu_seqlens, 0, rows_pad, 0, stats_ws, ns1, lse, raw_out, backwards, ride_along, ride_taps};
    auto sweep = [&](int which, const Plan& p, int ns, int row_base, float* raw) -> hipError_t {
        args.nsplit = ns;
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
    hipError_t e = lse ? hipSuccess : sweep(1, p1, ns1, 0, raw_out);
    if (e != hipSuccess) return e;
    if (between_sweeps) {
        e = hipEventRecord(between_sweeps, s);
        if (e != hipSuccess) return e;
    }
    Plan p2;
    if (!sweep2_is_split(rows, g.D)) {
        if (!make_plan(rows, g.D, 2, keys, &p2)) return hipErrorInvalidValue;
        return sweep(2, p2, num_splits(p2, g.H_kv, g.n_items, seqlens_host), 0, raw_out);
    }
    if (!raw_second) return hipErrorInvalidValue;
    Plan p2b;
    if (!make_plan(kSweep2MaxRows, g.D, 2, keys, &p2) || !make_plan(rows - kSweep2MaxRows, g.D, 2, keys, &p2b)) return hipErrorInvalidValue;
    e = sweep(2, p2, num_splits(p2, g.H_kv, g.n_items, seqlens_host), 0, raw_out);
    if (e != hipSuccess) return e;
    e = sweep(2, p2b, num_splits(p2b, g.H_kv, g.n_items, seqlens_host), kSweep2MaxRows, raw_second);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((raw_elems + 256 * 8 - 1) / (256 * 8));
    hipLaunchKernelGGL(score_detail::score_add_kernel, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, s, raw_out,
                       (const float*)raw_second, raw_elems);
    return hipGetLastError();
}

}  // namespace audiokv
