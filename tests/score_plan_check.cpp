// How score divides items of different lengths into key ranges (audiokv::score_ranges of the built library): which division a batch
// gets, that ranges of one size cover every item, and that as many ranges for every head are the number that trying them all gives.
// Built and run by tests/test_score_plan.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "common.h"

using namespace audiokv;

struct Tiling { int rows, D, tile, per_cu; };

// every number tried, in whole numbers; cost in half tiles
static int number_for_every_head(const Tiling& t, int H, const std::vector<int>& lens, long long* cost_out) {
    const long long slots = 256LL * t.per_cu, overhead = t.tile >= 64 ? 3 : 7, n = (long long)lens.size();
    int max_tiles = 1, best = 1;
    for (int L : lens) max_tiles = std::max(max_tiles, (L + t.tile - 1) / t.tile);
    long long best_cost = -1;
    for (int ns = 1; ns <= std::min(max_tiles, 64); ++ns) {
        long long sum = 0, most = 0;
        for (int L : lens) {
            const long long tiles = (L + t.tile - 1) / t.tile, tps = (tiles + ns - 1) / ns;
            sum += tiles + (tiles + tps - 1) / tps * overhead;
            most = std::max(most, tps);
        }
        const long long groups = n * H * ns, total = sum * H, rem = groups % slots;
        long long cost = 2 * ((total + slots - 1) / slots) + most + overhead;
        if (groups > slots && rem) cost += 2 * (total / groups) * (slots - rem) / slots;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = ns; }
    }
    *cost_out = best_cost;
    return best;
}

int main() {
    std::mt19937 rng(7);
    const auto spread = [&](double lo, double hi) { return (int)std::lround(std::exp(std::uniform_real_distribution<>(std::log(lo), std::log(hi))(rng))); };
    int sized = 0, same = 0, small = 0, both = 0, bad = 0;
    for (int round = 0; round < 6000; ++round) {
        const int D = std::vector<int>{64, 128, 256}[rng() % 3], H = std::vector<int>{1, 2, 4, 8}[rng() % 4];
        const int n = spread(2, round % 3 ? 64 : 400), top = spread(64, 40000), low = std::max(1, top / (int)(1 + rng() % 16) - 1);
        std::vector<int> lens;
        long long keys = 0;
        for (int i = 0; i < n; ++i) { lens.push_back(spread(low, top)); keys += (long long)lens.back() * H; }
        if (std::count(lens.begin(), lens.end(), lens[0]) == n) continue;
        std::vector<Tiling> tilings;
        for (int rows : {1, 32, 64, 128, 224}) tilings.push_back({rows, D, D == 256 ? 32 : 64, D == 256 ? (rows <= 64 ? 2 : 1) : 2});
        if (D == 256) tilings.push_back({256, D, 32, 1});
        else { tilings.push_back({256, D, 64, keys <= 3 << 17 ? 1 : 2}); tilings.push_back({448, D, 64, 1}); tilings.push_back({576, D, 64, 1}); }
        const Tiling t = tilings[rng() % tilings.size()];
        const ScoreRanges r = score_ranges(H, n, lens.data(), t.rows, D);
        const long long tiles = (*std::max_element(lens.begin(), lens.end()) + t.tile - 1) / t.tile;
        bool good = true;
        long long cost = 0, parts = 0;
        const int number = number_for_every_head(t, H, lens, &cost);
        const bool even = n * H > 64 && 5.0 * *std::max_element(lens.begin(), lens.end()) * n * H < 6.0 * keys;
        const bool fits = n <= 64 && keys * D * 2 <= 1 << 28 && !even;
        if (tiles <= 64 && n * H * tiles <= 256) {
            ++small;
            good = r.keys == 0 && r.parts == (long long)n * H * r.per_head;
        } else if (r.keys) {
            ++(n * H <= 128 ? sized : both);
            good = fits && r.keys % t.tile == 0;
            for (int L : lens) { parts += (long long)((L + r.keys - 1) / r.keys) * H; good &= r.of_length(L) == (L + r.keys - 1) / r.keys; }
            good &= r.parts == parts;
            // in whole rounds at a fifth less, where the other division is to be had
            const long long slots = 256LL * (t.rows <= 64 && D <= 128 && keys >= 512 * 64 ? 3 : t.per_cu), full = ((parts + slots - 1) / slots) * (r.keys / t.tile + (t.tile >= 64 ? 3 : 7));
            if (n * H > 128) good &= 5 * (parts <= 256 && t.rows == 224 && D <= 128 ? 3 : 4) * full < 4 * 2 * cost;
        } else {
            ++same;
            good = !(fits && n * H <= 128) && r.per_head == number && r.parts == (long long)n * H * r.per_head;
        }
        if (!good && ++bad <= 10)
            std::printf("%d items of up to %lld tiles, %d heads, %d rows, D %d, %lld keys: %d ranges per head, %d keys each, %lld parts\n", n, tiles,
                        H, t.rows, D, keys, r.per_head, r.keys, r.parts);
    }
    std::printf("%s: %d of one size, %d at a fifth less, %d as many for every head, %d small\n",
                !bad && sized > 500 && both > 50 && same > 500 && small > 200 ? "the ranges are as planned" : "not as planned", sized, both, same, small);
    return bad ? 1 : 0;
}
