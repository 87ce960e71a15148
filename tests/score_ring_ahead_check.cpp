// The ring through which the loader wave of the score kernels hands tiles of keys to the compute waves, run on the host with
// loads that complete as late as the loader's waits allow: every tile that an iteration reads has landed when the iteration
// opens, and no request goes into a slot that may still be read: the order that leaves the newest tile on its way across a barrier.
// Built and run by tests/test_score_ragged_code.py.
#include <cstdio>
#include <vector>

#include "score_ring.h"

using namespace audiokv::score_detail;

static int failures;

// in_flight: tiles that barrier(true) leaves outstanding; last: tiles that barrier(false) does
template <int STAGES>
static int violations(int n_tiles, int in_flight, int last) {
    std::vector<int> holds(STAGES, -1);              // tile last requested into a slot
    std::vector<bool> landed(n_tiles + 8, false);
    int requested = 0, bad = 0, open = -1;           // the iteration that is running
    fill_ring_ahead<STAGES>(n_tiles,
        [&](int t) {
            bad += t != requested++ || t >= n_tiles;
            // tiles open and open + 1 are being read
            const int old = holds[t % STAGES];
            bad += open >= 0 && (old == open || old == open + 1);
            holds[t % STAGES] = t;
        },
        [&](bool newest_may_fly) {
            for (int t = 0; t < requested - (newest_may_fly ? in_flight : last); ++t) landed[t] = true;
            ++open;
            for (int t = open; t <= open + 1 && t < n_tiles; ++t) bad += !landed[t] || holds[t % STAGES] != t;
        });
    bad += requested != n_tiles || open != n_tiles;  // a barrier in front and one for every tile, as the compute waves have
    return bad;
}

template <int STAGES>
static void check() {
    int caught = 0, caught_last = 0;
    for (int n = 1; n <= 40; ++n) {
        const int bad = violations<STAGES>(n, kLeftInFlight<STAGES>, 0);
        if (bad) { ++failures; std::printf("%d slots, %d tiles: %d violations\n", STAGES, n, bad); }
        // waits that are one tile short
        caught += violations<STAGES>(n, kLeftInFlight<STAGES> + 1, 0) > 0;
        caught_last += violations<STAGES>(n, kLeftInFlight<STAGES>, 1) > 0;
    }
    if (caught < 38 || caught_last < 40) { ++failures; std::printf("%d slots: a wait that is one tile short goes unnoticed\n", STAGES); }
}

int main() {
    check<4>();
    if (!failures) std::printf("the ring holds\n");
    return failures ? 1 : 0;
}
