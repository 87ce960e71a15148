// When the loader wave of a score workgroup requests a tile of keys, and what has landed at each barrier. A header of its own
// because the order is checked on the host as well (tests/score_ring_check.cpp).
#pragma once

#include <hip/hip_runtime.h>

namespace audiokv {
namespace score_detail {

// Iteration t of the compute waves lies between the barrier that ended tile t - 1 (for the first tile the one in front of the
// loop) and the one that ends tile t. In it they reduce tile t and already multiply the first block of the next one, so at the
// barrier that opens iteration t the tiles up to t + kLookAhead have to have landed.
constexpr int kLookAhead = 1;
// Tiles that may still be on their way when the loader enters a barrier.
constexpr int kInFlight = 0;

// STAGES slots, tile t in slot t % STAGES. issue(t) requests tile t, barrier() waits until at most kInFlight tiles' requests
// are outstanding (they complete in the order in which they were issued) and enters the workgroup's barrier.
template <int STAGES, class Issue, class Barrier>
__host__ __device__ __forceinline__ void fill_ring(int n_tiles, Issue issue, Barrier barrier) {
    constexpr int AHEAD = STAGES - 1;
    // At the barrier that ends tile t, tiles up to t + AHEAD are requested and t + 1 is opened.
    static_assert(AHEAD - kInFlight >= 1 + kLookAhead, "what an iteration reads has landed when it opens");
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (a < n_tiles) issue(a);
    barrier();                                      // opens iteration 0
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
        // its slot held tile t - 1, which every wave left at the barrier that ended it
        if (t + AHEAD < n_tiles) issue(t + AHEAD);
        barrier();                                  // ends tile t
    }
}

// The same with the newest tiles on their way across a barrier: barrier(true) may leave those that the iteration it opens does not
// read, STAGES - 2 - kLookAhead, barrier(false) none (the last tiles: what is outstanding is read next).
template <int STAGES>
constexpr int kLeftInFlight = STAGES - 2 - kLookAhead;
template <int STAGES, class Issue, class Barrier>
__host__ __device__ __forceinline__ void fill_ring_ahead(int n_tiles, Issue issue, Barrier barrier) {
    constexpr int AHEAD = STAGES - 1;
    static_assert(kLeftInFlight<STAGES> == 1, "a barrier that opens an iteration finds all its tiles or one more requested");
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (a < n_tiles) issue(a);
    barrier(AHEAD - 1 < n_tiles);                   // opens iteration 0
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
        if (t + AHEAD < n_tiles) issue(t + AHEAD);
        barrier(t + AHEAD < n_tiles);               // ends tile t
    }
}

}  // namespace score_detail
}  // namespace audiokv
