// Workgroups that ride along in another launch, against what a launch holds: fewer than 2^32 threads, half of them for riders.
// Compiled for the host; built and run by tests/test_launch_size.py.
#include <cstdio>

#include "conv_filter.h"

using namespace audiokv;

int main() {
    int bad = 0;
    for (int threads : {64, 128, 192, 256, 320, 448, 512, 576})
        for (long long n = 1; n <= 1 << 20; n = n < 16 ? n + 1 : n + n / 7)
            for (int L : {1, 500, 4000, 16383, 131071}) {
                ConvFilterJob job{};
                job.n_items = (int)n;
                job.max_length = L;
                const long long per = job.blocks_per_item(threads);
                // every tap and its mirror image have a thread, or the launch is as full as it may be
                const bool all = per * threads > L / 2;
                if (per < 1 || (!all && (per + 1) * n * threads <= 1LL << 31) || (per > 1 && per * n * threads > 1LL << 31)) {
                    ++bad;
                    std::printf("%d threads, %lld items of %d: %lld workgroups each\n", threads, n, L, per);
                }
            }
    if (!bad) std::printf("launches hold their riders\n");
    return bad ? 1 : 0;
}
