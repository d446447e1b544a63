// Checks the projectors' launch order on the CPU: every (projection, tile)
// pair taken by exactly one workgroup, with bounded padding, and no launch
// beyond 2^32 threads that the pairs alone would fit.  Ends with 1 and a
// message at the first failure.
#include <cstdio>
#include <vector>

#include "launch_order.h"

using namespace ctrex;

static int check(long long tiles, int n_views, bool walk) {
    const LaunchOrder o = launch_order(tiles, n_views);
    const long long total = tiles * n_views;
    if (o.grp < 1 || o.run < 1 || o.run > tiles || o.blocks < total || o.blocks % N_XCD)
        return std::printf("%lld x %d: order %d %d %lld\n", tiles, n_views, o.grp, o.run, o.blocks);
    if (total <= MAX_PROJ_BLOCKS - N_XCD && o.blocks > MAX_PROJ_BLOCKS)
        return std::printf("%lld x %d: %lld workgroups\n", tiles, n_views, o.blocks);
    // runs and groups are evened out to under twice their items, and units
    // (at most 1 / 112 of the pairs each where they hold several) fill whole XCDs
    if (o.blocks > 2 * total + total / 8 + N_XCD * o.grp * o.run)
        return std::printf("%lld x %d: %lld workgroups for %lld pairs\n", tiles, n_views, o.blocks, total);
    if (!walk) return 0;
    std::vector<char> seen(total, 0);
    long long n = 0;
    for (long long b = 0; b < o.blocks; ++b) {
        const Pair q = pair_of(static_cast<int>(b), o.grp, o.run, static_cast<int>(tiles), n_views);
        if (!q.valid) continue;
        if (q.k < 0 || q.k >= n_views || q.tile < 0 || q.tile >= tiles || seen[q.k * tiles + q.tile]++)
            return std::printf("%lld x %d: workgroup %lld takes (%d, %d)\n", tiles, n_views, b, q.k, q.tile);
        ++n;
    }
    return n == total ? 0 : std::printf("%lld x %d: %lld of %lld pairs\n", tiles, n_views, n, total);
}

int main() {
    const long long tiles[] = {1, 2, 3, 4, 9, 15, 16, 31, 32, 33, 63, 64, 65, 120, 576, 2304};
    const int views[] = {1, 2, 7, 8, 15, 16, 17, 31, 33, 60, 100, 255, 720, 1200, 5000, 65536};
    for (long long t : tiles)
        for (int v : views)
            if (check(t, v, t * v <= 2000000)) return 1;
    // long lists of small images, up to the most that a launch holds
    for (long long t : tiles)
        for (long long v = 1 << 17; t * v < (1ll << 25); v += v / 3)
            if (check(t, static_cast<int>(v), false)) return 1;
    std::puts("ok");
    return 0;
}
