// Checks the launch orders on the CPU: every (projection, tile) pair and every
// (brick, chunk) item taken by exactly one workgroup, with bounded padding, no
// launch beyond 2^32 threads that the work alone would fit, and no XCD with
// much more than the others.  Ends with 1 and a message at the first failure.
#include <climits>
#include <cstdio>
#include <vector>

#include "launch_order.h"

using namespace ctrex;

static int check(int row, int rows, int n_views, bool walk, bool narrow = false, int group = 0) {
    const LaunchOrder o = launch_order(row, rows, n_views, narrow, group);
    const long long tiles = 1ll * row * rows, total = tiles * n_views;
    if (o.grp < 1 || o.run < 1 || o.run > tiles || o.blocks < total || o.blocks % N_XCD)
        return std::printf("%lld x %d: order %d %d %lld\n", tiles, n_views, o.grp, o.run, o.blocks);
    if (total <= MAX_PROJ_BLOCKS - N_XCD && o.blocks > MAX_PROJ_BLOCKS)
        return std::printf("%lld x %d: %lld workgroups\n", tiles, n_views, o.blocks);
    // runs and groups are evened out to under twice their items, and units
    // fill whole XCDs
    if (o.blocks > 2 * total + total / 8 + N_XCD * o.grp * o.run)
        return std::printf("%lld x %d: %lld workgroups for %lld pairs\n", tiles, n_views, o.blocks, total);
    if (!walk) return 0;
    std::vector<char> seen(total, 0);
    long long n = 0;
    for (long long b = 0; b < o.blocks; ++b) {
        const Pair q = pair_of(static_cast<unsigned>(b), o.grp, o.run, o.runs, o.turn,
                               static_cast<int>(tiles), n_views);
        if (!q.valid) continue;
        if (q.k < 0 || q.k >= n_views || q.tile < 0 || q.tile >= tiles || seen[q.k * tiles + q.tile]++)
            return std::printf("%lld x %d: workgroup %lld takes (%d, %d)\n", tiles, n_views, b, q.k, q.tile);
        ++n;
    }
    return n == total ? 0 : std::printf("%lld x %d: %lld of %lld pairs\n", tiles, n_views, n, total);
}

// Work per XCD of an n x n detector whose middle columns (two of them, narrow,
// or half) have all of it, without its first and last rows: less than twice the
// mean, or twice the mean if narrow (small launches have 24 to 32 units, of which
// each XCD takes whole ones; units at fixed distances put all work on two or
// three XCDs, or on half of them).
static int balance(int n, int n_views, bool narrow, bool cyl) {
    const LaunchOrder o = launch_order(n, n, n_views, narrow, 0, cyl);
    const int half = narrow ? 1 : n / 4;
    long long busy[N_XCD] = {}, all = 0, most = 0;
    for (long long b = 0; b < o.blocks; ++b) {
        const Pair q = pair_of(static_cast<unsigned>(b), o.grp, o.run, o.runs, o.turn, n * n, n_views);
        const int u = q.tile % n, v = q.tile / n;
        if (q.valid && u >= n / 2 - half && u < n / 2 + half && v > 1 && v < n - 2)
            ++busy[b % N_XCD], ++all;
    }
    for (long long x : busy) most = x > most ? x : most;
    return N_XCD * most > (narrow ? 2 * all : 2 * all - 1) ? std::printf("%d^2 x %d: %lld of %lld\n", n, n_views, most, all) : 0;
}

// The backprojector's items: each taken once, and no XCD with more than a unit
// above the mean.
static int bricks(int rows, int per_row, int chunks) {
    const BrickOrder o = brick_order(rows, per_row, chunks);
    const long long total = 1ll * rows * per_row * chunks;
    if (o.run < 1 || o.blocks < total || o.blocks % N_XCD || o.blocks > total + N_XCD * o.run)
        return std::printf("bricks %d x %d x %d: %d %lld\n", rows, per_row, chunks, o.run, o.blocks);
    std::vector<char> seen(total, 0);
    long long busy[N_XCD] = {}, n = 0, most = 0;
    for (long long b = 0; b < o.blocks; ++b) {
        const unsigned i = item_of(static_cast<unsigned>(b), o.run, o.turn);
        if (i >= total) continue;
        if (seen[i]++) return std::printf("bricks %d x %d x %d: item %u twice\n", rows, per_row, chunks, i);
        ++n, ++busy[b % N_XCD];
    }
    for (long long x : busy) most = x > most ? x : most;
    if (n != total || (most - o.run) * N_XCD > total)
        return std::printf("bricks %d x %d x %d: %lld taken, %lld on one XCD\n", rows, per_row, chunks, n, most);
    // an XCD takes whole units: an eighth more than the mean from 64 units on
    if (total >= 64 && 8 * N_XCD * most > 9 * total + 8 * N_XCD)
        return std::printf("bricks %d x %d x %d: %lld on one XCD\n", rows, per_row, chunks, most);
    return 0;
}

int main() {
    for (int rows : {1, 2, 4, 7, 8, 9, 16, 25, 26, 49, 72, 100, 169, 256, 1024})
        for (int per_row : {1, 2, 3, 4, 8, 16})
            for (int chunks : {1, 2, 3, 8, 15, 25, 45, 250})
                if (bricks(rows, per_row, chunks)) return 1;
    const int sides[][2] = {{1, 1}, {2, 1}, {1, 3}, {2, 2}, {3, 3}, {15, 1}, {4, 4}, {31, 1}, {8, 4}, {33, 1},
                            {8, 8}, {5, 13}, {12, 10}, {16, 16}, {24, 24}, {48, 48}, {24, 2}, {1, 40}};
    const int views[] = {1, 2, 7, 8, 15, 16, 17, 31, 33, 60, 100, 255, 720, 1200, 5000, 65536};
    for (const auto &s : sides)
        for (int v : views) {
            const long long total = 1ll * s[0] * s[1] * v;
            if (check(s[0], s[1], v, total <= 2000000) || check(s[0], s[1], v, total <= 200000, true) ||
                check(s[0], s[1], v, total <= 200000, false, INT_MAX))
                return 1;
        }
    for (int n : {8, 12, 16, 24, 32, 40, 48})
        for (int v : {30, 75, 180, 720})
            if (balance(n, v, false, false) || balance(n, v, false, true) || (n > 8 && balance(n, v, true, false)))
                return 1;
    // long lists of small images, up to the most that a launch holds
    for (const auto &s : sides)
        for (long long v = 1 << 17; s[0] * s[1] * v < (1ll << 25); v += v / 3)
            if (check(s[0], s[1], static_cast<int>(v), false)) return 1;
    std::puts("ok");
    return 0;
}
