// Which work a workgroup takes: the order of the projectors' launches.
// Constant-expression functions without HIP types, shared by the host, which
// sizes the launch, and the kernels.
#pragma once

namespace ctrex {

constexpr int N_XCD = 8;
// A launch holds fewer than 2^32 threads: 2^24 workgroups of the projectors' 256.
constexpr long long MAX_PROJ_BLOCKS = (1ll << 24) - 1;

constexpr long long round_up_xcd(long long n) { return (n + N_XCD - 1) / N_XCD * N_XCD; }

// Units of the projectors' launch (pair_of): groups of grp projections x runs
// of run detector tiles, and the workgroups of whole units, a multiple of
// N_XCD.
struct LaunchOrder {
    int grp = 1, run = 1;
    long long blocks = 0;
};

// Groups of up to 16 projections, runs of up to 32 tiles, both evened out so
// that the last one is not mostly empty; runs shorter where there are too few
// pairs for 16 units per XCD.  Where the padding of whole units would exceed
// the threads of a launch, single pairs are handed out.
constexpr LaunchOrder launch_order(long long tiles, int n_views) {
    constexpr int kGroup = 16, kRun = 32, kUnits = 16 * N_XCD;
    LaunchOrder o;
    const long long total = tiles * n_views;
    o.blocks = round_up_xcd(total);
    if (total <= 0 || total > MAX_PROJ_BLOCKS) return o;
    const int groups = (n_views + kGroup - 1) / kGroup;
    const int grp = (n_views + groups - 1) / groups;
    long long run = total / (grp * kUnits);
    if (run > kRun) run = kRun;
    if (run > tiles) run = tiles;
    if (run < 1) run = 1;
    const long long runs = (tiles + run - 1) / run;
    run = (tiles + runs - 1) / runs;
    const long long blocks = round_up_xcd(runs * groups) * grp * run;
    if (blocks > MAX_PROJ_BLOCKS) return o;
    o.grp = grp;
    o.run = static_cast<int>(run);
    o.blocks = blocks;
    return o;
}

// The (projection, tile) pair of a workgroup: position k in the view list and
// tile index; valid is false for the padding.
struct Pair {
    int k, tile;
    bool valid;
};

constexpr Pair pair_of(int block, int grp, int run, int tiles, int n_views) {
    const int size = grp * run;
    const int j = block / N_XCD, ul = j / size, in = j - ul * size;
    const int unit = ul * N_XCD + block % N_XCD;
    const int runs = (tiles + run - 1) / run;
    const int gi = unit / runs, it = in / grp;
    const int k = gi * grp + in - it * grp;
    const int tile = (unit - gi * runs) * run + it;
    const bool valid = k < n_views && tile < tiles;
    return Pair{valid ? k : 0, valid ? tile : 0, valid};
}

}  // namespace ctrex
