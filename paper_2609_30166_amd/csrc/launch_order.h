// Which work a workgroup takes: the order of the projectors' and the
// backprojector's launches.
// Constant-expression functions without HIP types, shared by the host, which
// sizes the launch, and the kernels.
#pragma once

namespace ctrex {

constexpr int N_XCD = 8;
// A launch holds fewer than 2^32 threads: 2^24 workgroups of the projectors' 256.
constexpr long long MAX_PROJ_BLOCKS = (1ll << 24) - 1;

constexpr long long round_up_xcd(long long n) { return (n + N_XCD - 1) / N_XCD * N_XCD; }

// Units of the projectors' launch (pair_of): groups of grp projections x runs
// of run detector tiles (runs per group: runs), and the workgroups of whole
// units, a multiple of N_XCD.  turn: see xcd_turn.
struct LaunchOrder {
    int grp = 1, run = 1, runs = 1, turn = 0;
    long long blocks = 0;
};

// Turn of the j-th eight units against the XCDs: triangular numbers, so that
// units at any fixed distance from one eight to the next, which may be all that
// have work, go to all XCDs alike over 16 eights.
constexpr unsigned xcd_turn(unsigned j) { return (j & 15) * ((j & 15) + 1) / 2; }

constexpr long long gcd(long long a, long long b) { return b == 0 ? a : gcd(b, a % b); }

// Order for n_views images of rows x row tiles: groups of up to `group`
// projections (0: 16), runs of up to 32 tiles, both evened out so that the last
// one is not mostly empty; runs shorter where there are too few pairs for 16
// units per XCD.  Where the padding of whole units would exceed the threads of a
// launch, single pairs are handed out.
//
// narrow: the volume's image is much narrower than the detector, so only a few
// tiles of each row have work.  Every second or third unit then does, and where
// the units of a few rows are a multiple of eight, all that do go to two or
// three XCDs.  Runs are whole rows there, each with as much work as the next,
// and turned, since rows past the volume's ends have none: 30 views of 384^2 of
// a 256 x 32 x 32 volume (z, y, x) 161 -> 95 us, of 300 x 60 x 60 324 -> 174.
//
// Wider images are turned only if units come back to the same XCDs after one to
// three rows of at least eight (cyl, the cylindrical domain, whose rays differ
// more in length: one to four rows, and half of all rows at most) and not all of
// them run at once, three to a CU: some XCDs would have the detector's middle,
// others its sides, where rays are short.  30
// views at 80^3 (8 tiles to a row) 129 -> 114 us, 165^3 (16) 722 -> 598, 256^3
// (24, runs of 9) 2779 -> 2327.  Others keep the same columns on an XCD for
// longer (turned, 100^3 with 30 views took 181 us instead of 171, the SIRT step
// on a 96 x 603 x 192 cylinder 7.4 ms instead of 6.5).
constexpr LaunchOrder launch_order(int row, int rows, int n_views, bool narrow = false,
                                   int group = 0, bool cyl = false) {
    constexpr int kGroup = 16, kRun = 32, kUnits = 16 * N_XCD, kRound = 3 * 256;
    LaunchOrder o;
    const long long tiles = static_cast<long long>(row) * rows, total = tiles * n_views;
    o.runs = static_cast<int>(tiles);
    o.blocks = round_up_xcd(total);
    if (total <= 0 || total > MAX_PROJ_BLOCKS) return o;
    if (group <= 0) group = kGroup;
    const int groups = (n_views - 1) / group + 1;
    const int grp = (n_views + groups - 1) / groups;
    long long run = total / (static_cast<long long>(grp) * kUnits);
    if (run > kRun) run = kRun;
    if (run > tiles) run = tiles;
    if (run < 1) run = 1;
    narrow = narrow && static_cast<long long>(rows) * groups >= 2 * N_XCD;
    if (narrow) run = row;
    const long long runs = (tiles + run - 1) / run;
    run = (tiles + runs - 1) / runs;
    const long long blocks = round_up_xcd(runs * groups) * grp * run;
    if (blocks > MAX_PROJ_BLOCKS) return o;
    // rows after which units fall on the same XCDs again
    const long long period = N_XCD * run / gcd(row, N_XCD * run);
    const int limit = cyl ? (rows < 8 ? rows / 2 : 4) : rows < 8 ? 0 : 3;
    o.grp = grp;
    o.run = static_cast<int>(run);
    o.runs = static_cast<int>(runs);
    o.turn = narrow || (period <= limit && group == kGroup && total > kRound) ? 1 : 0;
    o.blocks = blocks;
    return o;
}

// The (projection, tile) pair of a workgroup: position k in the view list and
// tile index; valid is false for the padding.
struct Pair {
    int k, tile;
    bool valid;
};

constexpr Pair pair_of(unsigned block, int grp, int run, int runs, int turn, int tiles,
                       int n_views) {
    const unsigned size = static_cast<unsigned>(grp) * static_cast<unsigned>(run);
    const unsigned j = block / N_XCD, ul = j / size, in = j - ul * size;
    const unsigned unit = ul * N_XCD + (block + (turn ? xcd_turn(ul) : 0u)) % N_XCD;
    const unsigned gi = unit / static_cast<unsigned>(runs), it = in / static_cast<unsigned>(grp);
    const unsigned k = gi * static_cast<unsigned>(grp) + in - it * static_cast<unsigned>(grp);
    const unsigned tile = (unit - gi * static_cast<unsigned>(runs)) * static_cast<unsigned>(run) + it;
    const bool valid = k < static_cast<unsigned>(n_views) && tile < static_cast<unsigned>(tiles);
    return Pair{valid ? static_cast<int>(k) : 0, valid ? static_cast<int>(tile) : 0, valid};
}

// Order of the backprojector's (brick, projection chunk) items, bricks in rows
// along x, chunks fastest: units of run consecutive items (a brick's chunks stay
// on one XCD where they can, as they add to the same voxels) go to the XCDs in
// turn, so that those stay equally loaded where the ends of the volume see few
// rays; blocks is the launch's workgroups, whole units and a multiple of N_XCD.
//
// A multiple of eight rows goes out by rows.  Other counts would leave XCDs
// idle (one row of eight bricks, 16 x 16 x 256 with 180 views: 1046 us on one
// XCD, 222 now; 9 rows, 48^3: 493 -> 331 us), so units are bricks there, or
// parts of one for at least 16 units per XCD, turned (xcd_turn) because a row's
// last brick is often a narrow one: without the turn 100^3 takes 2870 us
// instead of 2650.  By bricks, 72 rows (117 x 133 x 121) took 968 us instead of
// 850 with each XCD's bricks far apart.
struct BrickOrder {
    int run = 1, turn = 0;
    long long blocks = 0;
};

constexpr BrickOrder brick_order(int rows, int per_row, int chunks) {
    constexpr long long kUnits = 16 * N_XCD;
    const long long bricks = static_cast<long long>(rows) * per_row;
    BrickOrder o;
    if (rows % N_XCD == 0) {
        o.run = per_row * chunks;
    } else {
        const long long parts = (kUnits + bricks - 1) / bricks;
        o.run = parts < chunks ? static_cast<int>(chunks / parts) : 1;
        o.turn = 1;
    }
    o.blocks = round_up_xcd((bricks * chunks + o.run - 1) / o.run) * o.run;
    return o;
}

// The item of a workgroup (past the last one for the padding).
constexpr unsigned item_of(unsigned block, int run, int turn) {
    const unsigned j = block / N_XCD, ul = j / static_cast<unsigned>(run);
    const unsigned unit = ul * N_XCD + (block + (turn ? xcd_turn(ul) : 0u)) % N_XCD;
    return unit * static_cast<unsigned>(run) + (j - ul * static_cast<unsigned>(run));
}

}  // namespace ctrex
