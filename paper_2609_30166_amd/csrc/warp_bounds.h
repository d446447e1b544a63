// Bounds of the displacement nodes that a brick of the warped backprojector
// looks up: host and device.
#pragma once

#include <cmath>

namespace ctrex {

// Starting positions that can land in a brick are bounded by the displacements
// of its nodes, less and more this part of a voxel and of the displacements,
// which covers the FP32 rounding of a displaced position.
constexpr float WALK_ROUND = 1e-5f;

// How far (voxels) a walked sample may lie outside its brick's box: the scan's
// displacement bound and its WALK_ROUND, the range estimate's margins of 1/64 +
// 2^-20 i samples (i steps are at most the hull's diagonal) and of 2^-22 of the
// largest side.
__host__ __device__ inline double walk_margin(int margin, double step, int nx, int ny, int nz) {
    return margin + 1.01 * WALK_ROUND * (1.0 + 2.0 * margin) + step / 64.0 +
           (static_cast<double>(nx) + ny + nz) * 0x1p-19;
}

// Rounding of an FP32 node coordinate of an axis of gn nodes, generously.
__host__ __device__ inline double node_slack(int gn) { return 1e-3 + gn * 0x1p-20; }

// Nodes that the lookups of positions in [lo - M, hi + M], clipped to the
// hull, can touch on an axis of n voxels and gn nodes at `scale` nodes per
// voxel.
__host__ __device__ inline void node_range(double lo, double hi, double M, int n, int gn,
                                           double scale, int &first, int &count) {
    const double a = fmax(lo - M, 0.0) * scale - node_slack(gn);
    const double b = fmin(hi + M, n - 1.0) * scale + node_slack(gn);
    const int i0 = static_cast<int>(fmin(fmax(floor(a), 0.0), gn - 2.0));
    const int i1 = static_cast<int>(fmin(fmax(floor(b), 0.0), gn - 2.0)) + 1;
    first = i0;
    count = i1 - i0 + 1;
}

}  // namespace ctrex
