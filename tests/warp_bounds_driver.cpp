// Checks on the CPU that the nodes a warped brick keeps hold every lookup of
// the samples it walks: for the outermost starting positions, formed as the
// kernel forms its bounds, on axes of up to 330 nodes (LDS holds 1320 of a
// brick, at least two on each of the other axes) and for displacements up to the
// largest, 64 voxels.  Ends with 1 at the first miss.
#include <algorithm>
#include <cstdio>

#include "warp_bounds.h"

using namespace ctrex;

int main() {
    const double step = 0.5;
    for (int n = 33; n <= 300; n += (n < 70 ? 1 : 23))
        for (int gn = 2; gn <= 330; ++gn)
            for (int margin = 1; margin <= 64; ++margin)
                for (int x0 = 0; x0 < n - 1; x0 += 32) {
                    const double scale = double(gn - 1) / (n - 1);
                    const int e = std::min(32, n - x0);
                    int first, count;
                    node_range(x0, x0 + e, walk_margin(margin, step, n, 2, 2), n, gn, scale, first, count);
                    // displacements up to the bound; FP32 as in the kernel
                    const float tol = static_cast<float>(n) * 2.38418579e-7f, u = static_cast<float>(margin);
                    const float r = WALK_ROUND * (1.0f + 2.0f * u);
                    const double walk = step / 64.0 + n * 0x1p-20;   // the index estimate's margin
                    const double lo = static_cast<double>(x0 - tol - u - r) - walk;
                    const double hi = static_cast<double>(x0 + e + tol + u + r) + walk;
                    for (double c : {lo, hi}) {
                        const double pos = std::min(std::max(c, 0.0), n - 1.0);
                        // node coordinate, off by up to 2^-22 of itself
                        for (double f : {1.0 - 0x1p-22, 1.0 + 0x1p-22}) {
                            const int k = std::min(static_cast<int>(std::min(pos * scale * f, gn - 1.0)), gn - 2);
                            if (k < first || k + 1 > first + count - 1)
                                return std::printf("n %d nodes %d margin %d brick at %d: lookup at %d outside %d + %d\n",
                                                   n, gn, margin, x0, k, first, count), 1;
                        }
                    }
                }
    std::puts("ok");
    return 0;
}
