// Exact-transpose backprojector with brick-resident LDS accumulation (gfx950).
//
// z += A^T r walks exactly the samples of the forward projector (same FP64
// ray set-up, same FP32 sample positions, warp and corners) and adds
// (h r / n_sub) times the eight trilinear weights of every sample to the
// volume (Sec. 4.1 backprojection operator, taken as the transpose of the
// projection operator; Sec. 3.4: a projection's residual is spread over its
// sub-views).
//
// Two forms share these ideas.  The default (bp_own_kernel) walks a sample only
// in the brick that holds its lower corner and adds the bricks' integers into a
// 64-bit volume; the direct form (bp_brick_kernel), for callers without room
// for that volume, is described here:
//
// Scattering every sample to HBM would cost eight L2 float atomics per
// sample.  A workgroup owns a brick of the volume (up to 32x15x16
// voxels) held in LDS for a whole chunk of projections, accumulated as 64-bit
// fixed point with LDS integer atomics: on gfx950 these sustain about twenty
// times the lane rate of LDS FP32 atomic adds, and the sums are exact (so the
// result does not depend on the order of the atomics).  A scale bounded from
// max|r| puts the largest possible contribution at 2^30, so each one is a
// 32-bit integer (weights formed in FP32, rounded to the nearest unit) while
// the 64-bit sums cannot overflow.  For every (projection, sub-view) it bounds
// the detector pixels whose rays can reach the brick (the projection of the brick grown by one voxel and the warp
// bound), redoes those rays' FP64 set-up, clips their sample range to the
// grown brick, and adds its eight corners with LDS 64-bit integer atomics.
// The LDS brick carries one halo cell on each side in x and y, which takes
// the corners that fall outside the brick there and is never written out; a
// corner outside in z gets weight zero.  A sample whose corner cube straddles
// a brick face is visited by each brick it touches, and each keeps only its
// own corners, so every corner is counted once.  There is no global atomic
// and no barrier inside the projection loop; the brick is written out once
// at the end (into a partial volume per projection chunk, summed in a fixed
// order, when several chunks share a brick).

#include "ray_common.h"
#include "warp_bounds.h"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace ctrex {
namespace {

using namespace dev;

// Launch shape of bp_brick_kernel (the direct form, and the warped owner form
// where a brick's displacement nodes do not fit in LDS).  Unwarped: 16 waves per
// workgroup, one workgroup per CU (its LDS brick and its waves' ray tables take
// 140 KB of the 160), so 4 waves per SIMD at up to 128 registers.  LDS
// instructions take about six CU cycles whatever their number of active lanes,
// so a hand-over reads the next ray from the table (four 16-byte reads by the
// lanes that hand over) instead of fifteen full-wave permutes.  Warped: the
// displacement loads need the latency hiding of 6 waves per SIMD (12 waves per
// workgroup, two per CU, no table), and hand-overs permute.
template <bool WARP> constexpr int bp_threads() { return WARP ? 768 : 1024; }
template <bool WARP> constexpr bool bp_table() { return !WARP; }

// Largest brick, and its LDS layout: rows of BRICK_X + 2 cells (halo on both
// sides, padded to an odd stride) and planes of BRICK_Y + 2 rows.  64-bit
// cells span two 4-byte banks; the odd row stride and a plane stride of 3
// (mod 16) put neighbours along y, z and the diagonals in other banks.  Two
// bricks (2 x 76 KB) share a CU's 160 KB of LDS.
constexpr int BRICK_X = 32, BRICK_Y = 15, BRICK_Z = 16;
constexpr int LDS_SY = (BRICK_X + 2) | 1;
constexpr int LDS_SZ = LDS_SY * (BRICK_Y + 2);
constexpr int LDS_CELLS = LDS_SZ * BRICK_Z;
static_assert(LDS_SZ % 16 == 3, "plane stride");

// Owner-computes bricks (the default form): a brick takes exactly the
// samples whose lower corner lies in it, so every sample is walked once and
// issues its eight atomics once, into LDS cells for the brick's voxels plus
// one halo layer on the high side of each axis (33 x 17 x 17 cells).  Row and
// plane strides are 2 and 7 (mod 16): a wave's samples lie near a plane
// parallel to a hull face, and with both 1 (mod 16) the cells along each
// diagonal of that patch shared a bank (SIRT step over 180 views of 768^2 at
// 512^3: 390 ms; 371 ms with 2 and 7, 371 to 374 ms with five other pairs).
// Every brick then adds its cells, halo included, into a 64-bit integer volume
// with global atomics; integer sums are exact, so neighbours' halos and
// projection chunks combine in any order and the result stays bitwise
// reproducible.  All workgroups use one fixed-point scale for that.  The
// direct form above (a sample walked by every brick it touches, each brick
// writing only its own voxels) needs no volume-sized buffer and serves the
// allocation-free entry point.
constexpr int OWN_X = 32, OWN_Y = 16, OWN_Z = 16;
constexpr int OWN_SY = OWN_X + 2;
constexpr int OWN_SZ = OWN_SY * (OWN_Y + 1) + 5;
constexpr int OWN_CELLS = OWN_SZ * (OWN_Z + 1);
constexpr int MAX_CELLS = OWN_CELLS > LDS_CELLS ? OWN_CELLS : LDS_CELLS;
static_assert(OWN_SY % 16 == 2 && OWN_SZ % 16 == 7, "owner strides");

struct BrickGrid {
    int bx, by, bz;       // brick size (voxels), at most BRICK_X x BRICK_Y x BRICK_Z
    int nbx, nby, nbz;    // bricks per axis
    int chunks;           // projection chunks per brick
    int views_per_chunk;
    int total;            // nbx * nby * nbz * chunks
    int run, turn;        // owner form: launch order (BrickOrder)
    int accumulate;       // add into vol (else overwrite; needs chunks == 1)
    float wscale;         // every contribution is multiplied by this factor
    double cube_samples;  // max samples of one ray inside a side-2 cube
    float *partials;      // direct form: [chunks][nx*ny*nz] per-chunk results when chunks > 1
    unsigned long long *acc64;  // owner form: the 64-bit integer volume the bricks add into
};

// Fixed-point exponent of the owner form, the same in every workgroup and in
// the finishing pass: the largest contribution cmax at or below 2^30, and the
// sum into any voxel below 2^62 (at most every ray of every listed sub-view
// passes through the voxel's corner cube, each with at most cube_samples
// samples there).
__device__ __forceinline__ int own_kexp(double cmax, const RayGrid &g, double cube_samples) {
    const double rays = static_cast<double>(g.n_views) * g.n_sub * g.n_u * g.n_v;
    return static_cast<int>(floor(fmin(30.0 - log2(cmax), 62.0 - log2(rays * cube_samples * cmax))));
}

// A lane merges at most OWN_MERGE_MAX samples into its register sums (it
// starts a new run every OWN_MERGE_MAX iterations), and only while the sum of their ray weights |c| (each bounds all eight corner
// contributions of a sample, the trilinear weights being at most 1) stays at
// or below OWN_MERGE_LIMIT: the FP32 sums then exceed the exact ones by at
// most (1024 + 4) 2^-24 of 2^31 < 2^18, inside the 2^19 margin, so a merged
// corner sum converts to a 32-bit integer.
constexpr int OWN_MERGE_MAX = 1024;
static_assert((OWN_MERGE_MAX & (OWN_MERGE_MAX - 1)) == 0, "power of two");
constexpr float OWN_MERGE_LIMIT = 2147483648.0f - 524288.0f;   // 2^31 - 2^19

// Largest contribution of one sample to one corner: step * max|r| / n_sub
// times the caller's factor (and a margin for FP32 rounding).
__device__ __forceinline__ double contribution_bound(const RayGrid &g, double rmax, float wscale) {
    return rmax * g.step * (1.0 + 1e-5) * fabs(static_cast<double>(wscale)) / g.n_sub;
}

// Project the 8 corners of an index-space box through the view matrix and
// return the detector pixel range whose rays can cross the box.  When all
// corners lie on one side of the plane through the source parallel to the
// detector (w of one sign), the box's image is the hull of the corner images;
// otherwise the image is unbounded and false asks for the whole detector.
__device__ __forceinline__ bool project_box(const double *P, const double lo[3],
                                            const double hi[3], const double off[3], int n_u,
                                            int n_v, int &u0, int &u1, int &v0, int &v1) {
    double umin = 1e300, umax = -1e300, vmin = 1e300, vmax = -1e300;
    bool pos = true, neg = true;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const double X = ((c & 1) ? hi[0] : lo[0]) - off[0];
        const double Y = ((c & 2) ? hi[1] : lo[1]) - off[1];
        const double Z = ((c & 4) ? hi[2] : lo[2]) - off[2];
        const double a = P[0] * X + P[1] * Y + P[2] * Z + P[3];
        const double b = P[4] * X + P[5] * Y + P[6] * Z + P[7];
        const double w = P[8] * X + P[9] * Y + P[10] * Z + P[11];
        pos = pos && w > 0.0;
        neg = neg && w < 0.0;
        const double u = a / w, v = b / w;
        umin = fmin(umin, u);
        umax = fmax(umax, u);
        vmin = fmin(vmin, v);
        vmax = fmax(vmax, v);
    }
    if (!(pos || neg)) return false;
    u0 = static_cast<int>(fmax(floor(umin) - 1.0, 0.0));
    v0 = static_cast<int>(fmax(floor(vmin) - 1.0, 0.0));
    u1 = static_cast<int>(fmin(ceil(umax) + 1.0, static_cast<double>(n_u - 1)));
    v1 = static_cast<int>(fmin(ceil(vmax) + 1.0, static_cast<double>(n_v - 1)));
    return true;
}

// Wave-uniform values computed by vector instructions (LDS reads, FP64 or
// float conversions) stay in vector registers unless moved to scalar ones;
// at 64 vector registers per lane they would be spilled.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uni(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ double uni(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)));
    const int hi = __builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32));
    return __longlong_as_double((static_cast<long long>(hi) << 32) | lo);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP lane moves:
// shifts by 1, 2, 4, 8 within each row of 16 lanes (zero shifted in), then
// the last lane of row 0 added to row 1 and of row 2 to row 3 (row broadcast
// 15), then lane 31 added to rows 2 and 3 (row broadcast 31).  No LDS and no
// per-lane addresses.  Called with all 64 lanes of the wave active.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 -> rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 -> rows 2, 3
    return x;
}

// First of the T samples of a wave that lane `lane` takes: floor(T lane / 64).
// T reaches 2^30 (64 rays of under 2^24 samples, as ctrex_set_geometry
// ensures), so the product itself does not fit 32 bits for steps below 1e-4.
__device__ __forceinline__ int share(int T, int lane) {
    return (T >> 6) * lane + (((T & 63) * lane) >> 6);
}

// One contribution as a 64-bit fixed-point integer: c (FP32, the scale
// folded in, |c| < 2^31) rounded to the nearest integer, then sign-extended.
// Rounding errs by at most half a unit and without bias, so the error of a
// voxel's sum grows with the square root of its number of contributions.
__device__ __forceinline__ unsigned long long to_fixed(float c) {
    return static_cast<unsigned long long>(static_cast<long long>(static_cast<int>(rintf(c))));
}

// One ray of a wave's 8x8 pixel block, as the lanes that walk its samples
// need it: position of its first sample in the brick range and its step (both
// 64-bit fixed point), its weight, the end of its samples in the wave's order
// and the next ray of the block with samples (64 bytes, four 16-byte reads).
struct alignas(16) RayRec {
    long long px, py, pz;
    long long tx, ty, tz;
    float wq;
    int end;
    int next;
    int pad;
};
static_assert(sizeof(RayRec) == 64, "ray record");

// Orders one wave's LDS writes before its other lanes' reads of them (and
// those reads before the next writes); no instruction beyond a wait.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename TS, int MODE, bool WARP, bool OWN>
__global__ __launch_bounds__(bp_threads<WARP>())
__attribute__((amdgpu_waves_per_eu(WARP ? 6 : 4, WARP ? 6 : 4))) void bp_brick_kernel(RayGrid g, WarpGrid w,
                                                              const double *__restrict__ Pmat,
                                                              const TS *__restrict__ sino,
                                                              const float *__restrict__ rmax,
                                                              float *__restrict__ vol,
                                                              BrickGrid bg) {
    static_assert(!OWN || WARP, "the unwarped owner form is bp_own_kernel");
    __shared__ unsigned long long acc[MAX_CELLS];
    constexpr int BP_THREADS = bp_threads<WARP>();
    constexpr bool TABLE = bp_table<WARP>();
    __shared__ double red[BP_THREADS / 64];
    __shared__ RayRec rays[TABLE ? BP_THREADS : 1];
    RayRec *const tabw = rays + (threadIdx.x & ~63);
    // ---- block -> (brick, projection chunk); XCD-aware so that one XCD
    // works on neighbouring bricks
    const int per = (bg.total + N_XCD - 1) / N_XCD;
    const int L = (blockIdx.x % N_XCD) * per + blockIdx.x / N_XCD;
    if (L >= bg.total) return;
    const int chunk = L % bg.chunks;
    int b = L / bg.chunks;
    const int ibx = b % bg.nbx;
    b /= bg.nbx;
    const int iby = b % bg.nby;
    const int ibz = b / bg.nby;
    const int x0 = ibx * bg.bx, y0 = iby * bg.by, z0 = ibz * bg.bz;
    const int ex = min(bg.bx, g.nx - x0), ey = min(bg.by, g.ny - y0), ez = min(bg.bz, g.nz - z0);
    const int nlds = OWN ? OWN_CELLS : LDS_SZ * ez;
    for (int i = threadIdx.x; i < nlds; i += BP_THREADS) acc[i] = 0ull;
    // cell (lx, ly, lz) of the brick: direct form lx in [-1, ex], ly in
    // [-1, ey]; owner form lx in [0, ex], ly in [0, ey], lz in [0, ez]
    unsigned long long *const cell0 = OWN ? acc : acc + LDS_SY + 1;

    const VolDims d = vol_dims(g);
    const float M = static_cast<float>(w.margin);
    // samples with an (unwarped) position in [lo, hi] can touch the brick,
    // for any projection (the warp bound of the whole scan)
    const double lod[3] = {x0 - 1.0 - M, y0 - 1.0 - M, z0 - 1.0 - M};
    const double hid[3] = {static_cast<double>(x0 + ex) + M, static_cast<double>(y0 + ey) + M,
                           static_cast<double>(z0 + ez) + M};
    const double off[3] = {0.5 * (g.nx - 1), 0.5 * (g.ny - 1), 0.5 * (g.nz - 1)};
    // 1 / n_sub and the caller's factor (1 unless scaled; exact when a power of 2)
    const float inv_sub = uni(bg.wscale / static_cast<float>(g.n_sub));
    // largest side times 2^-22: four times the FP32 rounding error of a
    // coordinate of a ray's start
    const float tol = uni(static_cast<float>(max(g.nx, max(g.ny, g.nz))) * 2.38418579e-7f);
    const int k_first = chunk * bg.views_per_chunk;
    const int k_end = min(k_first + bg.views_per_chunk, g.n_views);
    const int n_pairs = (k_end - k_first) * g.n_sub;

    // ---- fixed-point scale.  Each contribution is at most
    // cmax = step * max|r| / n_sub (times the caller's factor), and every
    // contribution to a voxel comes from a sample of a ray in some pair's
    // pixel box lying in the voxel's corner cube (side 2), at most
    // bg.cube_samples of them per ray.  The scale 2^kexp puts the largest
    // contribution at or below 2^30 (so it fits a 32-bit integer) and keeps
    // the bound on the sums below 2^62.
    double nrays = 0.0;
    for (int q = threadIdx.x; q < (OWN ? 0 : n_pairs); q += BP_THREADS) {
        const int k = k_first + q / g.n_sub;
        const int p = g.views ? g.views[k] : k;
        const int sv_idx = p * g.n_sub + q % g.n_sub;
        int u0, u1, v0, v1;
        if (project_box(Pmat + 12 * static_cast<size_t>(sv_idx), lod, hid, off, g.n_u, g.n_v, u0,
                        u1, v0, v1))
            nrays += (u0 <= u1 && v0 <= v1) ? double(u1 - u0 + 1) * double(v1 - v0 + 1) : 0.0;
        else
            nrays += double(g.n_u) * double(g.n_v);
    }
    for (int o = 32; o > 0; o >>= 1) nrays += __shfl_xor(nrays, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = nrays;
    __syncthreads();
    nrays = 0.0;
    for (int i = 0; i < BP_THREADS / 64; ++i) nrays += red[i];
    const double cmax =
        contribution_bound(g, (MODE == BP_ONES) ? 1.0 : static_cast<double>(*rmax), bg.wscale);
    const double bound = OWN ? cmax : nrays * bg.cube_samples * cmax;
    const bool bad = !(cmax < __builtin_inf());   // NaN or Inf in the input: propagate NaN
    const bool any = uni(static_cast<int>(bound > 0.0 && !bad)) != 0;
    const int kexp = uni(!any ? 0
                         : OWN ? own_kexp(cmax, g, bg.cube_samples)
                               : static_cast<int>(floor(fmin(30.0 - log2(cmax),
                                                             62.0 - log2(bound)))));
    const double scale = uni(ldexp(1.0, kexp));

    // each wave takes whole (projection, sub-view) pairs, so a pair's pixel
    // box is projected once, by the wave that walks its rays
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    for (int q = wave; q < n_pairs && any; q += BP_THREADS / 64) {
        const int k = k_first + q / g.n_sub;
        const int s = q - (q / g.n_sub) * g.n_sub;
        const int p = uni(g.views ? g.views[k] : k);
        {
            const int sv_idx = p * g.n_sub + s;
            const SubView &sv = g.tab[sv_idx];
            // this sub-view's warp moves samples by at most |tau| max|U| on
            // every axis: its samples within that margin of the brick can
            // touch it (time-linear fields: half the scan's bound on average)
            const double mv = WARP ? fabs(sv.tau) * w.umax : 0.0;
            const float Mp = uni(mv > 0.0 ? static_cast<float>(ceil(mv * (1.0 + 1e-6) + 1e-6)) : 0.0f);
            // direct form: samples with a corner in the brick, position in
            // [x0 - 1, x0 + ex]; owner form: lower corner in it, [x0, x0 + ex]
            // The ray-range estimate below takes the ray's start in FP32,
            // off by up to 2^-24 of a coordinate: the bounds are widened by
            // 2^-22 of the largest side (this adds samples that the
            // exact corner test then rejects; for a ray almost parallel to an
            // axis the one-sample widening would not cover it)
            const float g0 = (OWN ? 0.0f : 1.0f) + tol;
            const float lo[3] = {uni(x0 - g0 - Mp), uni(y0 - g0 - Mp), uni(z0 - g0 - Mp)};
            const float hi[3] = {uni(static_cast<float>(x0 + ex) + Mp + tol),
                                 uni(static_cast<float>(y0 + ey) + Mp + tol),
                                 uni(static_cast<float>(z0 + ez) + Mp + tol)};
            const double plo[3] = {lo[0], lo[1], lo[2]}, phi[3] = {hi[0], hi[1], hi[2]};
            int u0 = 0, u1 = g.n_u - 1, v0 = 0, v1 = g.n_v - 1;
            if (!project_box(Pmat + 12 * static_cast<size_t>(sv_idx), plo, phi, off, g.n_u, g.n_v,
                             u0, u1, v0, v1)) {
                u0 = 0;
                u1 = g.n_u - 1;
                v0 = 0;
                v1 = g.n_v - 1;
            }
            u0 = uni(u0);
            u1 = uni(u1);
            v0 = uni(v0);
            v1 = uni(v1);
            if (u0 > u1 || v0 > v1) continue;
            // rays in 8x8 pixel blocks, one block per pass; the wave shares
            // each block's samples evenly among its lanes
            const int bu = (u1 - u0 + 8) >> 3;
            const int nblk = bu * ((v1 - v0 + 8) >> 3);
            const float tau = uni(static_cast<float>(sv.tau));
            const int lane = threadIdx.x & 63;
            for (int blk = 0; blk < nblk; ++blk) {
                const int iv = v0 + (blk / bu) * 8 + (lane >> 3);
                const int iu = u0 + (blk % bu) * 8 + (lane & 7);
                // ---- this lane's ray: its samples that can reach the brick
                int len = 0, ib = 0;
                float wq = 0.0f;   // h r / n_sub in fixed-point units
                Ray r;
                r.qx = r.qy = r.qz = r.tx = r.ty = r.tz = 0;
                const float rv = (iu > u1 || iv > v1) ? 0.0f
                                 : (MODE == BP_ONES) ? 1.0f
                                                     : ld(sino, (k * g.n_v + iv) * g.n_u + iu);
                if (rv != 0.0f && setup_ray(sv, static_cast<double>(iu), static_cast<double>(iv),
                                            g.nx, g.ny, g.nz, g.step, r)) {
                    // sample indices i with b + i s inside [lo, hi] on every
                    // axis, in FP32 (corners are checked exactly below).  The
                    // FP32 start and step put b + i s within 2^-24 (|b| + L) <
                    // 2.8 2^-24 max side of the fixed-point position of sample
                    // i (L the ray length, at most sqrt(3) max side), and
                    // [lo, hi] is widened by tol = 4 2^-24 max side; the index estimate itself is three
                    // roundings, under 3 2^-24 |t|, inside the margin of
                    // 1/64 + 2^-20 |t| samples.  An axis the ray does not move
                    // along (|s| under 1e-30: its samples drift by less than
                    // tol) only decides whether the ray hits; branch-free.
                    float kmin = 0.0f, kmax = static_cast<float>(r.n - 1);
                    const float bv[3] = {r.bx, r.by, r.bz};
                    const float sv3[3] = {r.fx, r.fy, r.fz};
                    bool hit = true;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const bool flat = fabsf(sv3[q]) < 1e-30f;
                        const float inv = 1.0f / (flat ? 1.0f : sv3[q]);
                        const float t1 = (lo[q] - bv[q]) * inv, t2 = (hi[q] - bv[q]) * inv;
                        const float tl = fminf(t1, t2), th = fmaxf(t1, t2);
                        const float ml = fmaf(fabsf(tl), 9.5367431640625e-7f, 0.015625f);
                        const float mh = fmaf(fabsf(th), 9.5367431640625e-7f, 0.015625f);
                        kmin = flat ? kmin : fmaxf(kmin, tl - ml);
                        kmax = flat ? kmax : fminf(kmax, th + mh);
                        hit &= !(flat & ((bv[q] < lo[q]) | (bv[q] > hi[q])));
                    }
                    if (hit && kmin <= kmax) {
                        ib = max(static_cast<int>(ceilf(kmin)), 0);
                        const int ie = min(static_cast<int>(floorf(kmax)), r.n - 1);
                        len = max(ie - ib + 1, 0);
                        wq = static_cast<float>(static_cast<double>(r.h * rv * inv_sub) * scale);
                    }
                }
                // ---- exclusive prefix of the segment lengths over the wave
                const int incl = wave_inclusive_sum(len);
                const int S = incl - len;
                const int T = __builtin_amdgcn_readlane(incl, 63);
                if (T == 0) continue;   // uniform over the wave
                const unsigned long long live = __ballot(len > 0);
                // ---- this lane's ray (position of its first sample in the
                // brick range, step, weight, end of its samples in the wave's
                // order, next ray with samples) for the lanes that walk into
                // it: in the wave's LDS table, or permuted from this lane
                RayRec mine;
                {
                    const unsigned long long later =
                        lane < 63 ? (live & (~0ull << (lane + 1))) : 0ull;
                    mine.px = r.qx + static_cast<long long>(ib) * r.tx;
                    mine.py = r.qy + static_cast<long long>(ib) * r.ty;
                    mine.pz = r.qz + static_cast<long long>(ib) * r.tz;
                    mine.tx = r.tx;
                    mine.ty = r.ty;
                    mine.tz = r.tz;
                    mine.wq = wq;
                    mine.end = incl;
                    mine.next = later ? __ffsll(static_cast<long long>(later)) - 1 : lane;
                    mine.pad = 0;
                }
                // the record of ray `src` (every lane executes the permutes: a
                // permute skipped by the source lane returns 0)
                auto fetch = [&](int src) {
                    RayRec e;
                    if (TABLE) {
                        e = tabw[src];
                    } else {
                        e.px = __shfl(mine.px, src, 64);
                        e.py = __shfl(mine.py, src, 64);
                        e.pz = __shfl(mine.pz, src, 64);
                        e.tx = __shfl(mine.tx, src, 64);
                        e.ty = __shfl(mine.ty, src, 64);
                        e.tz = __shfl(mine.tz, src, 64);
                        e.wq = __shfl(mine.wq, src, 64);
                        e.end = __shfl(mine.end, src, 64);
                        e.next = __shfl(mine.next, src, 64);
                    }
                    return e;
                };
                if (TABLE) {
                    tabw[lane] = mine;
                    wave_sync();
                }
                // ---- lane takes samples [start, end) of the wave's T
                const int start = share(T, lane), end = share(T, lane + 1);
                int j = 0;   // last ray with S_j <= start: it owns sample `start`
#pragma unroll
                for (int st = 32; st > 0; st >>= 1) {
                    const int t = j + st;
                    if (__shfl(S, t, 64) <= start) j = t;
                }
                // the lane's first ray may be entered mid-way: `start - S_j`
                // samples after its first sample in the brick range
                const long long m = start - __shfl(S, j, 64);
                long long px, py, pz, ctx, cty, ctz;
                float cwq;
                int cend, cnext;
                {
                    const RayRec e = fetch(j);
                    ctx = e.tx;
                    cty = e.ty;
                    ctz = e.tz;
                    px = e.px + m * ctx;
                    py = e.py + m * cty;
                    pz = e.pz + m * ctz;
                    cwq = e.wq;
                    cend = e.end;
                    cnext = e.next;
                }
                const int trips = (T + 63) >> 6;
                {
                    int pos = start;
                    for (int it = 0; it < trips; ++it) {
                        // wave-uniform hand-over to the next ray with samples;
                        // it is entered at its first sample in the brick range
                        const bool need = pos < end && pos == cend;
                        if (TABLE ? need : __any(need)) {
                            // with the table only the lanes that hand over
                            // read; permutes run on every lane, and the others
                            // keep their ray
                            const RayRec f = fetch(TABLE ? cnext : (need ? cnext : lane));
                            const RayRec e = need ? f : RayRec{px, py, pz, ctx, cty, ctz,
                                                               cwq, cend, cnext, 0};
                            px = e.px;
                            py = e.py;
                            pz = e.pz;
                            ctx = e.tx;
                            cty = e.ty;
                            ctz = e.tz;
                            cwq = e.wq;
                            cend = e.end;
                            cnext = e.next;
                        }
                        if (pos >= end) continue;
                        ++pos;
                        const long long qx = px, qy = py, qz = pz;
                        px += ctx;
                        py += cty;
                        pz += ctz;
                        int ix, iy, iz;
                        float fx, fy, fz;
                        NodeCell nodes;
                        if (!sample_corner<WARP>(d, w, nodes, tau, qx, qy, qz, ix, iy, iz, fx, fy,
                                                 fz))
                            continue;
                        const int lx = ix - x0, ly = iy - y0, lz = iz - z0;
                        if (OWN) {
                            // another brick owns this sample's lower corner
                            if (static_cast<uint32_t>(lx) >= static_cast<uint32_t>(ex) ||
                                static_cast<uint32_t>(ly) >= static_cast<uint32_t>(ey) ||
                                static_cast<uint32_t>(lz) >= static_cast<uint32_t>(ez))
                                continue;
                            const float gx1 = fx, gx0 = 1.0f - fx;
                            const float gy1 = fy, gy0 = 1.0f - fy;
                            const float gz1 = fz * cwq, gz0 = (1.0f - fz) * cwq;
                            const float w00 = gz0 * gy0, w01 = gz0 * gy1, w10 = gz1 * gy0,
                                        w11 = gz1 * gy1;
                            const int cell = __mul24(lz, OWN_SZ) + __mul24(ly, OWN_SY) + lx;
                            unsigned long long *const a0 = cell0 + cell;
                            unsigned long long *const a1 = a0 + OWN_SZ;
                            atomicAdd(a0, to_fixed(w00 * gx0));
                            atomicAdd(a0 + 1, to_fixed(w00 * gx1));
                            atomicAdd(a0 + OWN_SY, to_fixed(w01 * gx0));
                            atomicAdd(a0 + OWN_SY + 1, to_fixed(w01 * gx1));
                            atomicAdd(a1, to_fixed(w10 * gx0));
                            atomicAdd(a1 + 1, to_fixed(w10 * gx1));
                            atomicAdd(a1 + OWN_SY, to_fixed(w11 * gx0));
                            atomicAdd(a1 + OWN_SY + 1, to_fixed(w11 * gx1));
                            continue;
                        }
                        // no corner in the brick: lx, ly outside [-1, e - 1] (the
                        // halo takes -1 and e - 1's upper neighbour), or lz
                        // outside [-1, ez - 1]
                        if (static_cast<uint32_t>(lx + 1) > static_cast<uint32_t>(ex) ||
                            static_cast<uint32_t>(ly + 1) > static_cast<uint32_t>(ey) ||
                            static_cast<uint32_t>(lz + 1) > static_cast<uint32_t>(ez))
                            continue;
                        const bool z_0 = lz >= 0, z_1 = lz + 1 < ez;
                        // corner weights in FP32 with the ray weight and the
                        // fixed-point scale folded in; each contribution becomes a
                        // 32-bit integer added into the 64-bit cell.  x and y
                        // neighbours outside the brick land in the halo; a z
                        // neighbour outside gets weight zero and a plane clamped
                        // into the brick (adding an integer zero changes no sum),
                        // so every lane issues the same eight atomics.
                        const float gx1 = fx, gx0 = 1.0f - fx;
                        const float gy1 = fy, gy0 = 1.0f - fy;
                        const float gz1 = (z_1 ? fz : 0.0f) * cwq;
                        const float gz0 = (z_0 ? 1.0f - fz : 0.0f) * cwq;
                        const float w00 = gz0 * gy0, w01 = gz0 * gy1, w10 = gz1 * gy0,
                                    w11 = gz1 * gy1;
                        const int row = __mul24(ly, LDS_SY) + lx;
                        unsigned long long *const a0 = cell0 + (__mul24(max(lz, 0), LDS_SZ) + row);
                        unsigned long long *const a1 =
                            cell0 + (__mul24(min(lz + 1, ez - 1), LDS_SZ) + row);
                        atomicAdd(a0, to_fixed(w00 * gx0));
                        atomicAdd(a0 + 1, to_fixed(w00 * gx1));
                        atomicAdd(a0 + LDS_SY, to_fixed(w01 * gx0));
                        atomicAdd(a0 + LDS_SY + 1, to_fixed(w01 * gx1));
                        atomicAdd(a1, to_fixed(w10 * gx0));
                        atomicAdd(a1 + 1, to_fixed(w10 * gx1));
                        atomicAdd(a1 + LDS_SY, to_fixed(w11 * gx0));
                        atomicAdd(a1 + LDS_SY + 1, to_fixed(w11 * gx1));
                    }
                }
                if (TABLE) wave_sync();   // the table is rewritten by the next block
            }
        }
    }
    __syncthreads();
    if (OWN) {
        // ---- add the brick's cells, halo included, into the integer volume
        for (int i = threadIdx.x; i < OWN_CELLS; i += BP_THREADS) {
            const int lz = i / OWN_SZ;
            const int rem = i - lz * OWN_SZ;
            const int ly = rem / OWN_SY;   // OWN_Y + 1 in a plane's padding
            const int lx = rem - ly * OWN_SY;
            const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
            const unsigned long long q = acc[i];
            if (q != 0ull && lx <= ex && ly <= ey && lz <= ez && gx < g.nx && gy < g.ny &&
                gz < g.nz)
                atomicAdd(bg.acc64 + (static_cast<size_t>(gz) * g.ny + gy) * g.nx + gx, q);
        }
        return;
    }
    // ---- write the brick out (x fastest)
    const double inv_scale = ldexp(1.0, -kexp);
    const int nvox = ex * ey * ez;
    for (int i = threadIdx.x; i < nvox; i += BP_THREADS) {
        const int lz = i / (ex * ey);
        const int rem = i - lz * ex * ey;
        const int ly = rem / ex;
        const int lx = rem - ly * ex;
        float *dst = vol + (static_cast<size_t>(z0 + lz) * g.ny + (y0 + ly)) * g.nx + (x0 + lx);
        const long long q = static_cast<long long>(cell0[lz * LDS_SZ + ly * LDS_SY + lx]);
        const float v = bad ? __builtin_nanf("") : static_cast<float>(static_cast<double>(q) * inv_scale);
        if (bg.chunks > 1) {
            // each chunk owns a slab; a fixed-order sum combines them
            bg.partials[static_cast<size_t>(chunk) * g.nx * g.ny * g.nz + (dst - vol)] = v;
        } else if (bg.accumulate) {
            *dst += v;
        } else {
            *dst = v;
        }
    }
}

// The owner form (the default backprojector).  One 16-wave workgroup per CU
// (its LDS brick, its waves' ray tables and, with the warp, its displacement
// nodes take up to 160 KB).
//
// Work is handed out in 8x8 pixel blocks: per batch of 64 (projection,
// sub-view) pairs, one wave projects the brick onto each pair's detector and
// prefix-sums the pairs' block counts, and the 16 waves take blocks from an
// LDS counter.  (A wave per pair left 7 of 16 waves idle in a 9-projection
// subset and 12 of 16 in a 4-projection chunk.)  Integer sums do not depend on
// the order, so the result stays bitwise reproducible.
//
// Bound by the LDS atomics (6.4 cycles of a CU each at least, 9 with their
// conflicts) and by VALU issue, so the sample loop is kept short: positions
// are relative to the brick; each ray's range holds exactly the samples whose
// lower corner the brick owns (trimmed with the exact positions in the
// set-up), so the loop tests nothing; the merged sums are cleared where they
// are flushed; one instruction rounds and converts.  Against a wave per pair
// with an ownership test, selects and separate rounding per sample, 180 views
// of 768^2 at 512^3 took 258 ms instead of 324, 9 views of 384^2 at 256^3
// 1.8 ms instead of 3.0.
constexpr int OWN_BATCH = 64;

// floor(c + 1/2) for |c| < 2^31: the nearest integer.
__device__ __forceinline__ unsigned long long to_fixed_near(float c) {
    int i;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(i) : "v"(c));
    return static_cast<unsigned long long>(static_cast<long long>(i));
}

// With the warp, a brick's samples lie within the scan's displacement bound of
// it, so the displacement nodes around that box are copied to LDS once: the
// eight 16-byte node loads per sample kept the L1 busy longer than the atomics
// took.  Nodes in LDS are three planes of floats (x-neighbours are one
// 8-byte read).  Grids so fine that a brick's nodes exceed OWN_NODES take
// bp_brick_kernel's loads instead.
constexpr int OWN_NODES = 1320;

struct NodeBox {
    int x0, y0, z0;    // first node
    int nx, ny, nz;    // nodes
};

__device__ inline NodeBox brick_nodes(const WarpGrid &w, const RayGrid &g, int x0, int y0, int z0,
                                      int ex, int ey, int ez) {
    NodeBox b;
    const double M = walk_margin(w.margin, g.step, g.nx, g.ny, g.nz);
    node_range(x0, x0 + ex, M, g.nx, w.gx, w.sx, b.x0, b.nx);
    node_range(y0, y0 + ey, M, g.ny, w.gy, w.sy, b.y0, b.ny);
    node_range(z0, z0 + ez, M, g.nz, w.gz, w.sz, b.z0, b.nz);
    return b;
}

// Whether every brick's nodes fit in LDS (on each axis the most over the bricks).
bool brick_nodes_fit(const WarpGrid &w, const RayGrid &g, const BrickGrid &bg) {
    const double M = walk_margin(w.margin, g.step, g.nx, g.ny, g.nz);
    auto most = [&](int size, int bricks, int n, int gn, double scale) {
        int m = 0;
        for (int k = 0; k < bricks; ++k) {
            int first, count;
            node_range(k * size, k * size + std::min(size, n - k * size), M, n, gn, scale, first,
                       count);
            m = std::max(m, count);
        }
        return static_cast<long long>(m);
    };
    const long long mx = most(bg.bx, bg.nbx, g.nx, w.gx, w.sx);
    const long long my = most(bg.by, bg.nby, g.ny, w.gy, w.sy);
    const long long mz = most(bg.bz, bg.nbz, g.nz, w.gz, w.sz);
    return mx <= OWN_NODES && my <= OWN_NODES && mz <= OWN_NODES && mx * my * mz <= OWN_NODES;
}

// `displacement` from the nodes in LDS, with the same arithmetic.
__device__ __forceinline__ float3 lds_displacement(const float *__restrict__ nodes,
                                                   const NodeBox &nb, const WarpGrid &w, int kx,
                                                   float fx, int ky, float fy, int kz, float fz) {
    const float gx = fmaf(fx, w.fsx, static_cast<float>(kx) * w.fsx);
    const float gy = fmaf(fy, w.fsy, static_cast<float>(ky) * w.fsy);
    const float gz = fmaf(fz, w.fsz, static_cast<float>(kz) * w.fsz);
    float ax, ay, az;
    const int ix = node_corner(gx, w.gx, ax);
    const int iy = node_corner(gy, w.gy, ay);
    const int iz = node_corner(gz, w.gz, az);
    const int sy = nb.nx, sz = __mul24(nb.nx, nb.ny);
    const float *p = nodes + (__mul24(iz - nb.z0, sz) + __mul24(iy - nb.y0, sy) + (ix - nb.x0));
    float r[3];
#pragma unroll
    for (int q = 0; q < 3; ++q, p += OWN_NODES) {
        const float u000 = p[0], u001 = p[1], u010 = p[sy], u011 = p[sy + 1];
        const float u100 = p[sz], u101 = p[sz + 1], u110 = p[sz + sy], u111 = p[sz + sy + 1];
        const float a00 = fmaf(ax, u001 - u000, u000);
        const float a01 = fmaf(ax, u011 - u010, u010);
        const float a10 = fmaf(ax, u101 - u100, u100);
        const float a11 = fmaf(ax, u111 - u110, u110);
        const float b0 = fmaf(ay, a01 - a00, a00);
        const float b1 = fmaf(ay, a11 - a10, a10);
        r[q] = fmaf(az, b1 - b0, b0);
    }
    return make_float3(r[0], r[1], r[2]);
}

template <typename TS, int MODE, bool WARP>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4))) void bp_own_kernel(
    RayGrid g, WarpGrid w, const double *__restrict__ Pmat, const TS *__restrict__ sino,
    const float *__restrict__ rmax, BrickGrid bg) {
    constexpr int NT = 1024;
    __shared__ unsigned long long acc[OWN_CELLS];
    __shared__ RayRec rays[NT];
    __shared__ int4 box[OWN_BATCH];        // u0, v0, blocks per row, u1 - u0
    __shared__ int box_v1[OWN_BATCH];
    __shared__ int blk_end[OWN_BATCH];     // inclusive prefix of the block counts
    __shared__ int next_item;
    __shared__ float nodes[WARP ? 3 * OWN_NODES : 1];
    RayRec *const tabw = rays + (threadIdx.x & ~63);
    const int lane = threadIdx.x & 63;
    // ---- block -> (brick, projection chunk)
    const unsigned item = item_of(blockIdx.x, bg.run, bg.turn);
    if (item >= static_cast<unsigned>(bg.total)) return;
    const int br = static_cast<int>(item / static_cast<unsigned>(bg.chunks));
    const int chunk = static_cast<int>(item) - br * bg.chunks;
    const int row = br / bg.nbx, ibx = br - row * bg.nbx;
    const int ibz = row / bg.nby, iby = row - ibz * bg.nby;
    const int x0 = ibx * bg.bx, y0 = iby * bg.by, z0 = ibz * bg.bz;
    const int ex = min(bg.bx, g.nx - x0), ey = min(bg.by, g.ny - y0), ez = min(bg.bz, g.nz - z0);
    const double cmax =
        contribution_bound(g, (MODE == BP_ONES) ? 1.0 : static_cast<double>(*rmax), bg.wscale);
    // nothing to add, or NaN / Inf in the input (the finishing pass writes
    // NaN then), or a brick past the last lower corner n - 2
    if (!(cmax > 0.0 && cmax < __builtin_inf()) || x0 > g.nx - 2 || y0 > g.ny - 2 || z0 > g.nz - 2)
        return;
    for (int i = threadIdx.x; i < OWN_CELLS; i += NT) acc[i] = 0ull;
    NodeBox nb{0, 0, 0, 0, 0, 0};
    if (WARP) {
        nb = brick_nodes(w, g, x0, y0, z0, ex, ey, ez);
        const int count = nb.nx * nb.ny * nb.nz;   // at most OWN_NODES (launch_back)
        for (int i = threadIdx.x; i < count; i += NT) {
            const int z = i / (nb.nx * nb.ny), r = i - z * nb.nx * nb.ny;
            const int y = r / nb.nx, x = r - y * nb.nx;
            const float4 u = w.U[((nb.z0 + z) * w.gy + nb.y0 + y) * w.gx + nb.x0 + x];
            nodes[i] = u.x;
            nodes[OWN_NODES + i] = u.y;
            nodes[2 * OWN_NODES + i] = u.z;
        }
    }
    const double scale = uni(ldexp(1.0, uni(own_kexp(cmax, g, bg.cube_samples))));
    const double off[3] = {0.5 * (g.nx - 1), 0.5 * (g.ny - 1), 0.5 * (g.nz - 1)};
    // 1 / n_sub and the caller's factor (1 unless scaled; exact when a power of 2)
    const float inv_sub = uni(bg.wscale / static_cast<float>(g.n_sub));
    // largest side times 2^-22: four times the FP32 rounding error of a
    // coordinate of a ray's start (the ray-range estimate is widened by it)
    const float tol = uni(static_cast<float>(max(g.nx, max(g.ny, g.nz))) * 2.38418579e-7f);
    const float lo0[3] = {uni(x0 - tol), uni(y0 - tol), uni(z0 - tol)};
    const float hi0[3] = {uni(static_cast<float>(x0 + ex) + tol),
                          uni(static_cast<float>(y0 + ey) + tol),
                          uni(static_cast<float>(z0 + ez) + tol)};
    // With the warp, samples that can land in the brick start within [lo0 -
    // max tau U, hi0 - min tau U], U between the least and the largest of the
    // brick's nodes (a trilinear value lies between its nodes).  Bounded by
    // the whole field's largest component instead, a brick of the helical scan
    // walked about twice the samples it owned.
    float un[3] = {0.0f, 0.0f, 0.0f}, ux[3] = {0.0f, 0.0f, 0.0f};
    if (WARP) {
        __syncthreads();
        const int count = nb.nx * nb.ny * nb.nz;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float mn = __builtin_inff(), mxv = -__builtin_inff();
            for (int i = lane; i < count; i += 64) {
                mn = fminf(mn, nodes[a * OWN_NODES + i]);
                mxv = fmaxf(mxv, nodes[a * OWN_NODES + i]);
            }
            for (int o = 32; o > 0; o >>= 1) {
                mn = fminf(mn, __shfl_xor(mn, o, 64));
                mxv = fmaxf(mxv, __shfl_xor(mxv, o, 64));
            }
            un[a] = uni(mn);
            ux[a] = uni(mxv);
        }
    }
    // the range of starting positions for a sub-view (the allowance covers
    // the FP32 rounding of the displaced position)
    auto range = [&](float tau, float (&lo)[3], float (&hi)[3]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float p = tau * un[a], q = tau * ux[a];
            const float e = WARP ? WALK_ROUND * (1.0f + fabsf(p) + fabsf(q)) : 0.0f;
            lo[a] = lo0[a] - fmaxf(p, q) - e;
            hi[a] = hi0[a] - fminf(p, q) + e;
        }
    };
    // owned lower corners, relative to the brick: [0, e) on every axis, open
    // towards the faces, where the clamp moves corners into the brick
    const int mx = g.nx - 2 - x0, my = g.ny - 2 - y0, mz = g.nz - 2 - z0;
    const int ax = x0 == 0 ? INT_MIN : 0, bx = mx < ex ? INT_MAX : ex - 1;
    const int ay = y0 == 0 ? INT_MIN : 0, by = my < ey ? INT_MAX : ey - 1;
    const int az = z0 == 0 ? INT_MIN : 0, bz = mz < ez ? INT_MAX : ez - 1;
    // with the warp: owned corners [0, w), none past n - 2
    const int wx = min(ex, mx + 1), wy = min(ey, my + 1), wz = min(ez, mz + 1);
    const bool last = mx < ex || my < ey || mz < ez;   // it holds a corner n - 2
    // no clamp can act where the brick holds neither the first lower corner
    // nor the last
    const bool interior = x0 >= 1 && mx >= ex && y0 >= 1 && my >= ey && z0 >= 1 && mz >= ez;
    const int k_first = chunk * bg.views_per_chunk;
    const int n_pairs = (min(k_first + bg.views_per_chunk, g.n_views) - k_first) * g.n_sub;

    for (int q0 = 0; q0 < n_pairs; q0 += OWN_BATCH) {
        __syncthreads();   // the cells are cleared; the previous batch is done
        if (threadIdx.x < OWN_BATCH) {
            int nblk = 0;
            const int q = q0 + threadIdx.x;
            if (q < n_pairs) {
                const int k = k_first + q / g.n_sub;
                const int p = g.views ? g.views[k] : k;
                const int sv_idx = p * g.n_sub + q % g.n_sub;
                float lo[3], hi[3];
                range(static_cast<float>(g.tab[sv_idx].tau), lo, hi);
                const double plo[3] = {lo[0], lo[1], lo[2]}, phi[3] = {hi[0], hi[1], hi[2]};
                int u0 = 0, u1 = g.n_u - 1, v0 = 0, v1 = g.n_v - 1;
                if (!project_box(Pmat + 12 * static_cast<size_t>(sv_idx), plo, phi, off, g.n_u,
                                 g.n_v, u0, u1, v0, v1)) {
                    u0 = v0 = 0;
                    u1 = g.n_u - 1;
                    v1 = g.n_v - 1;
                }
                const int bu = (u1 - u0 + 8) >> 3;
                if (u0 <= u1 && v0 <= v1) nblk = bu * ((v1 - v0 + 8) >> 3);
                box[threadIdx.x] = make_int4(u0, v0, bu, u1);
                box_v1[threadIdx.x] = v1;
            }
            blk_end[threadIdx.x] = wave_inclusive_sum(nblk);
            if (threadIdx.x == 0) next_item = 0;
        }
        __syncthreads();
        const int items = uni(blk_end[OWN_BATCH - 1]);
        const int my_end = blk_end[lane];
        for (;;) {
            int item = 0;
            if (lane == 0) item = atomicAdd(&next_item, 1);
            item = uni(item);
            if (item >= items) break;
            // the pair: the first whose prefix passes the item
            const int qb = __popcll(__ballot(my_end <= item));
            const int first = qb > 0 ? __builtin_amdgcn_readlane(my_end, qb - 1) : 0;
            const int blk = item - first;
            const int4 bxq = box[qb];
            const int u0 = uni(bxq.x), v0 = uni(bxq.y), bu = uni(bxq.z), u1 = uni(bxq.w);
            const int v1 = uni(box_v1[qb]);
            const int q = q0 + qb;
            const int kq = q / g.n_sub;
            const int k = k_first + kq;
            const int p = uni(g.views ? g.views[k] : k);
            const SubView &sv = g.tab[p * g.n_sub + (q - kq * g.n_sub)];
            const float tau = WARP ? uni(static_cast<float>(sv.tau)) : 0.0f;
            float lo[3], hi[3];
            range(tau, lo, hi);
            const int bv = blk / bu;
            const int iv = v0 + bv * 8 + (lane >> 3);
            const int iu = u0 + (blk - bv * bu) * 8 + (lane & 7);
            // ---- this lane's ray: the samples the brick owns
            int len = 0, ib = 0;
            float wq = 0.0f;   // h r / n_sub in fixed-point units
            Ray r;
            r.qx = r.qy = r.qz = r.tx = r.ty = r.tz = 0;
            const float rv = (iu > u1 || iv > v1) ? 0.0f
                             : (MODE == BP_ONES) ? 1.0f
                                                 : ld(sino, (k * g.n_v + iv) * g.n_u + iu);
            if (rv != 0.0f && setup_ray(sv, static_cast<double>(iu), static_cast<double>(iv), g.nx,
                                        g.ny, g.nz, g.step, r)) {
                // sample indices i with b + i s inside [lo, hi] on every axis,
                // in FP32: a superset of the owned ones.  The FP32 start and
                // step put b + i s within 2.8 2^-24 max side of the
                // fixed-point position of sample i, and [lo, hi] is widened
                // by 4 2^-24 max side; the index estimate itself is a
                // reciprocal to 1 ulp and two roundings, under 4 2^-24 |t|,
                // inside the margin of 1/64 + 2^-20 |t| samples.  An axis the ray does not move
                // along (|s| under 1e-30: its samples drift by less than tol)
                // only decides whether the ray hits.
                float kmin = 0.0f, kmax = static_cast<float>(r.n - 1);
                const float bv3[3] = {r.bx, r.by, r.bz};
                const float sv3[3] = {r.fx, r.fy, r.fz};
                bool hit = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const bool flat = fabsf(sv3[a]) < 1e-30f;
                    const float inv = __builtin_amdgcn_rcpf(flat ? 1.0f : sv3[a]);
                    const float t1 = (lo[a] - bv3[a]) * inv, t2 = (hi[a] - bv3[a]) * inv;
                    const float tl = fminf(t1, t2), th = fmaxf(t1, t2);
                    const float ml = fmaf(fabsf(tl), 9.5367431640625e-7f, 0.015625f);
                    const float mh = fmaf(fabsf(th), 9.5367431640625e-7f, 0.015625f);
                    kmin = flat ? kmin : fmaxf(kmin, tl - ml);
                    kmax = flat ? kmax : fminf(kmax, th + mh);
                    hit &= !(flat & ((bv3[a] < lo[a]) | (bv3[a] > hi[a])));
                }
                // positions relative to the brick (of the volume with the
                // warp, whose lookup comes first)
                if (!WARP) {
                    r.qx -= static_cast<long long>(x0) << FX;
                    r.qy -= static_cast<long long>(y0) << FX;
                    r.qz -= static_cast<long long>(z0) << FX;
                }
                if (hit && kmin <= kmax) {
                    ib = max(static_cast<int>(ceilf(kmin)), 0);
                    int ie = min(static_cast<int>(floorf(kmax)), r.n - 1);
                    // the owned samples are a run (each coordinate is linear
                    // in the index): trim the superset's ends to it
                    auto owned = [&](int i) {
                        const int kx = static_cast<int>((r.qx + i * r.tx) >> FX);
                        const int ky = static_cast<int>((r.qy + i * r.ty) >> FX);
                        const int kz = static_cast<int>((r.qz + i * r.tz) >> FX);
                        return kx >= ax && kx <= bx && ky >= ay && ky <= by && kz >= az && kz <= bz;
                    };
                    if (!WARP) {
                        while (ib <= ie && !owned(ib)) ++ib;
                        while (ib <= ie && !owned(ie)) --ie;
                    }
                    len = max(ie - ib + 1, 0);
                    wq = static_cast<float>(static_cast<double>(r.h * rv * inv_sub) * scale);
                }
            }
            // ---- exclusive prefix of the segment lengths over the wave
            const int incl = wave_inclusive_sum(len);
            const int S = incl - len;
            const int T = __builtin_amdgcn_readlane(incl, 63);
            if (T == 0) continue;   // uniform over the wave
            const unsigned long long live = __ballot(len > 0);
            {
                // this lane's ray for the lanes that walk into it
                const unsigned long long later = lane < 63 ? (live & (~0ull << (lane + 1))) : 0ull;
                RayRec mine;
                mine.px = r.qx + static_cast<long long>(ib) * r.tx;
                mine.py = r.qy + static_cast<long long>(ib) * r.ty;
                mine.pz = r.qz + static_cast<long long>(ib) * r.tz;
                mine.tx = r.tx;
                mine.ty = r.ty;
                mine.tz = r.tz;
                mine.wq = wq;
                mine.end = incl;
                mine.next = later ? __ffsll(static_cast<long long>(later)) - 1 : lane;
                mine.pad = 0;
                wave_sync();   // the previous block's reads of the table are done
                tabw[lane] = mine;
                wave_sync();
            }
            // ---- lane takes samples [start, end) of the wave's T
            const int start = share(T, lane), end = share(T, lane + 1);
            int jr0 = 0;   // last ray with S_j <= start: it owns sample `start`
#pragma unroll
            for (int st = 32; st > 0; st >>= 1) {
                const int t = jr0 + st;
                if (__shfl(S, t, 64) <= start) jr0 = t;
            }
            // the lane's first ray may be entered mid-way: `start - S_j`
            // samples after its first sample in the brick
            const long long m = start - __shfl(S, jr0, 64);
            RayRec c = tabw[jr0];
            c.px += m * c.tx;
            c.py += m * c.ty;
            c.pz += m * c.tz;
            int pos = start;
            // Each lane keeps the eight corner sums of the cell its last
            // samples fell in and adds them to LDS when the next sample falls
            // in another cell (consecutive samples, half a voxel apart, often
            // share one) or could take a sum past a 32-bit integer.
            auto walk = [&](auto clamp_tag) {
                constexpr bool CLAMP = decltype(clamp_tag)::value;
                auto corner = [&](int &lx, int &ly, int &lz, float &fx, float &fy, float &fz) {
                    fx_split(c.px, lx, fx);
                    fx_split(c.py, ly, fy);
                    fx_split(c.pz, lz, fz);
                    if (CLAMP) {
                        auto clamp = [](int &l, float &f, int first, int last) {
                            if (l < first) {
                                l = first;
                                f = 0.0f;
                            }
                            if (l > last) {
                                l = last;
                                f = 1.0f;
                            }
                        };
                        clamp(lx, fx, -x0, mx);
                        clamp(ly, fy, -y0, my);
                        clamp(lz, fz, -z0, mz);
                    }
                    return __mul24(lz, OWN_SZ) + (__mul24(ly, OWN_SY) + lx);
                };
                int mcell;   // the first sample's cell
                {
                    int lx, ly, lz;
                    float fx, fy, fz;
                    mcell = corner(lx, ly, lz, fx, fy, fz);
                }
                float msum = 0.0f;
                float m0 = 0.0f, m1 = 0.0f, m2 = 0.0f, m3 = 0.0f;
                float m4 = 0.0f, m5 = 0.0f, m6 = 0.0f, m7 = 0.0f;
                auto flush = [&]() {
                    unsigned long long *const f0 = acc + mcell;
                    unsigned long long *const f1 = f0 + OWN_SZ;
                    atomicAdd(f0, to_fixed_near(m0));
                    atomicAdd(f0 + 1, to_fixed_near(m1));
                    atomicAdd(f0 + OWN_SY, to_fixed_near(m2));
                    atomicAdd(f0 + OWN_SY + 1, to_fixed_near(m3));
                    atomicAdd(f1, to_fixed_near(m4));
                    atomicAdd(f1 + 1, to_fixed_near(m5));
                    atomicAdd(f1 + OWN_SY, to_fixed_near(m6));
                    atomicAdd(f1 + OWN_SY + 1, to_fixed_near(m7));
                };
                auto sample = [&]() {
                    if (pos == c.end) c = tabw[c.next];   // enter the next ray
                    ++pos;
                    int lx, ly, lz;
                    float fx, fy, fz;
                    const int cell = corner(lx, ly, lz, fx, fy, fz);
                    c.px += c.tx;
                    c.py += c.ty;
                    c.pz += c.tz;
                    const float aw = fabsf(c.wq);
                    msum += aw;
                    if (!(cell == mcell && msum <= OWN_MERGE_LIMIT)) {
                        flush();
                        m0 = m1 = m2 = m3 = m4 = m5 = m6 = m7 = 0.0f;
                        msum = aw;
                        mcell = cell;
                    }
                    const float gx0 = 1.0f - fx;
                    const float gz1 = fz * c.wq, gz0 = c.wq - gz1;
                    const float w01 = gz0 * fy, w00 = gz0 - w01, w11 = gz1 * fy, w10 = gz1 - w11;
                    m0 = fmaf(w00, gx0, m0);
                    m1 = fmaf(w00, fx, m1);
                    m2 = fmaf(w01, gx0, m2);
                    m3 = fmaf(w01, fx, m3);
                    m4 = fmaf(w10, gx0, m4);
                    m5 = fmaf(w10, fx, m5);
                    m6 = fmaf(w11, gx0, m6);
                    m7 = fmaf(w11, fx, m7);
                };
                // every lane has T / 64 samples, some one more; a run of
                // merges ends after OWN_MERGE_MAX
                for (int left = T >> 6; left > 0; left -= OWN_MERGE_MAX) {
                    const int cnt = min(left, OWN_MERGE_MAX);
                    for (int it = 0; it < cnt; ++it) sample();
                    if (left > OWN_MERGE_MAX) {
                        flush();
                        m0 = m1 = m2 = m3 = m4 = m5 = m6 = m7 = 0.0f;
                        msum = 0.0f;
                    }
                }
                if (pos < end) sample();
                if (start < end) flush();
            };
            // With the warp a sample's corner, and whether the brick owns it, is
            // known only after the displacement lookup, and samples change
            // cells too often for the merge to pay: each is added at once.
            auto walk_warped = [&]() {
                auto sample = [&]() {
                    if (pos == c.end) c = tabw[c.next];   // enter the next ray
                    ++pos;
                    int kx, ky, kz;
                    float lx, ly, lz;
                    fx_split(c.px, kx, lx);
                    fx_split(c.py, ky, ly);
                    fx_split(c.pz, kz, lz);
                    c.px += c.tx;
                    c.py += c.ty;
                    c.pz += c.tz;
                    const float3 u = lds_displacement(nodes, nb, w, kx, lx, ky, ly, kz, lz);
                    lx = fmaf(tau, u.x, lx);
                    ly = fmaf(tau, u.y, ly);
                    lz = fmaf(tau, u.z, lz);
                    // lower corner relative to the brick; one outside the hull
                    // is owned by no brick
                    const float flx = floorf(lx), fly = floorf(ly), flz = floorf(lz);
                    int ox = kx + static_cast<int>(flx) - x0;
                    int oy = ky + static_cast<int>(fly) - y0;
                    int oz = kz + static_cast<int>(flz) - z0;
                    float fx = lx - flx, fy = ly - fly, fz = lz - flz;
                    if (last) {   // uniform: corner n - 1 with weight 0 beyond it
                        auto face = [](int &o, float &f, int m) {
                            if (o == m + 1 && f == 0.0f) {
                                o = m;
                                f = 1.0f;
                            }
                        };
                        face(ox, fx, mx);
                        face(oy, fy, my);
                        face(oz, fz, mz);
                    }
                    if (static_cast<uint32_t>(ox) >= static_cast<uint32_t>(wx) ||
                        static_cast<uint32_t>(oy) >= static_cast<uint32_t>(wy) ||
                        static_cast<uint32_t>(oz) >= static_cast<uint32_t>(wz))
                        return;
                    const float gx0 = 1.0f - fx;
                    const float gz1 = fz * c.wq, gz0 = c.wq - gz1;
                    const float w01 = gz0 * fy, w00 = gz0 - w01, w11 = gz1 * fy, w10 = gz1 - w11;
                    unsigned long long *const f0 =
                        acc + (__mul24(oz, OWN_SZ) + (__mul24(oy, OWN_SY) + ox));
                    unsigned long long *const f1 = f0 + OWN_SZ;
                    atomicAdd(f0, to_fixed_near(w00 * gx0));
                    atomicAdd(f0 + 1, to_fixed_near(w00 * fx));
                    atomicAdd(f0 + OWN_SY, to_fixed_near(w01 * gx0));
                    atomicAdd(f0 + OWN_SY + 1, to_fixed_near(w01 * fx));
                    atomicAdd(f1, to_fixed_near(w10 * gx0));
                    atomicAdd(f1 + 1, to_fixed_near(w10 * fx));
                    atomicAdd(f1 + OWN_SY, to_fixed_near(w11 * gx0));
                    atomicAdd(f1 + OWN_SY + 1, to_fixed_near(w11 * fx));
                };
                for (int it = T >> 6; it > 0; --it) sample();
                if (pos < end) sample();
            };
            if constexpr (WARP)
                walk_warped();
            else if (interior)
                walk(std::false_type{});
            else
                walk(std::true_type{});
        }
    }
    __syncthreads();
    // ---- add the brick's cells, halo included, into the integer volume
    for (int i = threadIdx.x; i < OWN_CELLS; i += NT) {
        const int lz = i / OWN_SZ;
        const int rem = i - lz * OWN_SZ;
        const int ly = rem / OWN_SY;
        const int lx = rem - ly * OWN_SY;
        const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
        const unsigned long long q = acc[i];
        if (q != 0ull && lx <= ex && ly <= ey && lz <= ez && gx < g.nx && gy < g.ny && gz < g.nz)
            atomicAdd(bg.acc64 + (static_cast<size_t>(gz) * g.ny + gy) * g.nx + gx, q);
    }
}

// vol[i] (+)= sum over chunks c of part[c][i], in chunk order.
__global__ __launch_bounds__(256) void sum_chunks_kernel(const float *__restrict__ part, int chunks,
                                                         size_t n, int accumulate,
                                                         float *__restrict__ vol) {
    const size_t stride = static_cast<size_t>(gridDim.x) * 256;
    for (size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride) {
        float s = accumulate ? vol[i] : 0.0f;
        for (int c = 0; c < chunks; ++c) s += part[static_cast<size_t>(c) * n + i];
        vol[i] = s;
    }
}

// Owner form: vol[i] = (vol[i] if accumulate) + acc64[i] 2^-kexp, NaN for a
// non-finite max |r|, with the exponent every brick used.
template <int MODE>
__global__ __launch_bounds__(256) void own_finish_kernel(const unsigned long long *__restrict__ acc64,
                                                         size_t n, const float *__restrict__ rmax,
                                                         RayGrid g, double cube_samples,
                                                         float wscale, int accumulate,
                                                         float *__restrict__ vol) {
    const double cmax =
        contribution_bound(g, MODE == BP_ONES ? 1.0 : static_cast<double>(*rmax), wscale);
    const bool bad = !(cmax < __builtin_inf());
    const double inv = (cmax > 0.0 && !bad) ? ldexp(1.0, -own_kexp(cmax, g, cube_samples)) : 0.0;
    const size_t stride = static_cast<size_t>(gridDim.x) * 256;
    size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    auto put = [&](size_t j, unsigned long long a, float old) {
        const float v = bad ? __builtin_nanf("")
                            : static_cast<float>(static_cast<double>(static_cast<long long>(a)) * inv);
        vol[j] = accumulate ? old + v : v;
    };
    for (; i + 3 * stride < n; i += 4 * stride) {
        unsigned long long a[4];
        float old[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            a[k] = acc64[i + k * stride];
            old[k] = accumulate ? vol[i + k * stride] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) put(i + k * stride, a[k], old[k]);
    }
    for (; i < n; i += stride) put(i, acc64[i], accumulate ? vol[i] : 0.0f);
}

BrickGrid plan_bricks(const RayGrid &g, int cap_chunks, bool own) {
    BrickGrid bg;
    bg.bx = min(own ? OWN_X : BRICK_X, g.nx);
    bg.by = min(own ? OWN_Y : BRICK_Y, g.ny);
    bg.bz = min(own ? OWN_Z : BRICK_Z, g.nz);
    bg.nbx = (g.nx + bg.bx - 1) / bg.bx;
    bg.nby = (g.ny + bg.by - 1) / bg.by;
    bg.nbz = (g.nz + bg.bz - 1) / bg.bz;
    const long long bricks = static_cast<long long>(bg.nbx) * bg.nby * bg.nbz;
    // enough workgroups to fill 256 CUs a few times over, at least 4 views each
    long long want = (2048 + bricks - 1) / bricks;
    const long long max_chunks = (g.n_views + 3) / 4;
    if (want > max_chunks) want = max_chunks;
    if (cap_chunks > 0 && want > cap_chunks) want = cap_chunks;
    if (want < 1) want = 1;
    bg.views_per_chunk = static_cast<int>((g.n_views + want - 1) / want);
    bg.chunks = (g.n_views + bg.views_per_chunk - 1) / bg.views_per_chunk;
    bg.total = static_cast<int>(bricks * bg.chunks);
    // h >= step / 2 whenever a ray has two samples, and a side-2 cube holds a
    // chord of at most 2 sqrt(3)
    bg.cube_samples = floor(4.0 * 1.7320508075688772 / g.step) + 1.0;
    bg.run = 1;
    bg.turn = 0;
    bg.partials = nullptr;
    bg.acc64 = nullptr;
    bg.accumulate = 0;
    bg.wscale = 1.0f;
    return bg;
}

}  // namespace

size_t back_scratch_bytes(const RayGrid &g, int max_chunks, bool direct) {
    if (g.n_views <= 0) return 0;
    const size_t nvol = static_cast<size_t>(g.nx) * g.ny * g.nz;
    if (!direct) return sizeof(unsigned long long) * nvol;
    const BrickGrid bg = plan_bricks(g, max_chunks, false);
    return bg.chunks > 1 ? sizeof(float) * static_cast<size_t>(bg.chunks) * nvol : 0;
}

hipError_t launch_back(const RayGrid &g, const WarpGrid &w, const double *Pmat, const void *sino,
                       int sino_dtype, float *vol, int accumulate, int mode, float *scratch,
                       void *work, hipStream_t stream, float scale, int max_chunks, bool direct) {
    if (g.n_views <= 0) return hipSuccess;
    BrickGrid bg = plan_bricks(g, direct ? max_chunks : 0, !direct);
    bg.accumulate = accumulate;
    bg.wscale = scale;
    const size_t nvol = static_cast<size_t>(g.nx) * g.ny * g.nz;
    if (direct) {
        bg.partials = static_cast<float *>(work);
        if (bg.chunks > 1 && !work) return hipErrorInvalidValue;
    } else {
        bg.acc64 = static_cast<unsigned long long *>(work);
        if (!work) return hipErrorInvalidValue;
        hipError_t e = launch_fill_zero(work, sizeof(unsigned long long) * nvol, stream);
        if (e != hipSuccess) return e;
    }
    const int per = (bg.total + N_XCD - 1) / N_XCD;
    const bool wp = w.U != nullptr;
    const dim3 grid(static_cast<unsigned>(per * N_XCD));
    const dim3 block(static_cast<unsigned>(wp ? bp_threads<true>() : bp_threads<false>()));
    const bool nodes_fit = wp && !direct && brick_nodes_fit(w, g, bg);
    const BrickOrder order = brick_order(bg.nby * bg.nbz, bg.nbx, bg.chunks);
    bg.run = order.run;
    bg.turn = order.turn;
    const dim3 own_grid(static_cast<unsigned>(order.blocks));
    const size_t shmem = 0;   // the brick is static LDS
    size_t fblocks = (nvol + 255) / 256;
    if (fblocks > 65536) fblocks = 65536;
    // own_finish_kernel takes four voxels per pass and its workgroups stay: the
    // exponent's logarithm is taken once per workgroup, not once per 256 voxels
    // (256^3: 98 -> 35 us)
    const size_t oblocks = std::min<size_t>((nvol + 1023) / 1024, 2048);
    // after the bricks: the direct form's chunk partials summed in chunk
    // order, or the owner form's integer volume scaled into vol
    auto finish = [&](int m) -> hipError_t {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (!direct) {
            if (m == BP_ONES)
                hipLaunchKernelGGL(own_finish_kernel<BP_ONES>, dim3(static_cast<unsigned>(oblocks)),
                                   dim3(256), 0, stream, bg.acc64, nvol, scratch, g,
                                   bg.cube_samples, scale, accumulate, vol);
            else
                hipLaunchKernelGGL(own_finish_kernel<BP_PLAIN>,
                                   dim3(static_cast<unsigned>(oblocks)), dim3(256), 0, stream,
                                   bg.acc64, nvol, scratch, g, bg.cube_samples, scale, accumulate,
                                   vol);
            return hipGetLastError();
        }
        if (bg.chunks <= 1) return hipSuccess;
        hipLaunchKernelGGL(sum_chunks_kernel, dim3(static_cast<unsigned>(fblocks)), dim3(256), 0,
                           stream, bg.partials, bg.chunks, nvol, accumulate, vol);
        return hipGetLastError();
    };
#define CTREX_BP_LAUNCH(T, M, SP, RM)                                                           \
    {                                                                                           \
        if (direct) {                                                                           \
            if (wp)                                                                             \
                hipLaunchKernelGGL((bp_brick_kernel<T, M, true, false>), grid, block, shmem,    \
                                   stream, g, w, Pmat, SP, RM, vol, bg);                        \
            else                                                                                \
                hipLaunchKernelGGL((bp_brick_kernel<T, M, false, false>), grid, block, shmem,   \
                                   stream, g, w, Pmat, SP, RM, vol, bg);                        \
        } else {                                                                                \
            if (wp && !nodes_fit)                                                               \
                hipLaunchKernelGGL((bp_brick_kernel<T, M, true, true>), grid, block, shmem,     \
                                   stream, g, w, Pmat, SP, RM, vol, bg);                        \
            else if (wp)                                                                        \
                hipLaunchKernelGGL((bp_own_kernel<T, M, true>), own_grid, dim3(1024), 0,        \
                                   stream, g, w, Pmat, SP, RM, bg);                             \
            else                                                                                \
                hipLaunchKernelGGL((bp_own_kernel<T, M, false>), own_grid, dim3(1024), 0,       \
                                   stream, g, w, Pmat, SP, RM, bg);                             \
        }                                                                                       \
        return finish(M);                                                                       \
    }
    if (mode == BP_ONES) CTREX_BP_LAUNCH(float, BP_ONES, nullptr, nullptr)
    // max |r| over the sinogram sets the fixed-point scale
    const size_t n_sino = static_cast<size_t>(g.n_views) * g.n_u * g.n_v;
    hipError_t e = launch_max_abs(sino, sino_dtype, n_sino, scratch, stream);
    if (e != hipSuccess) return e;
    switch (sino_dtype) {
        case F32: CTREX_BP_LAUNCH(float, BP_PLAIN, static_cast<const float *>(sino), scratch)
        case BF16: CTREX_BP_LAUNCH(bf16_t, BP_PLAIN, static_cast<const bf16_t *>(sino), scratch)
        case F16: CTREX_BP_LAUNCH(_Float16, BP_PLAIN, static_cast<const _Float16 *>(sino), scratch)
        default: return hipErrorInvalidValue;
    }
#undef CTREX_BP_LAUNCH
}

}  // namespace ctrex
