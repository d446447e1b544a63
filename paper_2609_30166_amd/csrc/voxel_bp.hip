// The paper's voxel-driven backprojector (Sec. 4.1, backprojection operator):
// every voxel centre is projected through each selected view matrix onto its
// detector image and the image is sampled bilinearly there (pixel centres at
// integer (u, v), zero beyond the border), sub-views averaged:
//     z_j (+)= (1 / n_sub) sum_{p, s} r_p(u_{p,s}(X_j), v_{p,s}(X_j)).
// It is not the transpose of the ray-driven projector; SIRT pairs it with
// C = 1 / (B 1).
//
// Gather form: one thread owns a column of KZ voxels along z and keeps their
// sums in FP64 registers over all views, then writes each voxel once, so the
// result is deterministic and needs no atomics.  A workgroup is a 16 x 16
// (x, y) patch of such columns.  The view matrix and the view index are
// wave-uniform (scalar loads).
//
// Projection arithmetic: per (thread, view) the column's top voxel is
// projected in FP64 (a, b, w) = P (X, 1).  When the depth row of P has no
// z coefficient (every circular orbit about z), w is the same for the whole
// column and u_k = u_0 + k P[0][2] / w: the integer parts of u_0 and v_0 are
// taken in FP64 and the remainders plus k du in FP32 (within a footprint under
// 49 pixels, so positions stay within about 3e-6 pixel).  Otherwise, or when the
// column's numbers are huge, each voxel is projected in FP64 on its own.
//
// Detector lookups (vbp_tile_kernel): four global loads per voxel and view,
// two to an instruction, kept the L1 busy at one access per lane quad and
// clock, whatever the path's VALU count.  So each wave bounds one view's
// footprint of the patch and copies it to LDS (zeros outside the image, which
// also makes the borders need no code), and all four waves then sample the
// four footprints: two LDS reads per voxel and 13 VALU instructions, the bound.
// 360 views of 384^2 at 256^3: 7.36 -> 3.59 ms (without the footprints, but
// with a path of 13 instructions per voxel for columns inside the image: 6.2).
// Four waves per SIMD: at 3 (no spills) 4.2 ms, at 5 (spills) 14.  A view
// whose footprint does not fit, or whose depth row has a z coefficient, is
// sampled from global memory with the border handling; geometries in which more
// than a quarter are take vbp_kernel, which does nothing else (footprint_column).

#include "ray_common.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace ctrex {
namespace {

constexpr int VB_TX = 16;
constexpr int VB_TY = 16;
constexpr int VB_THREADS = VB_TX * VB_TY;
constexpr int FT_U = 49, FT_V = 36;    // largest footprint; an odd row stride
constexpr int FT_N = VB_THREADS / 64;  // views per round, one per wave
// Footprints are bounded in FP32, whose spacing is 1/128 below pixel 2^17; one
// that starts further out than this is sampled from memory, where columns come
// from FP64.
constexpr float FAR_PIXEL = 131072.0f - 64.0f;

typedef float f32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));

// Detector columns (c, c + 1) at element `off` of an image.  The byte offset
// is formed in 32 bits (images hold fewer than 2^30 pixels) and added to the
// wave-uniform image base, so the loads take the scalar-base form.
template <typename TS>
__device__ __forceinline__ const TS *at(const TS *img, unsigned off) {
    return reinterpret_cast<const TS *>(reinterpret_cast<const char *>(img) +
                                        off * static_cast<unsigned>(sizeof(TS)));
}
template <typename TS>
__device__ __forceinline__ float2 row_pair(const TS *__restrict__ img, unsigned off) {
    const TS *q = at(img, off);
    return make_float2(dev::ld(q, 0), dev::ld(q, 1));
}
template <>
__device__ __forceinline__ float2 row_pair<float>(const float *__restrict__ img, unsigned off) {
    const f32x2_a4 p = *reinterpret_cast<const f32x2_a4 *>(at(img, off));
    return make_float2(p.x, p.y);
}

// Bilinear sample of a detector image at (iu + fu, iv + fv) with zero
// outside, for iu in [-1, nu - 1] and iv in [-1, nv - 1] (nu, nv >= 2).  The
// loads stay inside the image for any (iu, iv): the column pair starts at
// c = clamp(iu, 0, nu - 2) and both rows are clamped to [0, nv - 1]; the
// weights (ea, eb) of the pair's two columns are those of columns iu and
// iu + 1 moved to where they sit in the pair (0 for a column outside).
// ONES: the sum of the in-image weights (no loads).
template <typename TS, bool ONES>
__device__ __forceinline__ float bilinear(const TS *__restrict__ img, int nu, int nv, int iu,
                                          int iv, float fu, float fv) {
    const float wt = iv >= 0 ? 1.0f - fv : 0.0f;
    const float wb = iv < nv - 1 ? fv : 0.0f;
    // iu == -1: pair (0, 1) holds column iu + 1 first; iu == nu - 1: pair
    // (nu - 2, nu - 1) holds column iu second
    const float ea = iu < 0 ? fu : (iu == nu - 1 ? 0.0f : 1.0f - fu);
    const float eb = iu < 0 ? 0.0f : (iu == nu - 1 ? 1.0f - fu : fu);
    if (ONES) return (ea + eb) * (wt + wb);
    const unsigned c = static_cast<unsigned>(min(max(iu, 0), nu - 2));
    const unsigned r0 = static_cast<unsigned>(min(max(iv, 0), nv - 1));
    const unsigned r1 = static_cast<unsigned>(min(max(iv + 1, 0), nv - 1));
    // 24-bit products (full-rate multiply; detector sides are below 2^24)
    const float2 p0 = row_pair(img, __umul24(r0, static_cast<unsigned>(nu)) + c);
    const float2 p1 = row_pair(img, __umul24(r1, static_cast<unsigned>(nu)) + c);
    return wt * fmaf(ea, p0.x, eb * p0.y) + wb * fmaf(ea, p1.x, eb * p1.y);
}

// Contribution at FP64 detector position (u, v), or 0 outside (-1, nu) x (-1, nv).
template <typename TS, bool ONES>
__device__ __forceinline__ float sample_at(const TS *__restrict__ img, int nu, int nv, double u,
                                           double v) {
    if (!(u > -1.0 && u < nu && v > -1.0 && v < nv)) return 0.0f;
    const double fu = floor(u), fv = floor(v);
    return bilinear<TS, ONES>(img, nu, nv, static_cast<int>(fu), static_cast<int>(fv),
                              static_cast<float>(u - fu), static_cast<float>(v - fv));
}

// Hardware hands workgroup b to XCD b mod 8; give every XCD one contiguous
// run of tiles (tiles enumerate z fastest, so an XCD's concurrent workgroups
// are z-neighbours whose detector footprints share rows).
__device__ __forceinline__ int xcd_tile(int b, int n_tiles) {
    const int q = n_tiles / N_XCD, rem = n_tiles % N_XCD;
    const int x = b % N_XCD;
    return x * q + min(x, rem) + b / N_XCD;
}

// The voxel column of one thread: top centre, step along z, voxels inside.
struct Column {
    double X, Y, Z0, sz;
    int kn;
};

__host__ __device__ __forceinline__ Column column_of(const VoxelGrid &vg, int ix, int iy, int z0, int ny,
                                            int nx, int nz, int kz) {
    Column c;
    c.kn = min(kz, nz - z0);
    if (vg.cyl) {
        // polar grid: ring ix, angle iy, slice z0
        const double r = (ix + 0.5) * vg.dr;
        const double phi = 6.283185307179586476925287 * iy / ny;
        double sn, cs;
        sincos(phi, &sn, &cs);
        c.X = r * cs;
        c.Y = r * sn;
        c.Z0 = (z0 - 0.5 * (nz - 1)) * vg.dz;
        c.sz = vg.dz;
    } else {
        c.X = ix - 0.5 * (nx - 1);
        c.Y = iy - 0.5 * (ny - 1);
        c.Z0 = z0 - 0.5 * (nz - 1);
        c.sz = 1.0;
    }
    return c;
}

// Box around the (x, y) positions of a patch's voxel centres.
struct PatchBox {
    double xa, xb, ya, yb;
};

__host__ __device__ __forceinline__ PatchBox patch_box(const VoxelGrid &vg, int tx, int ty, int nx,
                                                       int ny, int nz) {
    const int x1 = min(tx * VB_TX + VB_TX - 1, nx - 1), y1 = min(ty * VB_TY + VB_TY - 1, ny - 1);
    const Column c0 = column_of(vg, tx * VB_TX, ty * VB_TY, 0, ny, nx, nz, 1);
    const Column c1 = column_of(vg, x1, ty * VB_TY, 0, ny, nx, nz, 1);
    const Column c2 = column_of(vg, tx * VB_TX, y1, 0, ny, nx, nz, 1);
    const Column c3 = column_of(vg, x1, y1, 0, ny, nx, nz, 1);
    PatchBox b;
    b.xa = fmin(fmin(c0.X, c1.X), fmin(c2.X, c3.X));
    b.xb = fmax(fmax(c0.X, c1.X), fmax(c2.X, c3.X));
    b.ya = fmin(fmin(c0.Y, c1.Y), fmin(c2.Y, c3.Y));
    b.yb = fmax(fmax(c0.Y, c1.Y), fmax(c2.Y, c3.Y));
    if (vg.cyl) {
        // the outer arc bulges past its chord by r (1 - cos(half angle))
        const double r = (x1 + 0.5) * vg.dr;
        const double half = 3.14159265358979323846 * (y1 - ty * VB_TY) / ny;
        const double e = half < 1.5707963 ? r * (1.0 - cos(half)) + 1e-9 * r : 2.0 * r;
        b.xa -= e;
        b.xb += e;
        b.ya -= e;
        b.yb += e;
    }
    return b;
}

// acc[k] += the samples of one sub-view's image at the column's voxels.
template <typename TS, bool ONES, int KZ>
__device__ __forceinline__ void add_view(const Column &c, const double *__restrict__ M,
                                         const TS *__restrict__ img, int nu, int nv,
                                         double (&acc)[KZ]) {
    const double a0 = fma(M[0], c.X, fma(M[1], c.Y, fma(M[2], c.Z0, M[3])));
    const double b0 = fma(M[4], c.X, fma(M[5], c.Y, fma(M[6], c.Z0, M[7])));
    const double w0 = fma(M[8], c.X, fma(M[9], c.Y, fma(M[10], c.Z0, M[11])));
    // change of (a, b, w) per voxel down the column
    const double ca = M[2] * c.sz, cb = M[6] * c.sz, cw = M[10] * c.sz;
    bool fast = cw == 0.0 && w0 != 0.0;
    double u0 = 0.0, v0 = 0.0, du = 0.0, dv = 0.0;
    if (fast) {
        const double r = 1.0 / w0;
        u0 = a0 * r;
        v0 = b0 * r;
        du = ca * r;
        dv = cb * r;
        fast = fabs(u0) < 16777216.0 && fabs(v0) < 16777216.0 && fabs(du) < 65536.0 &&
               fabs(dv) < 65536.0;
    }
    if (fast) {
        // the column's u and v run linearly in k: skip it if it misses
        const double ue = fma(c.kn - 1.0, du, u0), ve = fma(c.kn - 1.0, dv, v0);
        if (!(fmax(u0, ue) > -1.0 && fmin(u0, ue) < nu && fmax(v0, ve) > -1.0 &&
              fmin(v0, ve) < nv))
            return;
        const double fu0 = floor(u0), fv0 = floor(v0);
        const int iu0 = static_cast<int>(fu0), iv0 = static_cast<int>(fv0);
        const float ru = static_cast<float>(u0 - fu0), rv = static_cast<float>(v0 - fv0);
        const float duf = static_cast<float>(du), dvf = static_cast<float>(dv);
        // branch-free over the column: every voxel's loads are issued
        // (at clamped, in-image addresses) before any is consumed, and
        // voxels off the detector or past the volume are selected out
#pragma unroll
        for (int k = 0; k < KZ; ++k) {
            const float uf = fmaf(static_cast<float>(k), duf, ru);
            const float vf = fmaf(static_cast<float>(k), dvf, rv);
            const int iu = iu0 + static_cast<int>(floorf(uf));
            const int iv = iv0 + static_cast<int>(floorf(vf));
            const bool in = k < c.kn &&
                            static_cast<unsigned>(iu + 1) <= static_cast<unsigned>(nu) &&
                            static_cast<unsigned>(iv + 1) <= static_cast<unsigned>(nv);
            const float val = bilinear<TS, ONES>(img, nu, nv, iu, iv, __builtin_amdgcn_fractf(uf),
                                                 __builtin_amdgcn_fractf(vf));
            acc[k] += in ? val : 0.0f;
        }
    } else {
#pragma unroll
        for (int k = 0; k < KZ; ++k) {
            if (k >= c.kn) break;
            const double w = fma(static_cast<double>(k), cw, w0);
            if (w == 0.0) continue;
            const double u = fma(static_cast<double>(k), ca, a0) / w;
            const double v = fma(static_cast<double>(k), cb, b0) / w;
            acc[k] += sample_at<TS, ONES>(img, nu, nv, u, v);
        }
    }
}

template <int KZ>
__device__ __forceinline__ void store_column(const double (&acc)[KZ], int n_sub, int kn, int ix,
                                             int iy, int z0, int nx, int ny, int accumulate,
                                             float *__restrict__ vol) {
    const double inv_sub = 1.0 / n_sub;
    const size_t col = static_cast<size_t>(iy) * nx + ix;
    const size_t plane = static_cast<size_t>(nx) * ny;
#pragma unroll
    for (int k = 0; k < KZ; ++k) {
        if (k >= kn) break;
        float *dst = vol + (static_cast<size_t>(z0) + k) * plane + col;
        const float add = static_cast<float>(acc[k] * inv_sub);
        *dst = accumulate ? *dst + add : add;
    }
}

// Every view through add_view, without barriers or LDS: B 1 (ONES: no image to
// read), and geometries whose views mostly have no footprint.
template <typename TS, bool ONES, int KZ>
__global__ __launch_bounds__(VB_THREADS) void vbp_kernel(
    const double *__restrict__ Pm, const int *__restrict__ views, int n_views, int n_sub, int nu,
    int nv, int nx, int ny, int nz, int tiles_y, int tiles_z, const TS *__restrict__ sino,
    float *__restrict__ vol, int accumulate, VoxelGrid vg) {
    int t = xcd_tile(blockIdx.x, gridDim.x);
    const int tz = t % tiles_z;
    t /= tiles_z;
    const int ty = t % tiles_y;
    const int tx = t / tiles_y;
    const int ix = tx * VB_TX + (threadIdx.x & (VB_TX - 1));
    const int iy = ty * VB_TY + (threadIdx.x / VB_TX);
    if (ix >= nx || iy >= ny) return;  // no barriers below
    const int z0 = tz * KZ;
    const Column c = column_of(vg, ix, iy, z0, ny, nx, nz, KZ);
    const size_t img_px = static_cast<size_t>(nu) * nv;
    double acc[KZ];
#pragma unroll
    for (int k = 0; k < KZ; ++k) acc[k] = 0.0;
    for (int j = 0; j < n_views; ++j) {
        const int p = views ? views[j] : j;
        const TS *img = ONES ? nullptr : sino + j * img_px;
        for (int s = 0; s < n_sub; ++s)
            add_view<TS, ONES, KZ>(c, Pm + 12 * (static_cast<size_t>(p) * n_sub + s), img, nu, nv,
                                   acc);
    }
    store_column<KZ>(acc, n_sub, c.kn, ix, iy, z0, nx, ny, accumulate, vol);
}

// Minimum over each group of 8 consecutive lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_min(float v) {
    const int x = __float_as_int(v);
    return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ float min8(float v) {
    v = dpp_min<0xB1>(v);           // lane ^ 1
    v = dpp_min<0x4E>(v);           // lane ^ 2
    return dpp_min<0x141>(v);       // mirrored within 8 lanes
}

// floor of a float below 2^31 in magnitude as an integer
__device__ __forceinline__ int floor_int(float x) {
    int i;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
    return i;
}

// One view's footprint in LDS: image column u0, row v0 of its first element;
// mode 0: the patch misses the image, 1: in LDS, 2: sampled from memory.
struct Footprint {
    int u0, v0, mode, pad;
};

template <typename TS, int KZ>
__global__ __launch_bounds__(VB_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) void
vbp_tile_kernel(
    const double *__restrict__ Pm, const int *__restrict__ views, int n_views, int n_sub, int nu,
    int nv, int nx, int ny, int nz, int tiles_y, int tiles_z, const TS *__restrict__ sino,
    float *__restrict__ vol, int accumulate, VoxelGrid vg) {
    __shared__ float tile[FT_N][FT_U * FT_V];
    __shared__ Footprint foot[FT_N];
    int t = xcd_tile(blockIdx.x, gridDim.x);
    const int tz = t % tiles_z;
    t /= tiles_z;
    const int ty = t % tiles_y;
    const int tx = t / tiles_y;
    // threads past the volume's edge repeat its last column and store nothing
    const int gx = tx * VB_TX + (threadIdx.x & (VB_TX - 1));
    const int gy = ty * VB_TY + (threadIdx.x / VB_TX);
    const int ix = min(gx, nx - 1), iy = min(gy, ny - 1);
    const int z0 = tz * KZ;
    const Column c = column_of(vg, ix, iy, z0, ny, nx, nz, KZ);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    // corner (lane & 7) of a box around the patch's voxel centres, over the
    // columns' full KZ voxels
    const PatchBox pb = patch_box(vg, tx, ty, nx, ny, nz);
    const double bx = (lane & 1) ? pb.xb : pb.xa;
    const double by = (lane & 2) ? pb.yb : pb.ya;
    const double bz = c.Z0 + ((lane & 4) ? (KZ - 1) * c.sz : 0.0);
    const size_t img_px = static_cast<size_t>(nu) * nv;
    const int n_pairs = n_views * n_sub;
    double acc[KZ];
#pragma unroll
    for (int k = 0; k < KZ; ++k) acc[k] = 0.0;

    for (int q0 = 0; q0 < n_pairs; q0 += FT_N) {
        // ---- this wave's view: bound the footprint and copy it
        const int q = q0 + wave;
        if (q < n_pairs) {
            const int j = q / n_sub;
            const int p = views ? views[j] : j;
            const double *M = Pm + 12 * (static_cast<size_t>(p) * n_sub + (q - j * n_sub));
            const double a = fma(M[0], bx, fma(M[1], by, fma(M[2], bz, M[3])));
            const double b = fma(M[4], bx, fma(M[5], by, fma(M[6], bz, M[7])));
            const double w = fma(M[8], bx, fma(M[9], by, fma(M[10], bz, M[11])));
            const unsigned long long pos = __ballot(w > 0.0), neg = __ballot(w < 0.0);
            const double r = 1.0 / w;
            // 0.01 pixel covers the FP32 rounding here (two of 1/256 at most up
            // to FAR_PIXEL and a footprint) and of the samples' offsets within a column
            const float u = static_cast<float>(a * r), v = static_cast<float>(b * r);
            const float ua = floorf(min8(u) - 0.01f), ub = floorf(0.01f - min8(-u)) + 1.0f;
            const float va = floorf(min8(v) - 0.01f), vb = floorf(0.01f - min8(-v)) + 1.0f;
            // column steps along u and v are linear in k only without a z
            // coefficient in the depth row; the corners bound the patch only
            // if it lies on one side of the source plane
            const bool fits = M[10] == 0.0 && (~pos == 0 || ~neg == 0) && ub - ua < FT_U &&
                              vb - va < FT_V && fabsf(ua) < FAR_PIXEL && fabsf(va) < FAR_PIXEL;
            Footprint f{0, 0, 2, 0};
            if (fits) {   // uniform
                f.u0 = __builtin_amdgcn_readfirstlane(static_cast<int>(ua));
                f.v0 = __builtin_amdgcn_readfirstlane(static_cast<int>(va));
                const int fw = __builtin_amdgcn_readfirstlane(static_cast<int>(ub - ua)) + 1;
                const int fh = __builtin_amdgcn_readfirstlane(static_cast<int>(vb - va)) + 1;
                f.mode = f.u0 < nu && f.u0 + fw > 0 && f.v0 < nv && f.v0 + fh > 0;
                if (f.mode) {
                    const TS *img = sino + j * img_px;
                    float *dst = tile[wave];
                    // 32 columns of two rows per step, or 64 of one
                    const bool two = fw <= 32;
                    const int cu = two ? lane & 31 : lane, cr = two ? lane >> 5 : 0;
                    const int rs = two ? 2 : 1;
                    const int gu = f.u0 + cu;
                    const bool cin = cu < fw && gu >= 0 && gu < nu;
                    constexpr int IN_FLIGHT = 6;
                    // rows [ra, rb) lie in the image
                    const int ra = cin ? max(0, -f.v0) : fh, rb = min(fh, nv - f.v0);
                    int o = (f.v0 + cr) * nu + gu;
                    int d = cr * FT_U + cu;
                    for (int row = cr; row < fh; row += IN_FLIGHT * rs) {
                        float px[IN_FLIGHT];
#pragma unroll
                        for (int i = 0; i < IN_FLIGHT; ++i) {
                            px[i] = 0.0f;
                            if (row + i * rs >= ra && row + i * rs < rb)
                                px[i] = dev::ld(img, o + i * rs * nu);
                        }
                        o += IN_FLIGHT * rs * nu;
#pragma unroll
                        for (int i = 0; i < IN_FLIGHT; ++i)
                            if (cu < fw && row + i * rs < fh) dst[d + i * rs * FT_U] = px[i];
                        d += IN_FLIGHT * rs * FT_U;
                    }
                }
            }
            if (lane == 0) foot[wave] = f;
        }
        __syncthreads();
        // ---- all columns sample the round's views
        const int nq = min(FT_N, n_pairs - q0);
        for (int i = 0; i < nq; ++i) {
            const int mode = __builtin_amdgcn_readfirstlane(foot[i].mode);
            if (mode == 0) continue;
            const int j = (q0 + i) / n_sub;
            const int p = views ? views[j] : j;
            const double *M = Pm + 12 * (static_cast<size_t>(p) * n_sub + (q0 + i - j * n_sub));
            if (mode == 2) {
                add_view<TS, false, KZ>(c, M, sino + j * img_px, nu, nv, acc);
                continue;
            }
            const double a0 = fma(M[0], c.X, fma(M[1], c.Y, fma(M[2], c.Z0, M[3])));
            const double b0 = fma(M[4], c.X, fma(M[5], c.Y, fma(M[6], c.Z0, M[7])));
            const double r = 1.0 / fma(M[8], c.X, fma(M[9], c.Y, fma(M[10], c.Z0, M[11])));
            const double u0 = a0 * r, v0 = b0 * r;
            const double fu0 = floor(u0), fv0 = floor(v0);
            const float ru = static_cast<float>(u0 - fu0), rv = static_cast<float>(v0 - fv0);
            const float dvf = static_cast<float>(M[6] * c.sz * r);
            const int rel = (static_cast<int>(fv0) - __builtin_amdgcn_readfirstlane(foot[i].v0)) * FT_U +
                            static_cast<int>(fu0) - __builtin_amdgcn_readfirstlane(foot[i].u0);
            const float *const img = tile[i] + rel;
            if (M[2] == 0.0) {   // uniform: the column stays at one u
                const float eb = ru, ea = 1.0f - ru;
#pragma unroll
                for (int k = 0; k < KZ; ++k) {
                    const float vf = fmaf(static_cast<float>(k), dvf, rv);
                    const float *s = img + __mul24(floor_int(vf), FT_U);
                    const float fv = __builtin_amdgcn_fractf(vf);
                    const float h0 = fmaf(ea, s[0], eb * s[1]);
                    const float h1 = fmaf(ea, s[FT_U], eb * s[FT_U + 1]);
                    acc[k] += fmaf(1.0f - fv, h0, fv * h1);
                }
            } else {
                const float duf = static_cast<float>(M[2] * c.sz * r);
#pragma unroll
                for (int k = 0; k < KZ; ++k) {
                    const float uf = fmaf(static_cast<float>(k), duf, ru);
                    const float vf = fmaf(static_cast<float>(k), dvf, rv);
                    const float *s = img + (__mul24(floor_int(vf), FT_U) + floor_int(uf));
                    const float eb = __builtin_amdgcn_fractf(uf), ea = 1.0f - eb;
                    const float fv = __builtin_amdgcn_fractf(vf);
                    const float h0 = fmaf(ea, s[0], eb * s[1]);
                    const float h1 = fmaf(ea, s[FT_U], eb * s[FT_U + 1]);
                    acc[k] += fmaf(1.0f - fv, h0, fv * h1);
                }
            }
        }
        __syncthreads();
    }
    if (gx < nx && gy < ny) store_column<KZ>(acc, n_sub, c.kn, ix, iy, z0, nx, ny, accumulate, vol);
}

// The longest column that still gives 400 workgroups (a column's FP64
// projection and a patch's footprint are shared by its voxels; fewer workgroups
// leave CUs idle), 60 views of (1.5 n)^2 at n^3, columns of 16 / 8 / 4: n = 64
// 97 / 73 / 55 us (64 / 128 / 256 workgroups), 96: 106 / 90 / 95, 128: 126 /
// 132 / 180, 200: 369 / 435 / 625 us.  Voxels past the volume's end cost what
// others do, so a shorter column is taken where it is cheaper in all, a column
// costing its voxels and `extra` more: four, or eight with upright detectors
// (M[2] = 0), whose voxels are cheaper.  Columns of 16 and 8, 20 x 512 x 512 (z,
// y, x): upright 293 and 303 us, rolled 346 and 226 (314 from memory).
int column_length(int nx, int ny, int nz, int extra) {
    constexpr long long FILL = 400;
    const long long patches = static_cast<long long>((nx + VB_TX - 1) / VB_TX) *
                              ((ny + VB_TY - 1) / VB_TY);
    int best = 4;
    long long least = LLONG_MAX;
    for (int kz = 16; kz >= 4; kz /= 2) {
        const long long columns = (nz + kz - 1) / kz;
        if (kz > 4 && patches * columns < FILL) continue;
        if (columns * (kz + extra) < least) {
            least = columns * (kz + extra);
            best = kz;
        }
    }
    return best;
}

// FOOT: with footprints.
template <typename TS, int KZ, bool FOOT, bool ONES = false>
hipError_t launch_columns(const RayGrid &g, const double *Pm, const TS *src, float *vol,
                          int accumulate, const VoxelGrid &vg, hipStream_t s) {
    const int tiles_x = (g.nx + VB_TX - 1) / VB_TX;
    const int tiles_y = (g.ny + VB_TY - 1) / VB_TY;
    const int tiles_z = (g.nz + KZ - 1) / KZ;
    const long long n_tiles = static_cast<long long>(tiles_x) * tiles_y * tiles_z;
    if (n_tiles <= 0 || n_tiles >= (1ll << 31)) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(n_tiles)), block(VB_THREADS);
    if constexpr (FOOT)
        hipLaunchKernelGGL((vbp_tile_kernel<TS, KZ>), grid, block, 0, s, Pm, g.views, g.n_views,
                           g.n_sub, g.n_u, g.n_v, g.nx, g.ny, g.nz, tiles_y, tiles_z, src, vol,
                           accumulate, vg);
    else
        hipLaunchKernelGGL((vbp_kernel<TS, ONES, KZ>), grid, block, 0, s, Pm, g.views, g.n_views,
                           g.n_sub, g.n_u, g.n_v, g.nx, g.ny, g.nz, tiles_y, tiles_z, src, vol,
                           accumulate, vg);
    return hipGetLastError();
}

template <typename TS>
hipError_t launch_typed(const RayGrid &g, const double *Pm, const void *sino, float *vol,
                        int accumulate, const VoxelGrid &vg, hipStream_t s) {
    const TS *src = static_cast<const TS *>(sino);
    const int kz = static_cast<long long>(g.n_views) * g.n_sub < 2 ? 0 : vg.foot_kz;
    if (kz == 16) return launch_columns<TS, 16, true>(g, Pm, src, vol, accumulate, vg, s);
    if (kz == 8) return launch_columns<TS, 8, true>(g, Pm, src, vol, accumulate, vg, s);
    if (kz == 4) return launch_columns<TS, 4, true>(g, Pm, src, vol, accumulate, vg, s);
    return column_length(g.nx, g.ny, g.nz, 4) >= 8
               ? launch_columns<TS, 8, false>(g, Pm, src, vol, accumulate, vg, s)
               : launch_columns<TS, 4, false>(g, Pm, src, vol, accumulate, vg, s);
}

// Whether a view's footprint of a patch, kz voxels about the middle of the
// volume, fits in LDS (vbp_tile_kernel's rule).
bool footprint_fits(const double *M, const VoxelGrid &vg, const PatchBox &b, int kz) {
    if (M[10] != 0.0) return false;
    const double dz = vg.cyl ? vg.dz : 1.0, hz = 0.5 * (kz - 1) * dz;
    double u0 = FAR_PIXEL, u1 = -FAR_PIXEL, v0 = FAR_PIXEL, v1 = -FAR_PIXEL;
    bool pos = true, neg = true;
    for (int i = 0; i < 8; ++i) {
        const double x = (i & 1) ? b.xb : b.xa, y = (i & 2) ? b.yb : b.ya, z = (i & 4) ? hz : -hz;
        const double w = M[8] * x + M[9] * y + M[11];
        const double u = (M[0] * x + M[1] * y + M[2] * z + M[3]) / w;
        const double v = (M[4] * x + M[5] * y + M[6] * z + M[7]) / w;
        pos = pos && w > 0.0;
        neg = neg && w < 0.0;
        u0 = std::min(u0, u);
        u1 = std::max(u1, u);
        v0 = std::min(v0, v);
        v1 = std::max(v1, v);
    }
    return (pos || neg) && u0 > -FAR_PIXEL && u1 < FAR_PIXEL && v0 > -FAR_PIXEL &&
           v1 < FAR_PIXEL && std::floor(u1) + 1.0 - std::floor(u0) < FT_U &&
           std::floor(v1) + 1.0 - std::floor(v0) < FT_V;
}

}  // namespace

// With a footprint a view costs vbp_tile_kernel half of what it costs
// vbp_kernel, without one a tenth to twice more, and patches that lack many hold
// the launch up: up to a quarter may lack it.  60 views of 384^2 at 256^3,
// vbp_tile_kernel and vbp_kernel: 606 and 1218 us with footprints, jittered
// (none has one) 2609 and 2090, of 768^2 (too large) 1401 and 1250; 2 x 512 x 512
// (z, y, x) jittered 139 and 101; cylinder of 150 x 400 x 100 (27 % lack it) 535
// and 508, 150 x 500 x 100 (16 %) 553 and 651, 100 x 400 x 150 (6 %) 367 and 508.
// A single view has too few loads in flight (256^3: 36 and 31 us).
int footprint_column(const double *P, size_t m, const VoxelGrid &vg, int nx, int ny, int nz) {
    // the middle patches of a division into 3 x 3
    const int px = (nx - 1) / VB_TX + 1, py = (ny - 1) / VB_TY + 1;
    PatchBox box[9];
    for (int i = 0; i < 9; ++i)
        box[i] = patch_box(vg, (2 * (i % 3) + 1) * px / 6, (2 * (i / 3) + 1) * py / 6, nx, ny, nz);
    const size_t step = (m + 63) / 64;
    bool upright = true;
    for (size_t k = 0; k < m; k += step) upright = upright && P[12 * k + 2] == 0.0;
    const int longest = column_length(nx, ny, nz, upright ? 8 : 4);
    for (int kz = longest; kz >= std::min(longest, 8); kz /= 2) {
        size_t all = 0, miss = 0;
        for (size_t k = 0; k < m; k += step)
            for (const PatchBox &b : box) {
                ++all;
                miss += !footprint_fits(P + 12 * k, vg, b, kz);
            }
        if (4 * miss <= all) return kz;
    }
    return 0;
}

hipError_t launch_back_voxel(const RayGrid &g, const double *Pm, const void *sino, int sino_dtype,
                             float *vol, int accumulate, int ones, const VoxelGrid &vg,
                             hipStream_t s) {
    if (g.n_views <= 0) return hipSuccess;
    if (g.n_u < 2 || g.n_v < 2 || g.n_u >= (1 << 24) || g.n_v >= (1 << 24) ||
        static_cast<long long>(g.n_u) * g.n_v >= (1ll << 30))
        return hipErrorInvalidValue;
    if (ones)
        return launch_columns<float, 8, false, true>(g, Pm, nullptr, vol, accumulate, vg, s);
    switch (sino_dtype) {
    case F32: return launch_typed<float>(g, Pm, sino, vol, accumulate, vg, s);
    case BF16: return launch_typed<bf16_t>(g, Pm, sino, vol, accumulate, vg, s);
    case F16: return launch_typed<_Float16>(g, Pm, sino, vol, accumulate, vg, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ctrex
