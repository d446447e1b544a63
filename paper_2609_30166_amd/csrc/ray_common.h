// Device-side building blocks shared by the projector kernels: storage
// conversions, FP64 ray set-up, trilinear corners, the displacement warp and
// the XCD-aware block mapping.  Included by the .hip translation units only.
#pragma once

#include "ctrex_internal.h"

namespace ctrex {
namespace dev {

// ---------------------------------------------------------------- storage --
__device__ __forceinline__ float ld(const float *p, int i) { return p[i]; }
__device__ __forceinline__ float ld(const bf16_t *p, int i) {
    return __uint_as_float(static_cast<uint32_t>(p[i].bits) << 16);
}
__device__ __forceinline__ float ld(const _Float16 *p, int i) { return static_cast<float>(p[i]); }

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ void st(float *p, int i, float v) { p[i] = v; }
__device__ __forceinline__ void st(bf16_t *p, int i, float v) { p[i].bits = f32_to_bf16_rne(v); }
__device__ __forceinline__ void st(_Float16 *p, int i, float v) { p[i] = static_cast<_Float16>(v); }

// ------------------------------------------------------------- ray set-up --
// Sample i of a ray sits at b + i s (index coordinates).  The FP64 set-up
// rounds b and s once to signed 64-bit fixed point with FX = 40 fractional
// bits; every sample position is then the exact integer q + i t, reached by
// stepping (q += t) in the forward projector and by one multiply-add or by
// stepping in the backprojector, so both see the same sample bit for bit.
// Against FP64 the positions are off by at most 2^-41 (the rounding of q)
// plus i 2^-41 (that of t): under 1e-8 voxel for 4096 samples and under
// 1e-5 voxel at the 2^24-sample limit.  The integer voxel is the top word
// shifted, the fraction its next 32 bits rounded to FP32: no FP64 in the
// sample loops and no re-anchoring along the ray.
constexpr int FX = 40;

struct Ray {
    long long qx, qy, qz;   // position of sample 0, fixed point
    long long tx, ty, tz;   // step vector, fixed point
    float bx, by, bz;       // position of sample 0 in FP32 (range estimates only)
    float fx, fy, fz;       // step vector in FP32 (range estimates only)
    float h;                // sample weight (path length per sample)
    int n;                  // number of samples
    int axis;               // axis across the hull face the ray enters through
};

__device__ __forceinline__ long long to_fx(double v) {
    return static_cast<long long>(rint(v * 1099511627776.0));   // v 2^FX, to nearest
}

// Integer voxel k = floor(p) and fraction f = p - k of a fixed-point
// coordinate: k from the top word, f from the top 32 fraction bits rounded to
// FP32 (so f may round up to 1.0, which the corner weights treat like any
// other fraction: weight 1 on the upper corner).
__device__ __forceinline__ void fx_split(long long p, int &k, float &f) {
    const unsigned long long u = static_cast<unsigned long long>(p);
    k = static_cast<int>(static_cast<uint32_t>(u >> 32)) >> (FX - 32);
    f = static_cast<float>(static_cast<uint32_t>(u >> (FX - 32))) * 2.3283064365386963e-10f;  // 2^-32
}

// FP64 clipping of one axis' slab.  Returns false when the ray misses.
__device__ __forceinline__ bool slab(double s, double d, double hi, double &t0, double &t1) {
    if (d == 0.0) return !(s < 0.0 || s > hi);
    const double inv = 1.0 / d;
    const double a = (0.0 - s) * inv;
    const double b = (hi - s) * inv;
    const double lo_t = a < b ? a : b;
    const double hi_t = a < b ? b : a;
    if (lo_t > t0) t0 = lo_t;
    if (hi_t < t1) t1 = hi_t;
    return true;
}

// Ray through pixel centre (u, v) of sub-view sv, in FP64: unit direction
// M^-1 (u, v, 1) / |.|, slab clip to the voxel-centre hull, n = ceil(L / step),
// h = L / n, samples at t_in + (i + 1/2) h.  Reciprocals are formed once (one
// division for the length, one per axis for the slabs); the sample count n
// is then an integer function of correctly rounded FP64 values, so it differs
// from a plain division-based evaluation only if L / step lies within an ulp
// of an integer.
__device__ __forceinline__ bool setup_ray(const SubView &sv, double u, double v, int nx, int ny,
                                          int nz, double step, Ray &r) {
    double dx = fma(sv.Mi[0], u, fma(sv.Mi[1], v, sv.Mi[2]));
    double dy = fma(sv.Mi[3], u, fma(sv.Mi[4], v, sv.Mi[5]));
    double dz = fma(sv.Mi[6], u, fma(sv.Mi[7], v, sv.Mi[8]));
    const double inv_len = 1.0 / sqrt(fma(dx, dx, fma(dy, dy, dz * dz)));
    dx *= inv_len;
    dy *= inv_len;
    dz *= inv_len;
    double t0 = -__builtin_inf(), t1 = __builtin_inf();
    if (!slab(sv.S[0], dx, static_cast<double>(nx - 1), t0, t1)) return false;
    const double t0x = t0;
    if (!slab(sv.S[1], dy, static_cast<double>(ny - 1), t0, t1)) return false;
    const double t0y = t0;
    if (!slab(sv.S[2], dz, static_cast<double>(nz - 1), t0, t1)) return false;
    r.axis = t0 > t0y ? 2 : (t0y > t0x ? 1 : 0);
    if (!(t1 > t0)) return false;
    const double L = t1 - t0;
    const double nd = ceil(L / step);
    const double h = L / nd;
    const double tb = fma(0.5, h, t0);
    const double bx = fma(tb, dx, sv.S[0]);
    const double by = fma(tb, dy, sv.S[1]);
    const double bz = fma(tb, dz, sv.S[2]);
    const double sx = h * dx, sy = h * dy, sz = h * dz;
    r.qx = to_fx(bx);
    r.qy = to_fx(by);
    r.qz = to_fx(bz);
    r.tx = to_fx(sx);
    r.ty = to_fx(sy);
    r.tz = to_fx(sz);
    r.bx = static_cast<float>(bx);
    r.by = static_cast<float>(by);
    r.bz = static_cast<float>(bz);
    r.fx = static_cast<float>(sx);
    r.fy = static_cast<float>(sy);
    r.fz = static_cast<float>(sz);
    r.h = static_cast<float>(h);
    r.n = static_cast<int>(nd);
    return true;
}

// ------------------------------------------------------------ trilinear ----
struct VolDims {
    int nx, ny, nz;
    int nxy;
    float mx, my, mz;   // n - 1 as float (clamp bounds)
};

struct Corner {
    int base;           // linear index of the lower corner
    float fx, fy, fz;   // fractions in [0, 1]
};

// Corner k and fraction f of a warped coordinate outside [0, n - 2] on some
// axis: true if it lies in [0, n - 1] on this one, with the last face turned
// into weight 1 on corner n - 2; the corner is clamped into the grid either way.
__device__ __forceinline__ bool axis_last(int &k, float &f, int n) {
    const bool in = k >= 0 && (k < n - 1 || (k == n - 1 && f == 0.0f));
    if (k < 0) {
        k = 0;
        f = 0.0f;
    }
    if (k > n - 2) {
        k = n - 2;
        f = 1.0f;
    }
    return in;
}

// Corner of an unwarped position already split into k + f with f in [0, 1]:
// the clamps (k < 0 rounds onto the first corner with weight 0 on the next;
// k > n - 2 is the last face, weight 1 on it).
__device__ __forceinline__ void axis_clamp(int k, float f, int n, int &kc, float &fc) {
    kc = k;
    fc = f;
    if (k < 0) {
        kc = 0;
        fc = 0.0f;
    }
    if (k > n - 2) {
        kc = n - 2;
        fc = 1.0f;
    }
}

__device__ __forceinline__ int base_x(const VolDims &d, int ix, int iy, int iz) {
    return (iz * d.ny + iy) * d.nx + ix;
}

// Trilinear blend of the eight corner values (x first, then y, then z).
__device__ __forceinline__ float blend(const Corner &k, float v000, float v001, float v010,
                                       float v011, float v100, float v101, float v110,
                                       float v111) {
    const float a00 = fmaf(k.fx, v001 - v000, v000);
    const float a01 = fmaf(k.fx, v011 - v010, v010);
    const float a10 = fmaf(k.fx, v101 - v100, v100);
    const float a11 = fmaf(k.fx, v111 - v110, v110);
    const float b0 = fmaf(k.fy, a01 - a00, a00);
    const float b1 = fmaf(k.fy, a11 - a10, a10);
    return fmaf(k.fz, b1 - b0, b0);
}

template <typename TV>
__device__ __forceinline__ float gather(const TV *__restrict__ vol, const VolDims &d,
                                        const Corner &k) {
    const int b = k.base;
    return blend(k, ld(vol, b), ld(vol, b + 1), ld(vol, b + d.nx), ld(vol, b + d.nx + 1),
                 ld(vol, b + d.nxy), ld(vol, b + d.nxy + 1), ld(vol, b + d.nxy + d.nx),
                 ld(vol, b + d.nxy + d.nx + 1));
}

// FP32 volumes: each x-adjacent pair of corners is one 8-byte load (4-byte
// aligned; gfx950 global loads accept it), halving the gather instructions.
typedef float f32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));

template <>
__device__ __forceinline__ float gather<float>(const float *__restrict__ vol, const VolDims &d,
                                               const Corner &k) {
    const int b = k.base;
    const f32x2_a4 p00 = *reinterpret_cast<const f32x2_a4 *>(vol + b);
    const f32x2_a4 p01 = *reinterpret_cast<const f32x2_a4 *>(vol + b + d.nx);
    const f32x2_a4 p10 = *reinterpret_cast<const f32x2_a4 *>(vol + b + d.nxy);
    const f32x2_a4 p11 = *reinterpret_cast<const f32x2_a4 *>(vol + b + d.nxy + d.nx);
    return blend(k, p00.x, p00.y, p01.x, p01.y, p10.x, p10.y, p11.x, p11.y);
}

// Lower corner in a y-fastest copy ([nz][nx][ny]).
__device__ __forceinline__ int base_t(const VolDims &d, int ix, int iy, int iz) {
    return (iz * d.nx + ix) * d.ny + iy;
}

// ----------------------------------------------------------------- warp ----
// Lower node and fraction of a node coordinate on an axis of n >= 2 nodes,
// clamped to [0, n - 1] (a coordinate of n - 1 is weight 1 on the last node).
__device__ __forceinline__ int node_corner(float c, int n, float &f) {
    c = fminf(fmaxf(c, 0.0f), static_cast<float>(n - 1));
    const int k = min(static_cast<int>(c), n - 2);
    f = c - static_cast<float>(k);
    return k;
}

// The eight displacement nodes of one grid cell, by component; node j is the
// x (bit 0), y (bit 1), z (bit 2) neighbour of the lower one.
struct NodeCell {
    int b = -1;        // index of the lower node
    float u[3][8];
    // a cell spans several voxels, so consecutive samples mostly share one
    __device__ __forceinline__ void load(const WarpGrid &w, int base) {
        if (base == b) return;
        b = base;
        const float4 *const p = w.U + base;
        const int sy = w.gx, sz = w.gx * w.gy;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float4 v = p[(j & 1) + ((j & 2) ? sy : 0) + ((j & 4) ? sz : 0)];
            u[0][j] = v.x;
            u[1][j] = v.y;
            u[2][j] = v.z;
        }
    }
};

// Displacement at the sample k + f (per axis: integer voxel and fraction):
// the node grid coordinate (k + f) (g - 1) / (n - 1) is formed in FP32 (it
// is at most g - 1, so its rounding is ~2^-19 of a grid cell) and U is
// interpolated trilinearly there, lookups clamped to the grid.  `cell` holds
// the nodes of the last sample's cell.
__device__ __forceinline__ float3 displacement(const WarpGrid &w, NodeCell &cell, int kx, float fx,
                                               int ky, float fy, int kz, float fz) {
    const float gx = fmaf(fx, w.fsx, static_cast<float>(kx) * w.fsx);
    const float gy = fmaf(fy, w.fsy, static_cast<float>(ky) * w.fsy);
    const float gz = fmaf(fz, w.fsz, static_cast<float>(kz) * w.fsz);
    float ax, ay, az;
    const int ix = node_corner(gx, w.gx, ax);
    const int iy = node_corner(gy, w.gy, ay);
    const int iz = node_corner(gz, w.gz, az);
    cell.load(w, (iz * w.gy + iy) * w.gx + ix);
    float r[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const float(&u)[8] = cell.u[q];
        const float a00 = fmaf(ax, u[1] - u[0], u[0]);
        const float a01 = fmaf(ax, u[3] - u[2], u[2]);
        const float a10 = fmaf(ax, u[5] - u[4], u[4]);
        const float a11 = fmaf(ax, u[7] - u[6], u[6]);
        const float b0 = fmaf(ay, a01 - a00, a00);
        const float b1 = fmaf(ay, a11 - a10, a10);
        r[q] = fmaf(az, b1 - b0, b0);
    }
    return make_float3(r[0], r[1], r[2]);
}

// Lower corner (ix, iy, iz) and fractions of the sample at fixed-point
// position (px, py, pz), after the pull-back warp c + tau U(c) (Sec. 3.1)
// when WARP; false if the warped sample leaves the hull.  The corner is
// always set and clamped into the grid, also for a sample outside (callers
// may form its address before discarding its value).  The forward and back
// projectors call this one function, so their corners and weights agree bit
// for bit.
template <bool WARP>
__device__ __forceinline__ bool sample_corner(const VolDims &d, const WarpGrid &w, NodeCell &cell,
                                              float tau, long long px, long long py, long long pz,
                                              int &ix, int &iy, int &iz, float &fx, float &fy,
                                              float &fz) {
    int kx, ky, kz;
    float lx, ly, lz;
    fx_split(px, kx, lx);
    fx_split(py, ky, ly);
    fx_split(pz, kz, lz);
    if (WARP) {
        const float3 u = displacement(w, cell, kx, lx, ky, ly, kz, lz);
        lx = fmaf(tau, u.x, lx);
        ly = fmaf(tau, u.y, ly);
        lz = fmaf(tau, u.z, lz);
        const float ex = floorf(lx), ey = floorf(ly), ez = floorf(lz);
        ix = kx + static_cast<int>(ex);
        iy = ky + static_cast<int>(ey);
        iz = kz + static_cast<int>(ez);
        fx = lx - ex;
        fy = ly - ey;
        fz = lz - ez;
        if (static_cast<unsigned>(ix) <= static_cast<unsigned>(d.nx - 2) &&
            static_cast<unsigned>(iy) <= static_cast<unsigned>(d.ny - 2) &&
            static_cast<unsigned>(iz) <= static_cast<unsigned>(d.nz - 2))
            return true;
        // on the last face (weight 1 on the last cell's upper corner), or
        // outside the hull
        const bool in = axis_last(ix, fx, d.nx) & axis_last(iy, fy, d.ny) & axis_last(iz, fz, d.nz);
        return in;
    } else {
        axis_clamp(kx, lx, d.nx, ix, fx);
        axis_clamp(ky, ly, d.ny, iy, fy);
        axis_clamp(kz, lz, d.nz, iz, fz);
    }
    return true;
}

// ------------------------------------------------------------- tiling ------
struct TileCoord {
    int k;      // position in the view list
    int p;      // projection index
    int iu, iv; // pixel of this lane
    int lidx;   // index of the (tile, projection) pair
    bool valid; // the pair exists
};

// XCD-aware block -> (tile, projection) mapping (launch_order, pair_of).
// Hardware hands workgroup b to XCD b mod 8.  The pairs are cut into units of
// g.grp consecutive projections of g.run consecutive tiles (u fastest),
// projections fastest, which the XCDs take in turn.  One unit's rays sample one part of the volume
// at nearly the same angle, so it stays in the XCD's 4 MB L2 while they march
// (with all projections of a tile first, the XCD's ~100 concurrent workgroups
// span 50 degrees or more of a scan); taking units in turn keeps the XCDs
// equally loaded where parts of a scan miss the volume, as at a helix's ends.
// SIRT step over 180 of 720 views of 768^2 at 512^3: 566 ms before, with this
// mapping and the choice of copy below 443 / 440 / 437 ms for units of 4 / 8 /
// 16 projections x 32 tiles (8 x 8: 437, 32 x 8: 434); helical 256^3 warp,
// 150 x 4 views of 512 x 256: 355 ms before, 347 / 347 / 345 ms (8 x 8: 373,
// 32 x 8: 369).  A wave's lanes are 16 x 4 pixels.
__device__ __forceinline__ TileCoord tile_coord(const RayGrid &g) {
    TileCoord t;
    const Pair q = pair_of(blockIdx.x, g.grp, g.run, g.runs, g.turn, g.tiles_u * g.tiles_v,
                           g.n_views);
    t.k = q.k;
    t.valid = q.valid;
    const int tile = q.tile;
    t.lidx = tile * g.n_views + t.k;
    const int tu = tile % g.tiles_u;
    const int tv = tile / g.tiles_u;
    t.p = g.views ? g.views[t.k] : t.k;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    t.iu = tu * TILE_U + (lane & 15);
    t.iv = tv * TILE_V + wave * 4 + (lane >> 4);
    return t;
}

// The same with 8 x 8 pixels to a wave.
__device__ __forceinline__ TileCoord square_waves(TileCoord t) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    t.iu += (wave & 1) * 8 + (lane & 7) - (lane & 15);
    t.iv += (wave >> 1) * 8 + (lane >> 3) - (wave * 4 + (lane >> 4));
    return t;
}

__device__ __forceinline__ VolDims vol_dims(const RayGrid &g) {
    VolDims d;
    d.nx = g.nx;
    d.ny = g.ny;
    d.nz = g.nz;
    d.nxy = g.nx * g.ny;
    d.mx = static_cast<float>(g.nx - 1);
    d.my = static_cast<float>(g.ny - 1);
    d.mz = static_cast<float>(g.nz - 1);
    return d;
}

// Block-wide sum of one double per lane into partials[L] (deterministic order).
__device__ __forceinline__ void block_sum_store(double v, double *out) {
    __shared__ double red[PROJ_THREADS / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < PROJ_THREADS / 64; ++i) s += red[i];
        *out = s;
    }
}


}  // namespace dev
}  // namespace ctrex
