// Forward projector on the aligned cylindrical domain (Sec. 3.5; the
// projector's geometry-level modification, Sec. 4.2.1).
//
// The volume is a polar grid [n_z][n_phi][n_r] about the z axis of a cylinder
// frame that a rigid pose maps the V frame to.  The host hands the kernel one
// table entry per (projection, sub-view) already in the cylinder frame: the
// source S_c and R_p M^-1, so a pixel ray's direction is R_p M^-1 (u, v, 1)
// normalised.  Per ray, in FP64: clip to the hull r <= R_h, |z| <= H (the
// infinite cylinder's quadratic and the z slab), n = ceil(L / step),
// h = L / n, sample t_i = t_in + (i + 1/2) h, position S_c + t_i d_c.  Per
// sample, in FP32: r = |(x, y)|, phi = atan2(y, x), continuous indices
// a = r / dr - 1/2 (clamped to [0, n_r - 1]: the core takes ring 0's values),
// b = phi n_phi / (2 pi) (periodic), c = z / dz + (n_z - 1) / 2, trilinear
// lookup (FP32 volumes: two 16-byte loads from a pair-packed copy).  Sub-views
// are averaged.  Positions are FP64 until the polar map, so their error is
// the FP32 rounding of r and phi (about 1e-7 of the hull radius).
//
// The grid of workgroups and the FP_* epilogues (plain, 1/(A 1), correction
// with residual partials) are those of the Cartesian projector.

#include "ray_common.h"

#include <climits>

namespace ctrex {
namespace {

using namespace dev;

constexpr double kTwoPi = 6.283185307179586476925287;

// Line S + t d (cylinder frame, |d| = 1) against the hull.  False if it misses.
__device__ __forceinline__ bool cyl_clip(const SubView &sv, const double d[3], const CylGrid &c,
                                         double &t0, double &t1) {
    double lo = -__builtin_inf(), hi = __builtin_inf();
    const double A = fma(d[0], d[0], d[1] * d[1]);
    const double B = fma(sv.S[0], d[0], sv.S[1] * d[1]);
    const double C = fma(sv.S[0], sv.S[0], sv.S[1] * sv.S[1]) - c.rh2;
    if (A == 0.0) {
        if (C > 0.0) return false;
    } else {
        const double disc = fma(B, B, -A * C);
        if (disc < 0.0) return false;
        const double sq = sqrt(disc);
        const double ia = 1.0 / A;
        lo = (-B - sq) * ia;
        hi = (-B + sq) * ia;
    }
    if (d[2] == 0.0) {
        if (fabs(sv.S[2]) > c.hz) return false;
    } else {
        const double iz = 1.0 / d[2];
        const double za = (-c.hz - sv.S[2]) * iz, zb = (c.hz - sv.S[2]) * iz;
        lo = fmax(lo, fmin(za, zb));
        hi = fmin(hi, fmax(za, zb));
    }
    t0 = lo;
    t1 = hi;
    return hi > lo;
}

// Unit direction of the ray through pixel (u, v) of sub-view sv (cylinder frame).
__device__ __forceinline__ void cyl_dir(const SubView &sv, double u, double v, double d[3]) {
    d[0] = fma(sv.Mi[0], u, fma(sv.Mi[1], v, sv.Mi[2]));
    d[1] = fma(sv.Mi[3], u, fma(sv.Mi[4], v, sv.Mi[5]));
    d[2] = fma(sv.Mi[6], u, fma(sv.Mi[7], v, sv.Mi[8]));
    const double il = 1.0 / sqrt(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2])));
    d[0] *= il;
    d[1] *= il;
    d[2] *= il;
}

__device__ __forceinline__ int cyl_steps(double L, double step) {
    const int n = static_cast<int>(ceil(L / step));
    return n < 1 ? 1 : n;
}

// Lower node and fractions of a lookup at (x, y, z): ring a0 (a0 + 1), angle
// j0 (the next one modulo n_phi), slice k0 (k0 + 1).
struct PolarCorner {
    int a0, j0, k0;
    float fa, fb, fz;
};

// atan(t) / t - 1 over t^2 for t in [0, tan(pi/8)], relative error 1.2e-9 of
// atan, 1.4e-9 with the coefficients in FP32 (minimax fit by Remez exchange).
__device__ __forceinline__ float atan_tail(float s) {
    float p = fmaf(s, -0.06034788f, 0.10573479f);
    p = fmaf(s, p, -0.14240083f);
    p = fmaf(s, p, 0.19998217f);
    return fmaf(s, p, -0.33333308f);
}

// The polar map in FP32 (clamped radial and axial index, periodic angle).
// r = sqrt(x^2 + y^2) from the hardware reciprocal square root with one
// correction step; the angle within an octant is 2 atan(t), t = min / (r +
// max) of |x|, |y| (the half angle's tangent, at most tan(pi/8), so a short
// polynomial serves), also with one correction step of the hardware
// reciprocal.  Both errors are about an ulp, as the library's sqrtf and atan2f
// give at four times the instructions: no scaling, no special cases, which
// finite positions within the hull do not need.  On the axis itself (x = y =
// 0) r and the angle are 0.
__device__ __forceinline__ PolarCorner polar_corner(const CylGrid &c, float x, float y, float z) {
    PolarCorner k;
    const float v = fmaxf(fmaf(x, x, y * y), 1e-36f);
    const float rs = __builtin_amdgcn_rsqf(v);
    float r = v * rs;
    r = fmaf(fmaf(-r, r, v), 0.5f * rs, r);
    const float ax = fabsf(x), ay = fabsf(y);
    const float mn = fminf(ax, ay), den = r + fmaxf(ax, ay);
    const float rc = __builtin_amdgcn_rcpf(den);
    float t = mn * rc;
    t = fmaf(fmaf(-t, den, mn), rc, t);
    const float s = t * t;
    float b = fmaf(t * s, atan_tail(s), t) * c.phi_scale2;
    b = ay > ax ? c.quarter - b : b;
    b = x < 0.0f ? c.half - b : b;
    b = y < 0.0f ? c.full - b : b;
    float bf = floorf(b);
    k.fb = b - bf;
    k.j0 = static_cast<int>(bf);
    if (k.j0 >= c.nphi) k.j0 = 0;   // rounded up to a full turn: fraction 0
    const float a = fminf(fmaxf(fmaf(r, c.inv_dr, -0.5f), 0.0f), static_cast<float>(c.nr - 1));
    const float af = fminf(floorf(a), static_cast<float>(c.nr - 2));
    k.fa = a - af;
    k.a0 = static_cast<int>(af);
    const float zz = fminf(fmaxf(fmaf(z, c.inv_dz, c.half_z), 0.0f), static_cast<float>(c.nz - 1));
    const float zf = fminf(floorf(zz), static_cast<float>(c.nz - 2));
    k.fz = zz - zf;
    k.k0 = static_cast<int>(zf);
    return k;
}

__device__ __forceinline__ float polar_blend(const PolarCorner &k, float v00, float v01, float v02,
                                             float v03, float v10, float v11, float v12,
                                             float v13) {
    // v?0, v?1: rings a0, a0 + 1 at j0; v?2, v?3: at the next angle
    const float q00 = fmaf(k.fa, v01 - v00, v00), q01 = fmaf(k.fa, v03 - v02, v02);
    const float q10 = fmaf(k.fa, v11 - v10, v10), q11 = fmaf(k.fa, v13 - v12, v12);
    const float s0 = fmaf(k.fb, q01 - q00, q00), s1 = fmaf(k.fb, q11 - q10, q10);
    return fmaf(k.fz, s1 - s0, s0);
}

template <typename TV>
__device__ __forceinline__ float cyl_sample(const TV *__restrict__ vol, const CylGrid &c, float x,
                                            float y, float z) {
    const PolarCorner k = polar_corner(c, x, y, z);
    const int j1 = k.j0 + 1 == c.nphi ? 0 : k.j0 + 1;
    const int plane = c.nphi * c.nr;
    const int b0 = k.k0 * plane + k.j0 * c.nr + k.a0, b1 = k.k0 * plane + j1 * c.nr + k.a0;
    return polar_blend(k, ld(vol, b0), ld(vol, b0 + 1), ld(vol, b1), ld(vol, b1 + 1),
                       ld(vol, b0 + plane), ld(vol, b0 + plane + 1), ld(vol, b1 + plane),
                       ld(vol, b1 + plane + 1));
}

// The same lookup from a pair-packed copy: two consecutive elements hold the
// four (ring, angle) corners of a slice, one 16-byte load; slice k0 + 1 is the
// second.  PHI: the angle-fastest copy.  p1: the copy at slice 1.
typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
template <bool PHI>
__device__ __forceinline__ float cyl_sample_pairs(const float2 *__restrict__ p0,
                                                  const float2 *__restrict__ p1, const CylGrid &c,
                                                  unsigned plane, float x, float y, float z) {
    const PolarCorner k = polar_corner(c, x, y, z);
    // 32 x 32 -> 64-bit multiply-adds run at the full rate
    const unsigned row =
        PHI ? static_cast<unsigned>(static_cast<unsigned long long>(static_cast<unsigned>(k.a0)) *
                                        static_cast<unsigned>(c.nphi + 1) +
                                    static_cast<unsigned>(k.j0))
            : static_cast<unsigned>(static_cast<unsigned long long>(static_cast<unsigned>(k.j0)) *
                                        static_cast<unsigned>(c.nr) +
                                    static_cast<unsigned>(k.a0));
    const unsigned long long e =
        static_cast<unsigned long long>(static_cast<unsigned>(k.k0)) * plane + row;
    const f32x4_a8 v = *reinterpret_cast<const f32x4_a8 *>(p0 + e);
    const f32x4_a8 w = *reinterpret_cast<const f32x4_a8 *>(p1 + e);
    return PHI ? polar_blend(k, v.x, v.y, v.z, v.w, w.x, w.y, w.z, w.w)
               : polar_blend(k, v.x, v.z, v.y, v.w, w.x, w.z, w.y, w.w);
}

// One ray's projection value.  FP32 volumes are read from the two pair-packed
// copies: where the rays of a wave run mainly towards or away from the axis,
// they lie side by side in angle and read the angle-fastest copy, where they
// pass the axis, side by side in radius, the ring-fastest one (decided by the
// majority of the wave for every four samples); neighbouring lanes then share
// cache lines.  The values do not depend on the choice.  The SIRT step named
// below took 8.5 ms with the library's square root and arc tangent and one
// corner-packed copy, 8.1 ms with polar_corner and the ring-fastest pairs, 6.8
// with both copies.
template <typename TV, int MODE>
__device__ __forceinline__ float cyl_march(const RayGrid &g, const CylGrid &c,
                                           const TV *__restrict__ vol, const FpExtra &ex,
                                           const TileCoord &t) {
    constexpr bool PK = sizeof(TV) == 4;   // 16-bit volumes come without copies
    float y = 0.0f;
    const unsigned plane_r = static_cast<unsigned>(c.nphi) * static_cast<unsigned>(c.nr);
    const unsigned plane_p = plane_r + static_cast<unsigned>(c.nr);
    const float2 *const r0 = static_cast<const float2 *>(ex.px), *const r1 = r0 + plane_r;
    const float2 *const p0 = static_cast<const float2 *>(ex.py), *const p1 = p0 + plane_p;
    for (int s = 0; s < g.n_sub; ++s) {
        const SubView &sv = g.tab[t.p * g.n_sub + s];
        double d[3], t0, t1;
        cyl_dir(sv, static_cast<double>(t.iu), static_cast<double>(t.iv), d);
        if (!cyl_clip(sv, d, c, t0, t1)) continue;
        const double L = t1 - t0;
        const int n = cyl_steps(L, g.step);
        const double h = L / n;
        if (MODE == FP_RECIP_ONES) {
            y += static_cast<float>(L);   // n samples of weight h
            continue;
        }
        // four independent samples per iteration keep several lookups in
        // flight; positions are stepped in FP64 (n roundings of 2^-53 stay
        // far below the FP32 rounding that follows)
        const double tb = fma(0.5, h, t0);
        double px = fma(tb, d[0], sv.S[0]), py = fma(tb, d[1], sv.S[1]), pz = fma(tb, d[2], sv.S[2]);
        const double sx = h * d[0], sy = h * d[1], sz = h * d[2];
        const float dx = static_cast<float>(d[0]), dy = static_cast<float>(d[1]);
        float acc0 = 0.0f, acc1 = 0.0f, acc2 = 0.0f, acc3 = 0.0f;
        auto four = [&](auto lookup) {
            const double x1 = px + sx, y1 = py + sy, z1 = pz + sz;
            const double x2 = x1 + sx, y2 = y1 + sy, z2 = z1 + sz;
            const double x3 = x2 + sx, y3 = y2 + sy, z3 = z2 + sz;
            acc0 += lookup(static_cast<float>(px), static_cast<float>(py), static_cast<float>(pz));
            acc1 += lookup(static_cast<float>(x1), static_cast<float>(y1), static_cast<float>(z1));
            acc2 += lookup(static_cast<float>(x2), static_cast<float>(y2), static_cast<float>(z2));
            acc3 += lookup(static_cast<float>(x3), static_cast<float>(y3), static_cast<float>(z3));
            px = x3 + sx;
            py = y3 + sy;
            pz = z3 + sz;
        };
        auto by_ring = [&](float x, float yy, float z) {
            if constexpr (PK)
                return cyl_sample_pairs<false>(r0, r1, c, plane_r, x, yy, z);
            else
                return cyl_sample(vol, c, x, yy, z);
        };
        auto by_angle = [&](float x, float yy, float z) {
            return cyl_sample_pairs<true>(p0, p1, c, plane_p, x, yy, z);
        };
        int i = 0;
        for (; i + 3 < n; i += 4) {
            if constexpr (PK) {
                const float x = static_cast<float>(px), yy = static_cast<float>(py);
                const bool radial = fabsf(fmaf(x, dx, yy * dy)) > fabsf(fmaf(x, dy, -yy * dx));
                if (2 * __popcll(__ballot(radial)) > __popcll(__ballot(true))) {
                    four(by_angle);
                    continue;
                }
            }
            four(by_ring);
        }
        for (; i < n; ++i) {
            acc0 += by_ring(static_cast<float>(px), static_cast<float>(py), static_cast<float>(pz));
            px += sx;
            py += sy;
            pz += sz;
        }
        y = fmaf(static_cast<float>(h), (acc0 + acc1) + (acc2 + acc3), y);
    }
    return y / static_cast<float>(g.n_sub);
}

// Occupancy cap for the FP32 (pair-packed) gathers, as for the Cartesian
// projector: SIRT step on 96 x 603 x 192 with 120 views of 288^2 6.84 ms at 2
// waves per SIMD, 6.66 at 3, 6.71 at 4 (100 x 628 x 200, 180 x 300^2: 12.50,
// 12.40, 13.01).  The ray-length mode (no gathers) keeps the default.
//
// 16-bit volumes have no copies, so most samples of a wave lie on lines of
// their own; its rays are 8 x 8 pixels there (40 x 250 x 80, 30 / 120 views of
// 120^2: 193 / 615 us, with 16 x 4 pixels 214 / 660; 48 x 300 x 96, 60 views 605
// and 615, but 32 x 200 x 64 229 and 205).  A volume beyond an XCD's L2 (BIG)
// lives from the few rays in flight sharing lines: 2 waves per SIMD and a tile's
// views one after the other (cyl_view_group).  60 views of 288^2, 96 x 603 x 192:
// 4.66 ms, without the cap 5.42, by 16 views 4.86, with neither 5.73; 128 x 800 x
// 256, 60 views of 384^2: 14.7 ms, 15.5, 17.8 and 18.5.  Smaller volumes keep the
// default (20 x 40 x 200: 197 us, with both 275).
template <typename TV, int MODE, bool BIG>
constexpr int fp_cyl_max_waves() {
    return MODE == FP_RECIP_ONES ? 8 : sizeof(TV) == 4 ? 3 : BIG ? 2 : 8;
}

template <typename TV, typename TS, int MODE, bool BIG = false>
__global__ __launch_bounds__(PROJ_THREADS) __attribute__((amdgpu_waves_per_eu(1, fp_cyl_max_waves<TV, MODE, BIG>())))
void fp_cyl_kernel(RayGrid g, CylGrid c,
                                                              const TV *__restrict__ vol,
                                                              TS *__restrict__ out, FpExtra ex) {
    TileCoord t = tile_coord(g);
    if (!t.valid) return;  // uniform over the block
    if constexpr (sizeof(TV) == 2) t = square_waves(t);
    const bool active = t.iu < g.n_u && t.iv < g.n_v;
    float y = 0.0f;
    if (active) y = cyl_march<TV, MODE>(g, c, vol, ex, t);
    const int pix = (t.k * g.n_v + t.iv) * g.n_u + t.iu;
    if (MODE == FP_PLAIN) {
        if (active) st(out, pix, y);
    } else if (MODE == FP_RECIP_ONES) {
        if (active) st(out, pix, y > 0.0f ? 1.0f / y : 0.0f);
    } else {
        double e2 = 0.0;
        if (active) {
            const float bval = ld(static_cast<const TS *>(ex.b), pix);
            const float res = bval - y;
            e2 = static_cast<double>(res) * static_cast<double>(res);
            if (MODE == FP_CORRECT) st(out, pix, ex.R[pix] * res);
        }
        block_sum_store(e2, ex.partials + t.lidx);
    }
}

__global__ __launch_bounds__(PROJ_THREADS) void count_cyl_kernel(RayGrid g, CylGrid c,
                                                                 unsigned long long *count) {
    const TileCoord t = tile_coord(g);
    if (!t.valid) return;
    unsigned long long n = 0;
    if (t.iu < g.n_u && t.iv < g.n_v) {
        for (int s = 0; s < g.n_sub; ++s) {
            const SubView &sv = g.tab[t.p * g.n_sub + s];
            double d[3], t0, t1;
            cyl_dir(sv, static_cast<double>(t.iu), static_cast<double>(t.iv), d);
            if (cyl_clip(sv, d, c, t0, t1))
                n += static_cast<unsigned long long>(cyl_steps(t1 - t0, g.step));
        }
    }
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(count, n);
}

inline dim3 cyl_grid(const RayGrid &g) { return dim3(g.blocks); }

template <typename TV, typename TS>
hipError_t fp_cyl_mode(const RayGrid &g, const CylGrid &c, const void *vol, void *out, int mode,
                       const FpExtra &ex, hipStream_t s) {
    const dim3 grid = cyl_grid(g), block(PROJ_THREADS);
    const TV *v = static_cast<const TV *>(vol);
    TS *o = static_cast<TS *>(out);
    switch (mode) {
    case FP_PLAIN:
        if constexpr (sizeof(TV) == 2) {
            if (cyl_view_group(c.nr, c.nphi, c.nz, BF16) > 0) {
                hipLaunchKernelGGL((fp_cyl_kernel<TV, TS, FP_PLAIN, true>), grid, block, 0, s, g,
                                   c, v, o, ex);
                break;
            }
        }
        hipLaunchKernelGGL((fp_cyl_kernel<TV, TS, FP_PLAIN>), grid, block, 0, s, g, c, v, o, ex);
        break;
    case FP_CORRECT:
        hipLaunchKernelGGL((fp_cyl_kernel<TV, TS, FP_CORRECT>), grid, block, 0, s, g, c, v, o, ex);
        break;
    case FP_RESIDUAL:
        hipLaunchKernelGGL((fp_cyl_kernel<TV, TS, FP_RESIDUAL>), grid, block, 0, s, g, c, v, o,
                           ex);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename TV>
hipError_t fp_cyl_out(const RayGrid &g, const CylGrid &c, const void *vol, void *out,
                      int out_dtype, int mode, const FpExtra &ex, hipStream_t s) {
    switch (out_dtype) {
    case F32: return fp_cyl_mode<TV, float>(g, c, vol, out, mode, ex, s);
    case BF16: return fp_cyl_mode<TV, bf16_t>(g, c, vol, out, mode, ex, s);
    case F16: return fp_cyl_mode<TV, _Float16>(g, c, vol, out, mode, ex, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_forward_cyl(const RayGrid &g, const CylGrid &c, const void *vol, int vol_dtype,
                              void *out, int out_dtype, int mode, const FpExtra &ex,
                              hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    if (c.nr < 2 || c.nphi < 3 || c.nz < 2) return hipErrorInvalidValue;
    if (mode == FP_RECIP_ONES) {
        hipLaunchKernelGGL((fp_cyl_kernel<float, float, FP_RECIP_ONES>), cyl_grid(g),
                           dim3(PROJ_THREADS), 0, s, g, c, nullptr, static_cast<float *>(out),
                           ex);
        return hipGetLastError();
    }
    switch (vol_dtype) {
    case F32: return fp_cyl_out<float>(g, c, vol, out, out_dtype, mode, ex, s);
    case BF16: return fp_cyl_out<bf16_t>(g, c, vol, out, out_dtype, mode, ex, s);
    case F16: return fp_cyl_out<_Float16>(g, c, vol, out, out_dtype, mode, ex, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sample_count_cyl(const RayGrid &g, const CylGrid &c, unsigned long long *count,
                                   hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(count_cyl_kernel, cyl_grid(g), dim3(PROJ_THREADS), 0, s, g, c, count);
    return hipGetLastError();
}

int cyl_view_group(int nr, int nphi, int nz, int vol_dtype) {
    const long long bytes = 2ll * nr * nphi * nz;
    return vol_dtype != F32 && bytes > (4ll << 20) ? INT_MAX : 0;
}

CylGrid make_cyl_grid(int nr, int nphi, int nz, double dr, double dz) {
    CylGrid c;
    c.nr = nr;
    c.nphi = nphi;
    c.nz = nz;
    c.inv_dr = static_cast<float>(1.0 / dr);
    c.inv_dz = static_cast<float>(1.0 / dz);
    c.half_z = static_cast<float>(0.5 * (nz - 1));
    c.phi_scale2 = static_cast<float>(2.0 * nphi / kTwoPi);
    c.full = static_cast<float>(nphi);
    c.half = static_cast<float>(0.5 * nphi);
    c.quarter = static_cast<float>(0.25 * nphi);
    const double rh = (nr - 0.5) * dr;
    c.rh2 = rh * rh;
    c.hz = 0.5 * (nz - 1) * dz;
    return c;
}

}  // namespace ctrex
