// Voxel-space and bookkeeping kernels of the SIRT loop (Eq. 1, term 3):
// x <- x + alpha C z with z = A^T r, the reciprocal weights, the 16-bit gather
// shadows, and deterministic reductions of the per-block residual sums.
// All are single streams over HBM: 64-bit-indexed grid-stride loops over
// elements (no alignment is asked of the arrays).

#include "ctrex_internal.h"

namespace ctrex {
namespace {

constexpr int THREADS = 256;

__device__ __forceinline__ uint16_t bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ float load_as_f32(const void *p, int dt, size_t i) {
    if (dt == F32) return static_cast<const float *>(p)[i];
    if (dt == BF16)
        return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(p)[i]) << 16);
    return static_cast<float>(static_cast<const _Float16 *>(p)[i]);
}

__device__ __forceinline__ void store_from_f32(void *p, int dt, size_t i, float v) {
    if (dt == F32)
        static_cast<float *>(p)[i] = v;
    else if (dt == BF16)
        static_cast<uint16_t *>(p)[i] = bf16_rne(v);
    else
        static_cast<_Float16 *>(p)[i] = static_cast<_Float16>(v);
}

inline unsigned grid_for(size_t n) {
    size_t b = (n + THREADS - 1) / THREADS;
    if (b > 65536) b = 65536;
    if (b == 0) b = 1;
    return static_cast<unsigned>(b);
}

// Grid of a stream whose threads take four elements per pass, so that four
// loads of each array are in flight before the first is used: at most 8
// workgroups per CU, which stay for the whole array.
inline unsigned grid_for4(size_t n) {
    size_t b = (n + 4 * THREADS - 1) / (4 * THREADS);
    if (b > 2048) b = 2048;
    if (b == 0) b = 1;
    return static_cast<unsigned>(b);
}

__global__ __launch_bounds__(THREADS) void fill_zero_kernel(uint32_t *p, size_t n_words) {
    const size_t stride = static_cast<size_t>(gridDim.x) * THREADS;
    for (size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x; i < n_words; i += stride)
        p[i] = 0u;
}

__global__ __launch_bounds__(THREADS) void fill_zero_bytes_kernel(uint8_t *p, size_t n) {
    const size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ __launch_bounds__(THREADS) void recip_kernel(float *a, size_t n) {
    const size_t stride = static_cast<size_t>(gridDim.x) * THREADS;
    for (size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x; i < n; i += stride) {
        const float v = a[i];
        a[i] = v > 0.0f ? 1.0f / v : 0.0f;
    }
}

// x <- x + alpha C w z (w: optional voxel weights; optionally clamped at 0),
// shadow <- x.  Four voxels per pass: 61 -> 44 us at 256^3
// (268 MB moved, 4.4 -> 6.0 TB/s) against one voxel a thread in 65536 workgroups.
__global__ __launch_bounds__(THREADS) void update_kernel(float *__restrict__ x,
                                                         const float *__restrict__ z,
                                                         const float *__restrict__ C,
                                                         const float *__restrict__ w, float alpha,
                                                         int nonneg, void *shadow, int sdt,
                                                         size_t n) {
    const size_t stride = static_cast<size_t>(gridDim.x) * THREADS;
    size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x;
    auto put = [&](size_t j, float c, float wj, float zj, float xj) {
        const float g = w ? alpha * c * wj : alpha * c;
        float v = fmaf(g, zj, xj);
        if (nonneg) v = fmaxf(v, 0.0f);
        x[j] = v;
        if (shadow) store_from_f32(shadow, sdt, j, v);
    };
    for (; i + 3 * stride < n; i += 4 * stride) {
        float c[4], wv[4], zv[4], xv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const size_t j = i + k * stride;
            c[k] = C[j];
            wv[k] = w ? w[j] : 0.0f;
            zv[k] = z[j];
            xv[k] = x[j];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) put(i + k * stride, c[k], wv[k], zv[k], xv[k]);
    }
    for (; i < n; i += stride) put(i, C[i], w ? w[i] : 0.0f, z[i], x[i]);
}

__global__ __launch_bounds__(THREADS) void convert_kernel(const void *src, int sdt, void *dst,
                                                          int ddt, size_t n) {
    const size_t stride = static_cast<size_t>(gridDim.x) * THREADS;
    for (size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x; i < n; i += stride)
        store_from_f32(dst, ddt, i, load_as_f32(src, sdt, i));
}

// One block: fixed-order sum of n doubles (each thread strides, then a tree).
__global__ __launch_bounds__(1024) void sum_partials_kernel(const double *p, int n, double *out) {
    __shared__ double red[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += p[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// Block max of |x| folded into *out with an integer max on the float bits
// (non-negative floats order like their bit patterns); NaN propagates as the
// largest pattern.  Four elements per pass and at most 2048 workgroups: every
// workgroup ends in an atomic on the one word, and those took longer than the
// loads (9 images of 384 x 384: 49 -> 17 us, from up to 4096 workgroups of
// one element per pass).
__global__ __launch_bounds__(THREADS) void max_abs_kernel(const void *x, int dt, size_t n,
                                                          unsigned *out) {
    __shared__ unsigned red[THREADS / 64];
    unsigned m = 0u;
    const size_t stride = static_cast<size_t>(gridDim.x) * THREADS;
    size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = load_as_f32(x, dt, i + k * stride);
#pragma unroll
        for (int k = 0; k < 4; ++k) m = max(m, __float_as_uint(fabsf(v[k])));
    }
    for (; i < n; i += stride) m = max(m, __float_as_uint(fabsf(load_as_f32(x, dt, i))));
    for (int o = 32; o > 0; o >>= 1) m = max(m, static_cast<unsigned>(__shfl_xor(m, o, 64)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < THREADS / 64; ++i) m = max(m, red[i]);
        atomicMax(out, m);
    }
}

__global__ __launch_bounds__(THREADS) void repack_warp_kernel(const float *U, float4 *out,
                                                              size_t n) {
    const size_t i = static_cast<size_t>(blockIdx.x) * THREADS + threadIdx.x;
    if (i < n) out[i] = make_float4(U[3 * i], U[3 * i + 1], U[3 * i + 2], 0.0f);
}

// Pair-packed copies (FpExtra): px element (x, y, z) holds v(x, y), v(x, y+1),
// x fastest; py element (y, x, z) holds v(x, y), v(x+1, y), y fastest (indices
// clamped at the last row and column, whose second values the gathers never
// read).  A block stages a 32 x 32 tile of one slice and its high-side border
// in LDS and writes both copies from it, so the volume is read once and every
// access is coalesced.  Bound by HBM: 4 bytes in, 16 out per FP32 voxel.
template <typename T> struct PairOf;
template <> struct PairOf<float> {
    typedef float2 type;
    static __device__ __forceinline__ float2 make(float a, float b) { return make_float2(a, b); }
};
template <> struct PairOf<uint16_t> {
    typedef uint32_t type;
    static __device__ __forceinline__ uint32_t make(uint16_t a, uint16_t b) {
        return a | (static_cast<uint32_t>(b) << 16);
    }
};

// PERIODIC (polar volumes, x = ring, y = angle): y wraps around, and py's rows
// hold ny + 1 elements, the last repeating the first.
template <typename T, bool PERIODIC>
__global__ __launch_bounds__(THREADS) void pack_pairs_kernel(const T *__restrict__ v,
                                                             typename PairOf<T>::type *__restrict__ px,
                                                             typename PairOf<T>::type *__restrict__ py,
                                                             int nx, int ny, int tiles_x,
                                                             int tiles_y, unsigned tiles) {
    __shared__ T tile[33][34];
    const int c = threadIdx.x & 31, r = threadIdx.x >> 5;   // 32 x 8
    for (unsigned t = blockIdx.x; t < tiles; t += gridDim.x) {
        const unsigned q = t / tiles_x;
        const int x0 = static_cast<int>(t - q * tiles_x) * 32;
        const unsigned z = q / tiles_y;
        const int y0 = static_cast<int>(q - z * tiles_y) * 32;
        const size_t plane = static_cast<size_t>(z) * nx * ny;
        if (t != blockIdx.x) __syncthreads();   // the previous tile's reads are done
        for (int i = threadIdx.x; i < 33 * 33; i += THREADS) {
            const int j = i / 33, k = i - j * 33;
            const int x = min(x0 + k, nx - 1);
            const int y = PERIODIC ? (y0 + j) % ny : min(y0 + j, ny - 1);
            tile[j][k] = v[plane + static_cast<size_t>(y) * nx + x];
        }
        __syncthreads();
#pragma unroll
        for (int j = r; j < 32; j += 8) {
            const int x = x0 + c, y = y0 + j;
            if (x < nx && y < ny)
                px[plane + static_cast<size_t>(y) * nx + x] =
                    PairOf<T>::make(tile[j][c], tile[j + 1][c]);
            const int xt = x0 + j, yt = y0 + c, rows = PERIODIC ? ny + 1 : ny;
            if (xt < nx && yt < rows)
                py[(static_cast<size_t>(z) * nx + xt) * rows + yt] =
                    PairOf<T>::make(tile[c][j], tile[c][j + 1]);
        }
    }
}

}  // namespace

hipError_t launch_pack_polar(const float *vol, float2 *px, float2 *py, int nr, int nphi, int nz,
                             hipStream_t s) {
    if (nr <= 0 || nphi <= 0 || nz <= 0) return hipSuccess;
    const int tx = (nr + 31) / 32, ty = (nphi + 32) / 32;
    const unsigned long long all = static_cast<unsigned long long>(tx) * ty * nz;
    const unsigned tiles = static_cast<unsigned>(all);   // no more than there are voxels: below 2^31
    const dim3 grid(tiles < (1u << 20) ? tiles : (1u << 20)), block(THREADS);
    hipLaunchKernelGGL((pack_pairs_kernel<float, true>), grid, block, 0, s, vol, px, py, nr, nphi,
                       tx, ty, tiles);
    return hipGetLastError();
}

hipError_t launch_pack_pairs(const void *vol, int dtype, void *px, void *py, int nx, int ny, int nz,
                             hipStream_t s) {
    if (nx <= 0 || ny <= 0 || nz <= 0) return hipSuccess;
    const int tx = (nx + 31) / 32, ty = (ny + 31) / 32;
    // fewer tiles than voxels, so below 2^31
    const unsigned tiles = static_cast<unsigned>(tx) * static_cast<unsigned>(ty) * static_cast<unsigned>(nz);
    const dim3 grid(tiles < (1u << 20) ? tiles : (1u << 20)), block(THREADS);
    if (dtype == F32)
        hipLaunchKernelGGL((pack_pairs_kernel<float, false>), grid, block, 0, s,
                           static_cast<const float *>(vol), static_cast<float2 *>(px),
                           static_cast<float2 *>(py), nx, ny, tx, ty, tiles);
    else
        hipLaunchKernelGGL((pack_pairs_kernel<uint16_t, false>), grid, block, 0, s,
                           static_cast<const uint16_t *>(vol), static_cast<uint32_t *>(px),
                           static_cast<uint32_t *>(py), nx, ny, tx, ty, tiles);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    const size_t words = bytes / 4;
    if (words) hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(words)), dim3(THREADS), 0, s,
                                  static_cast<uint32_t *>(ptr), words);
    const size_t tail = bytes - words * 4;
    if (tail)
        hipLaunchKernelGGL(fill_zero_bytes_kernel, dim3(1), dim3(THREADS), 0, s,
                           static_cast<uint8_t *>(ptr) + words * 4, tail);
    return hipGetLastError();
}

hipError_t launch_recip(float *a, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(recip_kernel, dim3(grid_for(n)), dim3(THREADS), 0, s, a, n);
    return hipGetLastError();
}

hipError_t launch_update(float *x, const float *z, const float *C, const float *w, float alpha,
                         int nonneg, void *shadow, int shadow_dtype, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(update_kernel, dim3(grid_for4(n)), dim3(THREADS), 0, s, x, z, C, w, alpha,
                       nonneg, shadow, shadow_dtype, n);
    return hipGetLastError();
}

hipError_t launch_convert(const void *src, int src_dtype, void *dst, int dst_dtype, size_t n,
                          hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(convert_kernel, dim3(grid_for(n)), dim3(THREADS), 0, s, src, src_dtype,
                       dst, dst_dtype, n);
    return hipGetLastError();
}

hipError_t launch_sum_partials(const double *partials, int n, double *out, hipStream_t s) {
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(1024), 0, s, partials, n, out);
    return hipGetLastError();
}

hipError_t launch_max_abs(const void *x, int dtype, size_t n, float *out, hipStream_t s) {
    hipError_t e = launch_fill_zero(out, sizeof(float), s);
    if (e != hipSuccess || n == 0) return e;
    hipLaunchKernelGGL(max_abs_kernel, dim3(grid_for4(n)), dim3(THREADS), 0, s, x, dtype, n,
                       reinterpret_cast<unsigned *>(out));
    return hipGetLastError();
}

hipError_t launch_repack_warp(const float *U, float4 *out, size_t n_nodes, hipStream_t s) {
    if (n_nodes == 0) return hipSuccess;
    hipLaunchKernelGGL(repack_warp_kernel, dim3((n_nodes + THREADS - 1) / THREADS), dim3(THREADS),
                       0, s, U, out, n_nodes);
    return hipGetLastError();
}

}  // namespace ctrex
