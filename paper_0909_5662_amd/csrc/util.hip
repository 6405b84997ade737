// Element-wise utilities: the split-BF16 operand format (x = hi + lo with
// hi = bf16(x), lo = bf16(x - hi), both rounded to nearest even; x - hi is
// exact in FP32) and a zero-fill kernel that is safe under stream capture.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rot_internal.h"

namespace rot {
namespace {

// FP32 -> BF16 round to nearest even (the hardware conversion,
// v_cvt_pk_bf16_f32), as a bit pattern.
__device__ inline uint16_t rne_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__global__ void split_kernel(const float* __restrict__ x, int64_t n, uint16_t* __restrict__ hi,
                             uint16_t* __restrict__ lo) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = x[i];
    const uint16_t h = rne_bf16(v);
    hi[i] = h;
    lo[i] = rne_bf16(v - bf16_to_f32(h));
}

__global__ void zero_kernel(uint32_t* __restrict__ p, int64_t words) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

__global__ void zero_bytes_kernel(unsigned char* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// dst[i] = (accumulate ? dst[i] : 0) + part_0[i] + part_1[i] + ... in that
// fixed order (parts `stride` elements apart), so split-K results do not
// depend on scheduling.
template <typename T>
__global__ void sum_parts_kernel(T* __restrict__ dst, const T* __restrict__ src, int64_t n, int parts,
                                 int64_t stride, bool accumulate) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        T acc = accumulate ? dst[i] : T(0);
#pragma unroll 8
        for (int p = 0; p < parts; p++) acc += src[i + p * stride];
        dst[i] = acc;
    }
}

// dst[b][r][c] (row stride ld, matrix stride bs) = sum over p of
// src[p*pstride + (b*rows + r)*cols + c], in ascending p (deterministic).
template <typename T>
__global__ void sum_parts_2d_kernel(T* __restrict__ dst, int64_t ld, int64_t bs, const T* __restrict__ src, int rows,
                                    int cols, int64_t n, int parts, int64_t pstride) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / ((int64_t)rows * cols);
        const int64_t rc = i - b * rows * cols;
        const int64_t r = rc / cols, c = rc - r * cols;
        T acc = T(0);
#pragma unroll 8
        for (int p = 0; p < parts; p++) acc += src[i + p * pstride];
        dst[b * bs + r * ld + c] = acc;
    }
}

// out[i][j] = sum over b of src[b][i][j], FP64 additions: four waves take the
// matrices b = wave, wave + 4, ..., their sums are added in wave order.  A
// workgroup covers 64 groups of V columns of one row.  Bound by the one read
// of the matrices.
template <typename T, int V>
__global__ __launch_bounds__(256) void sum_matrices_kernel(T* __restrict__ dst, const T* __restrict__ src, int m,
                                                           int64_t ld, int64_t bs, int n) {
    typedef T VT __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    __shared__ double red[4][64 * V];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.y, j = (blockIdx.x * 64 + lane) * V;
    const T* p = src + (int64_t)i * ld + j;
    double acc[V];
#pragma unroll
    for (int e = 0; e < V; e++) acc[e] = 0.0;
    if (j + V <= m) {
#pragma unroll 8
        for (int b = wave; b < n; b += 4) {
            const VT v = *reinterpret_cast<const VT*>(p + (int64_t)b * bs);
#pragma unroll
            for (int e = 0; e < V; e++) acc[e] += (double)v[e];
        }
    } else {
        for (int b = wave; b < n; b += 4)
#pragma unroll
            for (int e = 0; e < V; e++)
                if (j + e < m) acc[e] += (double)p[(int64_t)b * bs + e];
    }
#pragma unroll
    for (int e = 0; e < V; e++) red[wave][lane * V + e] = acc[e];
    __syncthreads();
    for (int x = threadIdx.x; x < 64 * V; x += 256) {
        const int c = blockIdx.x * 64 * V + x;
        if (c < m) dst[(int64_t)i * m + c] = (T)(((red[0][x] + red[1][x]) + red[2][x]) + red[3][x]);
    }
}

// Element i of the first matrix to the n - 1 that follow it.
template <typename T, int V>
__global__ __launch_bounds__(256) void repeat_kernel(T* __restrict__ dst, int64_t count, int n) {
    typedef T VT __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= count) return;
    const int b0 = 1 + blockIdx.y * 8, b1 = min(b0 + 8, n);
    if (i + V <= count) {
        const VT v = *reinterpret_cast<const VT*>(dst + i);
        for (int b = b0; b < b1; b++) *reinterpret_cast<VT*>(dst + (int64_t)b * count + i) = v;
    } else {
        for (int64_t k = i; k < count; k++)
            for (int b = b0; b < b1; b++) dst[(int64_t)b * count + k] = dst[k];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void add_transpose_kernel(T* __restrict__ dst, const T* __restrict__ G, int mp) {
    __shared__ T tile[32][33];
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int k = ty; k < 32; k += 8)
        tile[k][tx] = c0 + k < mp && r0 + tx < mp ? G[(int64_t)(c0 + k) * mp + r0 + tx] : T(0);
    __syncthreads();
    for (int k = ty; k < 32; k += 8)
        if (r0 + k < mp && c0 + tx < mp)
            dst[(int64_t)(r0 + k) * mp + c0 + tx] = G[(int64_t)(r0 + k) * mp + c0 + tx] + tile[tx][k];
}

}  // namespace

hipError_t sum_matrices(void* dst, const void* src, int m, int64_t ld, int64_t bs, int n, bool is_double,
                        hipStream_t stream) {
    const int v = is_double ? 2 : 4;
    const dim3 grid((unsigned)((m + 64 * v - 1) / (64 * v)), (unsigned)m);
    if (is_double)
        hipLaunchKernelGGL((sum_matrices_kernel<double, 2>), grid, dim3(256), 0, stream, static_cast<double*>(dst),
                           static_cast<const double*>(src), m, ld, bs, n);
    else
        hipLaunchKernelGGL((sum_matrices_kernel<float, 4>), grid, dim3(256), 0, stream, static_cast<float*>(dst),
                           static_cast<const float*>(src), m, ld, bs, n);
    return hipGetLastError();
}

hipError_t repeat(void* dst, int64_t count, int n, bool is_double, hipStream_t stream) {
    if (n < 2 || count <= 0) return hipSuccess;
    const int v = is_double ? 2 : 4;
    const dim3 grid((unsigned)((count + 256 * v - 1) / (256 * v)), (unsigned)((n - 1 + 7) / 8));
    if (is_double)
        hipLaunchKernelGGL((repeat_kernel<double, 2>), grid, dim3(256), 0, stream, static_cast<double*>(dst), count, n);
    else
        hipLaunchKernelGGL((repeat_kernel<float, 4>), grid, dim3(256), 0, stream, static_cast<float*>(dst), count, n);
    return hipGetLastError();
}

hipError_t add_transpose(void* dst, const void* G, int mp, bool is_double, hipStream_t stream) {
    const dim3 grid((unsigned)((mp + 31) / 32), (unsigned)((mp + 31) / 32));
    if (is_double)
        hipLaunchKernelGGL(add_transpose_kernel<double>, grid, dim3(256), 0, stream, static_cast<double*>(dst),
                           static_cast<const double*>(G), mp);
    else
        hipLaunchKernelGGL(add_transpose_kernel<float>, grid, dim3(256), 0, stream, static_cast<float*>(dst),
                           static_cast<const float*>(G), mp);
    return hipGetLastError();
}

hipError_t sum_parts_2d(void* dst, int64_t ld, int64_t bs, const void* src, int rows, int cols, int nmat, int parts,
                        int64_t pstride, bool is_double, hipStream_t stream) {
    const int64_t n = (int64_t)rows * cols * nmat;
    if (n <= 0) return hipSuccess;
    const dim3 grid((unsigned)std::min<int64_t>((n + 255) / 256, 8192));
    if (is_double)
        hipLaunchKernelGGL(sum_parts_2d_kernel<double>, grid, dim3(256), 0, stream, static_cast<double*>(dst), ld, bs,
                           static_cast<const double*>(src), rows, cols, n, parts, pstride);
    else
        hipLaunchKernelGGL(sum_parts_2d_kernel<float>, grid, dim3(256), 0, stream, static_cast<float*>(dst), ld, bs,
                           static_cast<const float*>(src), rows, cols, n, parts, pstride);
    return hipGetLastError();
}

hipError_t sum_parts(void* dst, const void* src, int64_t n, int parts, int64_t stride, bool accumulate,
                     bool is_double, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((unsigned)std::min<int64_t>((n + 255) / 256, 8192));
    if (is_double)
        hipLaunchKernelGGL(sum_parts_kernel<double>, grid, dim3(256), 0, stream, static_cast<double*>(dst),
                           static_cast<const double*>(src), n, parts, stride, accumulate);
    else
        hipLaunchKernelGGL(sum_parts_kernel<float>, grid, dim3(256), 0, stream, static_cast<float*>(dst),
                           static_cast<const float*>(src), n, parts, stride, accumulate);
    return hipGetLastError();
}

hipError_t split_bf16(const float* x, int64_t n, uint16_t* hi, uint16_t* lo, hipStream_t stream) {
    hipLaunchKernelGGL(split_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, x, n, hi, lo);
    return hipGetLastError();
}

hipError_t fill_zero(void* p, int64_t bytes, hipStream_t stream) {
    if (bytes <= 0) return hipSuccess;
    if ((reinterpret_cast<uintptr_t>(p) & 3) == 0 && bytes % 4 == 0) {
        const int64_t words = bytes / 4;
        const int64_t blocks = std::min<int64_t>((words + 255) / 256, 4096);
        hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                           static_cast<uint32_t*>(p), words);
    } else {
        hipLaunchKernelGGL(zero_bytes_kernel, dim3((unsigned)((bytes + 255) / 256)), dim3(256), 0, stream,
                           static_cast<unsigned char*>(p), bytes);
    }
    return hipGetLastError();
}

}  // namespace rot
