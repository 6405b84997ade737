// Superblock measurements in FP64 (one-point values of block operators and
// products of operators of the two blocks): the reductions that follow the
// products done by the GEMM kernels.
#include <hip/hip_runtime.h>

#include "rot_internal.h"

namespace rot {
namespace {

constexpr int kDotParts = 8;  // workgroups per operator

// partial[b][p] = sum over elements e = p*256*... of Z_b[e] * rho[e] in FP64:
// workgroup (p, b) takes the strided elements tid + 256*(p + kDotParts*q).
template <typename T>
__global__ __launch_bounds__(256) void dot_partial_kernel(const T* __restrict__ Z, int64_t stride_z, int64_t n,
                                                          const double* __restrict__ rho, double* __restrict__ partial) {
    __shared__ double red[256];
    const int p = blockIdx.x, b = blockIdx.y;
    const T* z = Z + (int64_t)b * stride_z;
    double acc = 0.0;
    for (int64_t e = (int64_t)p * 256 + threadIdx.x; e < n; e += (int64_t)kDotParts * 256)
        acc += (double)z[e] * rho[e];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(int64_t)b * kDotParts + p] = red[0];
}

__global__ void dot_final_kernel(const double* __restrict__ partial, int n_ops, double* __restrict__ e) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_ops) return;
    double acc = 0.0;
    for (int p = 0; p < kDotParts; p++) acc += partial[(int64_t)b * kDotParts + p];
    e[b] = acc;
}

__global__ __launch_bounds__(256) void sum_groups_kernel(double* __restrict__ dst, const double* __restrict__ src,
                                                         int64_t count, int groups) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const int b = blockIdx.y;
    const double* p = src + (int64_t)b * groups * count + i;
    double acc = 0.0;
#pragma unroll 4
    for (int x = 0; x < groups; x++) acc += p[(int64_t)x * count];
    dst[(int64_t)b * count + i] = acc;
}

}  // namespace

size_t expect_dot_scratch(int n_ops) { return (size_t)n_ops * kDotParts * sizeof(double); }

hipError_t expect_dots(const void* Z, bool z_double, int64_t stride_z, int64_t n, int n_ops, const double* rho,
                       double* partial, double* e, hipStream_t s) {
    if (n_ops <= 0) return hipSuccess;
    const dim3 grid(kDotParts, (unsigned)n_ops);
    if (z_double)
        hipLaunchKernelGGL(dot_partial_kernel<double>, grid, dim3(256), 0, s, static_cast<const double*>(Z), stride_z,
                           n, rho, partial);
    else
        hipLaunchKernelGGL(dot_partial_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(Z), stride_z, n,
                           rho, partial);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(dot_final_kernel, dim3((unsigned)((n_ops + 255) / 256)), dim3(256), 0, s, partial, n_ops, e);
    return hipGetLastError();
}

hipError_t sum_groups(double* dst, const void* src, int64_t count, int groups, int nmat, hipStream_t s) {
    if (nmat <= 0) return hipSuccess;
    const dim3 grid((unsigned)((count + 255) / 256), (unsigned)nmat);
    hipLaunchKernelGGL(sum_groups_kernel, grid, dim3(256), 0, s, dst, static_cast<const double*>(src), count, groups);
    return hipGetLastError();
}

}  // namespace rot
