// Superblock measurements in FP64 (one-point values of block operators and
// products of operators of the two blocks): the reductions that follow the
// products done by the GEMM kernels.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rot_internal.h"

namespace rot {
namespace {

constexpr int kDotParts = 8;  // workgroups per operator

// partial[b][p] = sum over elements e = p*256*... of Z_b[e] * rho[e] in FP64:
// workgroup (p, b) takes the strided elements tid + 256*(p + kDotParts*q).
// Bound by the read of Z, with eight elements' loads in flight (65 FP32
// operators of 400 states: one at a time 34 us, now 18).
template <typename T>
__global__ __launch_bounds__(256) void dot_partial_kernel(const T* __restrict__ Z, int64_t stride_z, int64_t n,
                                                          const double* __restrict__ rho, double* __restrict__ partial) {
    __shared__ double red[256];
    const int p = blockIdx.x, b = blockIdx.y;
    const T* z = Z + (int64_t)b * stride_z;
    double acc = 0.0;
    constexpr int64_t kStep = (int64_t)kDotParts * 256;
    constexpr int kAhead = 8;
    int64_t e = (int64_t)p * 256 + threadIdx.x;
    for (; e + (kAhead - 1) * kStep < n; e += kAhead * kStep) {
        T x[kAhead];
        double y[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; q++) {
            x[q] = z[e + q * kStep];
            y[q] = rho[e + q * kStep];
        }
#pragma unroll
        for (int q = 0; q < kAhead; q++) acc += (double)x[q] * y[q];
    }
    for (; e < n; e += kStep) acc += (double)z[e] * rho[e];
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

constexpr int kPairTile = 8;

// Sums of the 64 values of all lanes, lane l ending with that of value l: each
// step hands half of the values left to the lane across and adds its half.
template <int S>
__device__ __attribute__((always_inline)) inline double transpose_sum(const double (&v)[2 * S], int lane) {
    const bool upper = lane & S;
    double half[S];
#pragma unroll
    for (int k = 0; k < S; k++) {
        const double keep = upper ? v[k + S] : v[k], send = upper ? v[k] : v[k + S];
        half[k] = keep + __shfl_xor(send, S, 64);
    }
    if constexpr (S > 1) return transpose_sum<S / 2>(half, lane);
    else return half[0];
}

// partial[p][b][k] = sum over e of part p of Q_b[e] W_k[e] in FP64, 8 x 8 pairs
// (b, k) per workgroup (p, pair tile): a product with so few rows and columns
// leaves a matrix tile almost empty.  Bound by latency: every element is read
// once per eight of the other side (6 x 7 operators of 380 states: 49 us as a
// product in 256 K parts plus 10 us for their sum; now 13).
__global__ __launch_bounds__(256) void cross_partial_kernel(const double* __restrict__ Q, int64_t stride_q, int nl,
                                                            const double* __restrict__ W, int64_t stride_w, int nr,
                                                            int64_t n, int parts, double* __restrict__ partial) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tk = (nr + kPairTile - 1) / kPairTile;
    const int b0 = (blockIdx.y / tk) * kPairTile, k0 = (blockIdx.y % tk) * kPairTile;
    const int p = blockIdx.x;
    const int64_t e1 = n * (p + 1) / parts;
    double v[64];
#pragma unroll
    for (int i = 0; i < 64; i++) v[i] = 0.0;
    for (int64_t e = n * p / parts + threadIdx.x; e < e1; e += 256) {
        double x[kPairTile], y[kPairTile];
        // operators past the last repeat it (their pairs are not stored)
#pragma unroll
        for (int i = 0; i < kPairTile; i++) {
            x[i] = Q[min(b0 + i, nl - 1) * stride_q + e];
            y[i] = W[min(k0 + i, nr - 1) * stride_w + e];
        }
#pragma unroll
        for (int i = 0; i < kPairTile; i++)
#pragma unroll
            for (int j = 0; j < kPairTile; j++) v[i * kPairTile + j] = fma(x[i], y[j], v[i * kPairTile + j]);
    }
    red[wave][lane] = transpose_sum<32>(v, lane);
    __syncthreads();
    const int b = b0 + lane / kPairTile, k = k0 + lane % kPairTile;
    if (wave == 0 && b < nl && k < nr)
        partial[((int64_t)p * nl + b) * nr + k] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// c[i] = sum over the parts, one wave per pair.
__global__ __launch_bounds__(64) void cross_final_kernel(const double* __restrict__ partial, int64_t n_pairs, int parts,
                                                         double* __restrict__ c) {
    const int64_t i = blockIdx.x;
    double acc = 0.0;
    for (int p = threadIdx.x; p < parts; p += 64) acc += partial[p * n_pairs + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (threadIdx.x == 0) c[i] = acc;
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

// c[b][k] = sum over n elements of Q_b W_k, nl x nr pairs; scratch: as many parts
// as it holds, of 512 elements and more (none: one part, straight into c).
hipError_t cross_dots(const double* Q, int64_t stride_q, int nl, const double* W, int64_t stride_w, int nr, int64_t n,
                      double* c, void* scratch, size_t scratch_bytes, hipStream_t s) {
    const int64_t pairs = (int64_t)nl * nr;
    const int64_t tiles = (int64_t)((nl + kPairTile - 1) / kPairTile) * ((nr + kPairTile - 1) / kPairTile);
    const int64_t fit = (int64_t)(scratch_bytes / ((size_t)pairs * sizeof(double)));
    const int parts = (int)std::max<int64_t>(1, std::min<int64_t>({n / 512, fit, 1024}));
    double* out = parts > 1 ? static_cast<double*>(scratch) : c;
    hipLaunchKernelGGL(cross_partial_kernel, dim3((unsigned)parts, (unsigned)tiles), dim3(256), 0, s, Q, stride_q, nl, W,
                       stride_w, nr, n, parts, out);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || parts == 1) return err;
    hipLaunchKernelGGL(cross_final_kernel, dim3((unsigned)pairs), dim3(64), 0, s, out, pairs, parts, c);
    return hipGetLastError();
}

hipError_t sum_groups(double* dst, const void* src, int64_t count, int groups, int nmat, hipStream_t s) {
    if (nmat <= 0) return hipSuccess;
    const dim3 grid((unsigned)((count + 255) / 256), (unsigned)nmat);
    hipLaunchKernelGGL(sum_groups_kernel, grid, dim3(256), 0, s, dst, static_cast<const double*>(src), count, groups);
    return hipGetLastError();
}

}  // namespace rot
