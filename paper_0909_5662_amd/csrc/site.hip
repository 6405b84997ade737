// Operators blocked together with the added site, out = U^T (X (x) S) U:
// the sum over the site index is folded into the stage-2 operand,
//   U'[(i,t), alpha] = x_i sum_s S[s,t] U[(i,s), alpha]  =  ((diag(x) (x) S^T) U)[(i,t), alpha],
// so that out = U'^T (X U_r) for a dense block operator X and out = U'^T U
// for X = diag(x) (the identity when x is absent).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rot_internal.h"

namespace rot {
namespace {

// Bound by the read of U and the write of U'.  A thread takes one column of
// the d rows of one i, so U is read once (D: d if it is 4 or 2, else 0 and
// each U' entry reads its d entries of U); 500 states, d = 4, kept 480: one
// entry per thread 7.1 us, now 4.9.
template <typename T, int D>
__global__ __launch_bounds__(256) void site_mix_kernel(const T* __restrict__ U, int m, int d, int mp, SiteMatrix S,
                                                       const T* __restrict__ x, T* __restrict__ Up) {
    const int a = blockIdx.x * 64 + (threadIdx.x & 63);
    if (a >= mp) return;
    for (int64_t i = blockIdx.y * 4 + (threadIdx.x >> 6); i < m; i += (int64_t)gridDim.y * 4) {
        const T* u = U + i * (D ? D : d) * mp + a;  // U[(i, 0), a]
        T* up = Up + i * (D ? D : d) * mp + a;
        const T f = x ? x[i] : T(1);
        if (D) {
            T v[D ? D : 1];
#pragma unroll
            for (int s = 0; s < D; s++) v[s] = u[(int64_t)s * mp];
#pragma unroll
            for (int t = 0; t < D; t++) {
                T acc = T(0);
#pragma unroll
                for (int s = 0; s < D; s++) acc += (T)S.v[s * D + t] * v[s];
                up[(int64_t)t * mp] = x ? f * acc : acc;
            }
        } else {
            for (int t = 0; t < d; t++) {
                T acc = T(0);
                for (int s = 0; s < d; s++) acc += (T)S.v[s * d + t] * u[(int64_t)s * mp];
                up[(int64_t)t * mp] = x ? f * acc : acc;
            }
        }
    }
}

template <typename T>
void launch_mix(const void* U, int m, int d, int mp, const SiteMatrix& S, const void* x, void* Up, hipStream_t s) {
    const dim3 grid((unsigned)((mp + 63) / 64), (unsigned)std::min((m + 3) / 4, 16384)), block(256);
    const T *u = static_cast<const T*>(U), *xs = static_cast<const T*>(x);
    T* up = static_cast<T*>(Up);
    if (d == 4)
        hipLaunchKernelGGL((site_mix_kernel<T, 4>), grid, block, 0, s, u, m, d, mp, S, xs, up);
    else if (d == 2)
        hipLaunchKernelGGL((site_mix_kernel<T, 2>), grid, block, 0, s, u, m, d, mp, S, xs, up);
    else
        hipLaunchKernelGGL((site_mix_kernel<T, 0>), grid, block, 0, s, u, m, d, mp, S, xs, up);
}

}  // namespace

hipError_t site_mix(const void* U, int m, int d, int mp, const SiteMatrix& S, const void* x, void* Up,
                    bool is_double, hipStream_t stream) {
    if (m <= 0 || mp <= 0) return hipSuccess;
    if (is_double)
        launch_mix<double>(U, m, d, mp, S, x, Up, stream);
    else
        launch_mix<float>(U, m, d, mp, S, x, Up, stream);
    return hipGetLastError();
}

}  // namespace rot
