// Batched FP32 / FP64 products in 64 x 64 tiles on CDNA4 matrix cores: every
// layout, extent and alignment of GemmDesc (the direct-to-LDS FP32 kernel of
// gemm.hip takes the large aligned products).
//
// A workgroup of four waves owns a tile, each wave 32 x 32 of it (one
// v_mfma_f32_32x32x2f32 block, or 2 x 2 of v_mfma_f64_16x16x4f64), and walks
// K in slices of 16 through two LDS buffers with the next two slices in
// registers.  The matrix instructions of either type take 64 cycles, so a
// 32 x 32 block per wave asks little of the LDS (about 32 bytes per cycle and
// CU); the small tile leaves room for four and more workgroups per CU, which
// hide each other's loads and barriers, and a ragged extent wastes at most
// 63 rows.  128 x 128 tiles before it, one or two workgroups per CU: FP64 rotation of
// 8 operators of 1024 states 2.33 -> 2.04 ms (67 of the 73 TFLOP/s that a
// large library product reaches here), 12 of 400: 464 -> 261 us, 16 of 128:
// 57.7 -> 30.6 us.
//
// Loads are 16-byte buffer loads through registers.  They need 4-byte
// alignment only, and a descriptor that ends with the operand returns zero,
// dword by dword, past it: no element-wise path at edges or odd strides.
//
// The assignment of k to the matrix instruction's k slots is permuted the same
// way for both operands (lane group h takes k = h*(16/groups) + j of a slice
// at step j), so slices are stored in LDS in their global orientation: a
// K-contiguous operand is read with 128-bit LDS loads, an M/N-contiguous one
// with loads contiguous across the lanes of a group.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "buffer_rsrc.h"
#include "lds_slice.h"
#include "rot_internal.h"

namespace rot {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kT = 64;   // tile edge
constexpr int kS = 16;   // k per slice

// How a kernel addresses its operands: one descriptor per operand and 32-bit
// offsets (kNear: a batch entry under 4 GiB, one K batch), a descriptor per
// slice (kRebase), or plain loads with bounds checks (kFar: row strides so
// long that offsets inside a slice pass 4 GiB).
enum Addr { kNear, kRebase, kFar };

// One operand slice of 64 rows (M or N extent) by 16 k in chunks of 16 bytes,
// NCH per thread.  K-contiguous (KC): rows of NQ chunks, chunk q of row r in
// slot q ^ ((r / RPB) % NQ), so that the stores and the fragment reads of 16
// lanes touch all 64 LDS banks once; otherwise k rows at a pitch of 64
// elements and one chunk.
template <typename T, bool KC, Addr ADDR>
struct Slice {
    typedef typename Vec16<T>::type V;
    static constexpr int VW = 16 / sizeof(T), NQ = kS / VW, RPB = 16 / NQ;
    static constexpr int NCH = kT * kS / VW / 256;
    static constexpr int PITCH = KC ? kS : kT + VW;
    static constexpr int ELEMS = KC ? kT * kS : kS * PITCH;
    V r[NCH];

    __device__ static inline int kc_off(int row, int q) { return row * kS + (q ^ ((row / RPB) % NQ)) * VW; }
    // row (M/N) and k of chunk x of this thread inside the slice
    __device__ static inline int row_of(int tid, int x) {
        return KC ? tid / NQ + (256 / NQ) * x : (tid % (kT / VW)) * VW;
    }
    __device__ static inline int k_of(int tid, int x) {
        return KC ? (tid % NQ) * VW : tid / (kT / VW) + (256 / (kT / VW)) * x;
    }

    // What a kernel keeps per operand.
    struct Source {
        const T* base;  // element (0, 0) of the operand's K batch
        int64_t ld;
        int r0, rows, ks;      // the tile's first row, the extents
        uint32_t off[NCH];     // byte offsets of this thread's chunks
        __amdgpu_buffer_rsrc_t rs;
        uint32_t step;         // kNear: bytes from one slice to the next

        // Descriptor from the tile's first element of slice k0 to the operand's end.
        __device__ inline __amdgpu_buffer_rsrc_t descriptor(const T* b, int k0) const {
            const T* p = b + (KC ? (int64_t)r0 * ld + k0 : (int64_t)k0 * ld + r0);
            const int64_t extent =
                KC ? (int64_t)(rows - 1 - r0) * ld + (ks - k0) : (int64_t)(ks - 1 - k0) * ld + (rows - r0);
            const int64_t bytes = extent * (int64_t)sizeof(T);
            return __builtin_amdgcn_make_buffer_rsrc(
                const_cast<T*>(p), (short)0, (int)(uint32_t)(bytes < 0 ? 0 : bytes > 0xffffffff ? 0xffffffff : bytes),
                kBufferFlags);
        }
        __device__ inline void init(const T* b, int64_t ld_, int r0_, int rows_, int ks_, int tid) {
            base = b;
            ld = ld_;
            r0 = r0_;
            rows = rows_;
            ks = ks_;
#pragma unroll
            for (int x = 0; x < NCH; x++)
                off[x] = ((uint32_t)(KC ? row_of(tid, x) : k_of(tid, x)) * (uint32_t)ld +
                          (uint32_t)(KC ? k_of(tid, x) : row_of(tid, x))) * (uint32_t)sizeof(T);
            if (ADDR == kNear) rs = descriptor(b, 0);
            step = (uint32_t)((KC ? kS : kS * ld) * (int64_t)sizeof(T));
        }
    };

    // Slice kt of K batch `kb` (ks_stride elements apart).
    __device__ inline void load(const Source& s, int kt, int kb, int64_t ks_stride, int tid) {
        const int k0 = kt * kS;
        const T* b = ADDR == kNear ? s.base : s.base + (int64_t)kb * ks_stride;
        if (ADDR == kFar) {
#pragma unroll
            for (int x = 0; x < NCH; x++)
#pragma unroll
                for (int e = 0; e < VW; e++) {
                    const int gr = s.r0 + row_of(tid, x) + (KC ? 0 : e), gk = k0 + k_of(tid, x) + (KC ? e : 0);
                    r[x][e] = gr < s.rows && gk < s.ks ? b[KC ? (int64_t)gr * s.ld + gk : (int64_t)gk * s.ld + gr] : T(0);
                }
            return;
        }
        const __amdgpu_buffer_rsrc_t rs = ADDR == kNear ? s.rs : s.descriptor(b, k0);
#pragma unroll
        for (int x = 0; x < NCH; x++)
            r[x] = __builtin_bit_cast(
                V, __builtin_amdgcn_raw_buffer_load_b128(rs, s.off[x], ADDR == kNear ? (int)((uint32_t)kt * s.step) : 0, 0));
        // a K-contiguous row is followed by the next row, not by zeros
        if (KC && k0 + kS > s.ks) {
#pragma unroll
            for (int x = 0; x < NCH; x++)
#pragma unroll
                for (int e = 0; e < VW; e++)
                    if (k0 + k_of(tid, x) + e >= s.ks) r[x][e] = T(0);
        }
    }
    __device__ inline void store(T* lds, int tid) const {
#pragma unroll
        for (int x = 0; x < NCH; x++) {
            const int row = row_of(tid, x), k = k_of(tid, x);
            *reinterpret_cast<V*>(lds + (KC ? kc_off(row, k / VW) : k * PITCH + row)) = r[x];
        }
    }
};

// A wave's accumulator for 32 x 32, its products over one slice, and the C
// position of its elements (relative to the wave's block).
template <typename T> struct Acc;
template <> struct Acc<float> {
    static constexpr int N = 16;
    f32x16 a;
    __device__ inline void clear() {
#pragma unroll
        for (int v = 0; v < 16; v++) a[v] = 0.f;
    }
    // v_mfma_f32_32x32x2f32: lane l supplies A(row l%32, k l/32), B(k l/32, col
    // l%32); element v of lane l is C(8*(v/4) + 4*(l/32) + v%4, l%32)
    __device__ static inline int row(int lane, int v) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
    __device__ static inline int col(int lane, int) { return lane & 31; }
    __device__ inline float at(int v) const { return a[v]; }
    template <typename SA, typename SB, bool AK, bool BK>
    __device__ inline void products(const float* as, const float* bs, int m, int n, int lane) {
        const int h = lane >> 5, c = lane & 31;
        float av[8], bv[8];
        if (AK) {
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(as + SA::kc_off(m + c, 2 * h));
            const f32x4 x1 = *reinterpret_cast<const f32x4*>(as + SA::kc_off(m + c, 2 * h + 1));
#pragma unroll
            for (int e = 0; e < 4; e++) { av[e] = x0[e]; av[4 + e] = x1[e]; }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) av[j] = as[(h * 8 + j) * SA::PITCH + m + c];
        }
        if (BK) {
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(bs + SB::kc_off(n + c, 2 * h));
            const f32x4 x1 = *reinterpret_cast<const f32x4*>(bs + SB::kc_off(n + c, 2 * h + 1));
#pragma unroll
            for (int e = 0; e < 4; e++) { bv[e] = x0[e]; bv[4 + e] = x1[e]; }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) bv[j] = bs[(h * 8 + j) * SB::PITCH + n + c];
        }
#pragma unroll
        for (int j = 0; j < 8; j++) a = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[j], a, 0, 0, 0);
    }
};
template <> struct Acc<double> {
    static constexpr int N = 16;
    f64x4 a[2][2];
    __device__ inline void clear() {
#pragma unroll
        for (int x = 0; x < 4; x++)
#pragma unroll
            for (int v = 0; v < 4; v++) a[x >> 1][x & 1][v] = 0.0;
    }
    // v_mfma_f64_16x16x4f64: lane l supplies A(row l%16, k l/16), B(k l/16, col
    // l%16); element v of lane l is C(4*v + l/16, l%16)
    __device__ static inline int row(int lane, int v) { return (v >> 3) * 16 + 4 * (v & 3) + (lane >> 4); }
    __device__ static inline int col(int lane, int v) { return ((v >> 2) & 1) * 16 + (lane & 15); }
    __device__ inline double at(int v) const { return a[v >> 3][(v >> 2) & 1][v & 3]; }
    template <typename SA, typename SB, bool AK, bool BK>
    __device__ inline void products(const double* as, const double* bs, int m, int n, int lane) {
        const int h = lane >> 4, c = lane & 15;
        double av[2][4], bv[2][4];
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int row = m + i * 16 + c, col = n + i * 16 + c;
            if (AK) {
                const f64x2 x0 = *reinterpret_cast<const f64x2*>(as + SA::kc_off(row, 2 * h));
                const f64x2 x1 = *reinterpret_cast<const f64x2*>(as + SA::kc_off(row, 2 * h + 1));
                av[i][0] = x0[0]; av[i][1] = x0[1]; av[i][2] = x1[0]; av[i][3] = x1[1];
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++) av[i][j] = as[(h * 4 + j) * SA::PITCH + row];
            }
            if (BK) {
                const f64x2 x0 = *reinterpret_cast<const f64x2*>(bs + SB::kc_off(col, 2 * h));
                const f64x2 x1 = *reinterpret_cast<const f64x2*>(bs + SB::kc_off(col, 2 * h + 1));
                bv[i][0] = x0[0]; bv[i][1] = x0[1]; bv[i][2] = x1[0]; bv[i][3] = x1[1];
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++) bv[i][j] = bs[(h * 4 + j) * SB::PITCH + col];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int k = 0; k < 2; k++)
                    a[i][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i][j], bv[k][j], a[i][k], 0, 0, 0);
    }
};

// Tile `lin` of the launch.  SUM: K parts one after the other, added as the pass
// over their partial results would.
template <typename T, bool AK, bool BK, Addr ADDR, bool SUM>
__device__ __attribute__((always_inline)) inline void gemm_tile64_tile(const GemmDesc& g, int lin, int per_part,
                                                                       int tiles_m, int tiles_n) {
    typedef Slice<T, AK, ADDR> SA;
    typedef Slice<T, BK, ADDR> SB;
    __shared__ __attribute__((aligned(16))) T As[2][SA::ELEMS];
    __shared__ __attribute__((aligned(16))) T Bs[2][SB::ELEMS];
    int part = 0;
    if (!SUM && g.parts > 1) {
        part = lin / per_part;
        lin -= part * per_part;
    }
    int gb, m0, n0;
    if (g.upper) {
        // tiles (i, j), i <= j, column by column: r -> j(j+1)/2 + i
        const int per_batch = tiles_m * (tiles_m + 1) / 2;
        gb = lin / per_batch;
        const int r = lin % per_batch;
        int j = (int)((sqrtf(8.0f * (float)r + 1.0f) - 1.0f) * 0.5f);
        while (j * (j + 1) / 2 > r) j--;
        while ((j + 1) * (j + 2) / 2 <= r) j++;
        m0 = (r - j * (j + 1) / 2) * kT;
        n0 = j * kT;
    } else {
        // M tiles fastest: neighbouring workgroups share the B panel
        const int per_batch = tiles_m * tiles_n;
        gb = lin / per_batch;
        lin -= gb * per_batch;
        m0 = (lin % tiles_m) * kT;
        n0 = (lin / tiles_m) * kT;
    }
    if (g.only && !g.only[gb]) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int inner = g.inner > 1 ? g.inner : 1, go = gb / inner, gi = gb - go * inner;
    const T* Ab = static_cast<const T*>(g.A) + (int64_t)go * g.a_bs + (int64_t)gi * g.a_is;
    const T* Bb = static_cast<const T*>(g.B) + (int64_t)go * g.b_bs + (int64_t)gi * g.b_is;
    // slices: of one K batch after the other, or of this part's K range
    const int nk = (g.K + kS - 1) / kS;
    int s0 = g.parts > 1 ? part * (g.kp / kS) : 0;
    int total = g.parts > 1 ? min(g.kp / kS, nk - s0) : nk * g.kbatch;

    Acc<T> acc;
    typename SA::Source sa;
    typename SB::Source sb;
    sa.init(Ab, g.lda, m0, g.M, g.K, tid);
    sb.init(Bb, g.ldb, n0, g.N, g.K, tid);
    SA a0, a1;
    SB b0, b1;
    auto fetch = [&](int t, SA& a, SB& b) __attribute__((always_inline)) {
        int kb = 0, kt = s0 + t;
        if (ADDR != kNear && g.kbatch > 1) {
            kb = kt / nk;
            kt -= kb * nk;
        }
        a.load(sa, kt, kb, g.a_ks, tid);
        b.load(sb, kt, kb, g.b_ks, tid);
    };
    // slice t lies in LDS buffer `buf`, slice t + 1 in the registers na, nb;
    // the free registers ca, cb take slice t + 2
    auto step = [&](int t, int buf, SA& ca, SB& cb, SA& na, SB& nb) __attribute__((always_inline)) {
        if (t + 2 < total) fetch(t + 2, ca, cb);
        acc.template products<SA, SB, AK, BK>(As[buf], Bs[buf], wm, wn, lane);
        if (t + 1 < total) {
            na.store(As[buf ^ 1], tid);
            nb.store(Bs[buf ^ 1], tid);
        }
        __syncthreads();
    };
    auto walk = [&]() __attribute__((always_inline)) {
        acc.clear();
        if (total > 0) {
            fetch(0, a0, b0);
            if (total > 1) fetch(1, a1, b1);
            a0.store(As[0], tid);
            b0.store(Bs[0], tid);
            __syncthreads();
        }
        for (int t = 0; t < total; t += 2) {
            step(t, 0, a0, b0, a1, b1);
            if (t + 1 < total) step(t + 1, 1, a1, b1, a0, b0);
        }
    };
    T sum[SUM ? Acc<T>::N : 1];
    if (SUM) {
#pragma unroll
        for (int v = 0; v < Acc<T>::N; v++) sum[SUM ? v : 0] = T(0);
        for (int q = 0; q < max(g.parts, 1); q++) {
            if (g.parts > 1) {
                s0 = q * (g.kp / kS);
                total = min(g.kp / kS, nk - s0);
            }
            walk();
#pragma unroll
            for (int v = 0; v < Acc<T>::N; v++) sum[SUM ? v : 0] += acc.at(v);
        }
    } else {
        walk();
    }
    auto value = [&](int v) __attribute__((always_inline)) { return SUM ? sum[SUM ? v : 0] : acc.at(v); };

    T* Cb = static_cast<T*>(g.C) + (int64_t)gb * g.c_bs + (int64_t)part * g.c_ps;
    // symmetric output: off-diagonal tiles are also stored transposed, a
    // diagonal tile keeps row <= col and mirrors it (exactly symmetric)
    const bool mirror = g.upper && m0 != n0, diag = g.upper && m0 == n0;
    T old[Acc<T>::N];
    if (g.accumulate) {
        // all previous values in flight together
#pragma unroll
        for (int v = 0; v < Acc<T>::N; v++) {
            const int row = m0 + wm + Acc<T>::row(lane, v), col = n0 + wn + Acc<T>::col(lane, v);
            old[v] = row < g.M && col < g.N ? Cb[(int64_t)row * g.ldc + col] : T(0);
        }
    }
#pragma unroll
    for (int v = 0; v < Acc<T>::N; v++) {
        const int row = m0 + wm + Acc<T>::row(lane, v), col = n0 + wn + Acc<T>::col(lane, v);
        if (row < g.M && col < g.N && (!diag || row <= col)) {
            const T x = g.accumulate ? old[v] + value(v) : value(v);
            Cb[(int64_t)row * g.ldc + col] = x;
            if (mirror || (diag && row < col)) Cb[(int64_t)col * g.ldc + row] = x;
        }
    }
}

template <typename T, bool AK, bool BK, Addr ADDR>
__global__ __launch_bounds__(256, 4) void gemm_tile64_kernel(GemmDesc g, int tiles_m, int tiles_n) {
    gemm_tile64_tile<T, AK, BK, ADDR, false>(g, xcd_linear_id(), g.parts > 1 ? gridDim.x / g.parts : 0, tiles_m, tiles_n);
}

// The products of flagged batch entries (g.only), normally none: a few
// workgroups look at one flag and end, or walk all tiles.  K parts are summed by
// the workgroup, so that an entry has the bits of the split product.  (65 operators of 403
// states: one workgroup per tile 10.1 us for stage 1 with its 11375, now 4.6.)
template <typename T, bool AK, bool BK, Addr ADDR>
__global__ __launch_bounds__(256, 4) void gemm_tile64_only_kernel(GemmDesc g, int tiles_m, int tiles_n, int tiles) {
    if (!*g.any) return;
    for (int lin = blockIdx.x; lin < tiles; lin += gridDim.x)
        gemm_tile64_tile<T, AK, BK, ADDR, true>(g, lin, 0, tiles_m, tiles_n);
}

template <typename T>
hipError_t launch(const GemmDesc& g, hipStream_t stream) {
    const int tm = (g.M + kT - 1) / kT, tn = (g.N + kT - 1) / kT;
    const int64_t tiles =
        (g.upper ? (int64_t)tm * (tm + 1) / 2 : (int64_t)tm * tn) * g.batch * (g.parts > 1 && !g.only ? g.parts : 1);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    const int64_t lim = ((int64_t)1 << 32) / (int64_t)sizeof(T);
    auto addr = [&](bool kc, int64_t ld, int64_t rows) {
        if ((kc ? kT : kS) * ld + kT >= lim) return kFar;
        return g.kbatch == 1 && (kc ? (rows + kT) * ld : (g.K + kS) * ld + kT) < lim ? kNear : kRebase;
    };
    const Addr a = std::max(addr(g.a_kcontig, g.lda, g.M), addr(g.b_kcontig, g.ldb, g.N));
    if (g.only) {
        // rotations only: A is O (K-contiguous) or U, B is M/N-contiguous
        if (!g.any || g.b_kcontig || sizeof(T) != 4) return hipErrorInvalidValue;
        auto only = [&](auto ak) {
            constexpr bool AK = decltype(ak)::value;
            return a == kNear     ? gemm_tile64_only_kernel<float, AK, false, kNear>
                   : a == kRebase ? gemm_tile64_only_kernel<float, AK, false, kRebase>
                                  : gemm_tile64_only_kernel<float, AK, false, kFar>;
        };
        hipLaunchKernelGGL((g.a_kcontig ? only(std::true_type{}) : only(std::false_type{})),
                           dim3((unsigned)std::min<int64_t>(tiles, 1024)), dim3(256), 0, stream, g, tm, tn, (int)tiles);
        return hipGetLastError();
    }
    auto pick = [&](auto ak, auto bk) {
        constexpr bool AK = decltype(ak)::value, BK = decltype(bk)::value;
        return a == kNear     ? gemm_tile64_kernel<T, AK, BK, kNear>
               : a == kRebase ? gemm_tile64_kernel<T, AK, BK, kRebase>
                              : gemm_tile64_kernel<T, AK, BK, kFar>;
    };
    auto kernel = g.a_kcontig ? (g.b_kcontig ? pick(std::true_type{}, std::true_type{})
                                             : pick(std::true_type{}, std::false_type{}))
                              : (g.b_kcontig ? pick(std::false_type{}, std::true_type{})
                                             : pick(std::false_type{}, std::false_type{}));
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(256), 0, stream, g, tm, tn);
    return hipGetLastError();
}

}  // namespace

hipError_t gemm_tile64(const GemmDesc& g, bool is_double, hipStream_t stream) {
    return is_double ? launch<double>(g, stream) : launch<float>(g, stream);
}

}  // namespace rot
