// Batched FP32 products of the operator rotation (stage 1: T_b = O_b U_r;
// stage 2: out_b = U^T T_b) and its adjoint in 128 x 128 tiles, and the
// dispatch between them and the 64 x 64 tiles of gemm_tile64.hip.
//
// A 256-thread workgroup (four 64-wide waves in a 2 x 2 grid) owns a
// 128 x 128 tile of C and walks K in slices of 16 elements, double-buffered in
// LDS.  Each operand slice is stored in LDS in the same orientation it has in
// global memory; the assignment of k to matrix-instruction slots is permuted
// instead: in every slice, lane group h of a wave handles k = h*8 + j for step
// j, for both operands (as in gemm_tile64.hip, so both give the same bits).  A
// K-contiguous operand is then read with 128-bit LDS loads (all steps of the
// slice at once) and an M/N-contiguous one with 32-bit loads that are
// contiguous across the 32 lanes of a group.
//
// Workgroup ids are remapped so that each of the 8 XCDs (hardware assigns
// consecutive ids round-robin over them) processes a contiguous range of
// tiles, and tiles sharing an operand panel stay on one XCD's L2.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "buffer_rsrc.h"
#include "lds_slice.h"
#include "rot_internal.h"

namespace rot {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int kTile = kGemmTile;   // BM = BN
constexpr int kSlice = 16;   // K elements per LDS slice

struct TileCoord {
    int g, m0, n0;
};

__device__ inline TileCoord tile_coord(int lin, int tiles_m, int tiles_n, bool upper) {
    TileCoord t;
    if (upper) {
        // tiles (i, j) with i <= j of a tiles_m x tiles_m grid, column by
        // column (neighbours share the B panel): r -> j(j+1)/2 + i
        const int per_batch = tiles_m * (tiles_m + 1) / 2;
        t.g = lin / per_batch;
        const int r = lin % per_batch;
        int j = (int)((sqrtf(8.0f * (float)r + 1.0f) - 1.0f) * 0.5f);
        while (j * (j + 1) / 2 > r) j--;
        while ((j + 1) * (j + 2) / 2 <= r) j++;
        t.m0 = (r - j * (j + 1) / 2) * kTile;
        t.n0 = j * kTile;
        return t;
    }
    const int per_batch = tiles_m * tiles_n;
    t.g = lin / per_batch;
    const int r = lin % per_batch;
    t.m0 = (r % tiles_m) * kTile;  // M tiles fastest: neighbours share the B panel
    t.n0 = (r / tiles_m) * kTile;
    return t;
}

// FP32 product of whole tiles with both K slices filled by buffer loads with
// LDS destination (DmaSlice128): no staging registers, no per-slice address
// arithmetic, one wait and barrier per slice.  Same fragment reads,
// products and stores as gemm_tile64_kernel, so the same bits.  MODE 0: one K
// batch, plain stores; 1: symmetric output; 2: K batches (the slices of
// batch kb after those of kb - 1) and, with g.accumulate, C += result.
// Requires K (and a part's) a multiple of 16, 16-byte aligned rows, and each
// operand's batch entry (all its K batches) under 4 GiB (direct_lds_ok).
// EDGE (M or N not a multiple of 128): slices of a last, partial tile read
// whatever lies past the operand's rows or columns (zero past the batch
// entry, whose extent bounds the descriptors); those values only reach rows
// and columns of C that are not stored.
template <bool AK, bool BK, int MODE, bool EDGE>
__device__ __attribute__((always_inline)) inline void gemm_f32_dl_tile(const GemmDesc& g, int lin, int tiles_m,
                                                                       int tiles_n) {
    constexpr bool UPPER = MODE == 1;
    typedef DmaSlice128<AK> DA;
    typedef DmaSlice128<BK> DB;
    static_assert(kTile == DA::R && kSlice == DA::SK, "slice shape");
    __shared__ __attribute__((aligned(1024))) float As[2][DA::ELEMS];
    __shared__ __attribute__((aligned(1024))) float Bs[2][DB::ELEMS];

    int part = 0;
    if (MODE == 0 && g.parts > 1) {
        const int per = gridDim.x / g.parts;
        part = lin / per;
        lin -= part * per;
    }
    const TileCoord tc = tile_coord(lin, tiles_m, tiles_n, UPPER);
    if (g.only && !g.only[tc.g]) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int h = lane >> 5, c = lane & 31;

    const float* Ab = static_cast<const float*>(g.A) + (int64_t)tc.g * g.a_bs;
    const float* Bb = static_cast<const float*>(g.B) + (int64_t)tc.g * g.b_bs;
    const int kb1 = MODE == 2 ? g.kbatch - 1 : 0;
    const int64_t ea = (AK ? (int64_t)(g.M - 1) * g.lda + g.K : (int64_t)(g.K - 1) * g.lda + g.M) + kb1 * g.a_ks;
    const int64_t eb = (BK ? (int64_t)(g.N - 1) * g.ldb + g.K : (int64_t)(g.K - 1) * g.ldb + g.N) + kb1 * g.b_ks;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Ab), (short)0, EDGE ? (int)(uint32_t)(ea * 4) : (int)0xffffffff, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Bb), (short)0, EDGE ? (int)(uint32_t)(eb * 4) : (int)0xffffffff, kBufferFlags);
    DA da;
    DB db;
    da.init(g.lda, tc.m0, wave, lane);
    db.init(g.ldb, tc.n0, wave, lane);

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

    const int nk = g.K / kSlice;
    // a part's K range: slices s0 .. s0 + total - 1
    const int s0 = MODE == 0 && g.parts > 1 ? part * (g.kp / kSlice) : 0;
    const int total = MODE == 2 ? nk * g.kbatch : MODE == 0 && g.parts > 1 ? min(g.kp / kSlice, nk - s0) : nk;
    // slice t: K batch t / nk, slice t % nk of it
    auto issue = [&](int t, int buf) __attribute__((always_inline)) {
        if (MODE == 2) {
            const int kb = t / nk, kt = t - kb * nk;
            da.issue_at(ra, As[buf], (uint32_t)kb * (uint32_t)(g.a_ks * 4) + (uint32_t)kt * da.step, wave);
            db.issue_at(rb, Bs[buf], (uint32_t)kb * (uint32_t)(g.b_ks * 4) + (uint32_t)kt * db.step, wave);
        } else {
            da.issue(ra, As[buf], s0 + t, wave);
            db.issue(rb, Bs[buf], s0 + t, wave);
        }
    };
    issue(0, 0);
    dma_slice_sync();
    for (int t = 0; t < total; t++) {
        const int cur = t & 1;
        if (t + 1 < total) issue(t + 1, cur ^ 1);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        const float* a_s = As[cur];
        const float* b_s = Bs[cur];
        // 8 steps of k = 2: lane group h takes k = h*8 + j at step j
        float av[2][8], bv[2][8];
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int row = wm * 64 + i * 32 + c;
            if (AK) {
                const f32x4 x0 = *reinterpret_cast<const f32x4*>(a_s + DA::kc_off(row, 2 * h));
                const f32x4 x1 = *reinterpret_cast<const f32x4*>(a_s + DA::kc_off(row, 2 * h + 1));
#pragma unroll
                for (int e = 0; e < 4; e++) { av[i][e] = x0[e]; av[i][4 + e] = x1[e]; }
            } else {
#pragma unroll
                for (int j = 0; j < 8; j++) av[i][j] = a_s[DA::mn_off(h * 8 + j, row)];
            }
        }
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int col = wn * 64 + i * 32 + c;
            if (BK) {
                const f32x4 x0 = *reinterpret_cast<const f32x4*>(b_s + DB::kc_off(col, 2 * h));
                const f32x4 x1 = *reinterpret_cast<const f32x4*>(b_s + DB::kc_off(col, 2 * h + 1));
#pragma unroll
                for (int e = 0; e < 4; e++) { bv[i][e] = x0[e]; bv[i][4 + e] = x1[e]; }
            } else {
#pragma unroll
                for (int j = 0; j < 8; j++) bv[i][j] = b_s[DB::mn_off(h * 8 + j, col)];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int k = 0; k < 2; k++)
                    acc[i][k] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][j], bv[k][j], acc[i][k], 0, 0, 0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        dma_slice_sync();
    }

    float* Cb = static_cast<float*>(g.C) + (int64_t)tc.g * g.c_bs + (int64_t)part * g.c_ps;
    // symmetric output: a diagonal tile keeps row <= col and mirrors it; an
    // off-diagonal tile is also stored transposed (a lane's rows 8q + 4h ..
    // +3 become four consecutive entries of row `col`)
    const bool diag = UPPER && tc.m0 == tc.n0;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int col = tc.n0 + wn * 64 + k * 32 + c;
            if (EDGE && col >= g.N) continue;
            if (MODE == 2 && g.accumulate) {
                // the previous values of each group of four rows are loaded
                // before the group's stores (unconditionally, from element 0
                // outside C), four loads in flight together
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = tc.m0 + wm * 64 + i * 32 + 8 * q + 4 * h;
                    float old[4];
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        old[e] = Cb[!EDGE || row0 + e < g.M ? (int64_t)(row0 + e) * g.ldc + col : 0];
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        if (!EDGE || row0 + e < g.M)
                            Cb[(int64_t)(row0 + e) * g.ldc + col] = old[e] + acc[i][k][4 * q + e];
                }
                continue;
            }
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int row = tc.m0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                if ((!EDGE || row < g.M) && (!diag || row <= col)) {
                    Cb[(int64_t)row * g.ldc + col] = acc[i][k][v];
                    if (diag && row < col) Cb[(int64_t)col * g.ldc + row] = acc[i][k][v];
                }
            }
        }
    if (UPPER && !diag) {
        const bool vec4 = (g.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(Cb) & 15) == 0;
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int k = 0; k < 2; k++) {
                const int col = tc.n0 + wn * 64 + k * 32 + c;
                if (EDGE && col >= g.N) continue;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = tc.m0 + wm * 64 + i * 32 + 8 * q + 4 * h;
                    float* p = Cb + (int64_t)col * g.ldc + row0;
                    if (vec4 && (!EDGE || row0 + 4 <= g.M)) {
                        *reinterpret_cast<f32x4*>(p) = f32x4{acc[i][k][4 * q], acc[i][k][4 * q + 1],
                                                             acc[i][k][4 * q + 2], acc[i][k][4 * q + 3]};
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (!EDGE || row0 + e < g.M) p[e] = acc[i][k][4 * q + e];
                    }
                }
            }
    }
}

template <bool AK, bool BK, int MODE, bool EDGE>
__global__ __launch_bounds__(kThreads) void gemm_f32_dl_kernel(GemmDesc g, int tiles_m, int tiles_n) {
    gemm_f32_dl_tile<AK, BK, MODE, EDGE>(g, xcd_linear_id(), tiles_m, tiles_n);
}

// The products of flagged batch entries (g.only), normally none: workgroups that
// fit the chip at once look at one flag and end, or walk all tiles (64 operators
// of 1024 states, all flagged: both stages 8.9 ms in 64 x 64 tiles, 8.0 here).
template <bool AK, int MODE, bool EDGE>
__global__ __launch_bounds__(kThreads) void gemm_f32_dl_only_kernel(GemmDesc g, int tiles_m, int tiles_n, int tiles) {
    if (!*g.any) return;
    for (int lin = xcd_linear_id(); lin < tiles; lin += gridDim.x)
        gemm_f32_dl_tile<AK, false, MODE, EDGE>(g, lin, tiles_m, tiles_n);
}

// Conditions of the direct-to-LDS kernel: 16-byte aligned rows, whole K slices
// (also of a part), no two-level batch, and every byte offset of an operand's
// batch entry (over all K batches, and the rows or columns a last partial
// tile reads) below 2^32.
bool direct_lds_ok(const GemmDesc& g) {
    auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    if (!(al(g.A) && al(g.B) && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.a_bs % 4 == 0 && g.b_bs % 4 == 0 &&
          g.a_ks % 4 == 0 && g.b_ks % 4 == 0 && g.inner <= 1))
        return false;
    if (g.kbatch < 1 || (g.parts > 1 && (g.kp % kSlice != 0 || g.accumulate))) return false;
    if (g.K % kSlice != 0 || g.K <= 0) return false;
    if (g.kbatch > 1 && (g.a_ks < 0 || g.b_ks < 0)) return false;
    const int64_t ea = (g.a_kcontig ? (int64_t)(g.M - 1) * g.lda + g.K : (int64_t)(g.K - 1) * g.lda + g.M) +
                       (int64_t)(g.kbatch - 1) * g.a_ks;
    const int64_t eb = (g.b_kcontig ? (int64_t)(g.N - 1) * g.ldb + g.K : (int64_t)(g.K - 1) * g.ldb + g.N) +
                       (int64_t)(g.kbatch - 1) * g.b_ks;
    // a partial tile's slices reach up to 127 rows (K-contiguous) or columns
    // past the operand
    const int64_t ra = g.a_kcontig ? (int64_t)kTile * g.lda : kTile;
    const int64_t rb = g.b_kcontig ? (int64_t)kTile * g.ldb : kTile;
    return (ea + ra) * 4 < ((int64_t)1 << 32) && (eb + rb) * 4 < ((int64_t)1 << 32);
}

// Tiles of 128 x 128 from which the direct-to-LDS kernel is the faster one:
// four of its workgroups share a CU, so fewer than 4 x 256 leave room that
// 64 x 64 tiles fill (both stages, 128 against 64 wide: 48 operators of 512
// states, 3072 and 768 tiles, 787 / 833 us; 40 of 256, 640: 131 / 132; 10 of
// 500, 600: 203 / 194; 2 of 512, 128: 78 / 55).
constexpr int64_t kWideTiles = 1024;

hipError_t gemm_any(const GemmDesc& g, bool is_double, hipStream_t stream) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
    if (g.upper && (g.M != g.N || g.accumulate)) return hipErrorInvalidValue;
    const int parts = g.parts > 1 && !g.only ? g.parts : 1;
    if (g.parts > 1 && ((g.upper && !is_double) || g.accumulate || g.kbatch != 1 || g.kp <= 0 || g.kp % kSlice != 0 ||
                      (int64_t)g.kp * (g.parts - 1) >= g.K))
        return hipErrorInvalidValue;
    const int tm = (g.M + kTile - 1) / kTile, tn = (g.N + kTile - 1) / kTile;
    const int64_t tiles = (g.upper ? (int64_t)tm * (tm + 1) / 2 : (int64_t)tm * tn) * g.batch * parts;
    if (is_double || tiles < kWideTiles || (g.only && g.parts > 1) || !direct_lds_ok(g))
        return gemm_tile64(g, is_double, stream);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    const bool edge = g.M % kTile != 0 || g.N % kTile != 0;
    if (g.only) {
        // rotations only (as in gemm_tile64.hip)
        if (!g.any || g.b_kcontig || g.accumulate || g.kbatch != 1) return hipErrorInvalidValue;
        auto only = [&](auto ak, auto mode) {
            constexpr bool AK = decltype(ak)::value;
            constexpr int MD = decltype(mode)::value;
            return edge ? gemm_f32_dl_only_kernel<AK, MD, true> : gemm_f32_dl_only_kernel<AK, MD, false>;
        };
        auto only_mode = [&](auto ak) {
            return g.upper ? only(ak, std::integral_constant<int, 1>{}) : only(ak, std::integral_constant<int, 0>{});
        };
        hipLaunchKernelGGL((g.a_kcontig ? only_mode(std::true_type{}) : only_mode(std::false_type{})),
                           dim3((unsigned)kWideTiles), dim3(kThreads), 0, stream, g, tm, tn, (int)tiles);
        return hipGetLastError();
    }
    auto pick = [&](auto mode, auto e) {
        constexpr int MD = decltype(mode)::value;
        constexpr bool E = decltype(e)::value;
        if (g.a_kcontig)
            return g.b_kcontig ? gemm_f32_dl_kernel<true, true, MD, E> : gemm_f32_dl_kernel<true, false, MD, E>;
        return g.b_kcontig ? gemm_f32_dl_kernel<false, true, MD, E> : gemm_f32_dl_kernel<false, false, MD, E>;
    };
    auto pick_mode = [&](auto e) {
        if (g.upper) return pick(std::integral_constant<int, 1>{}, e);
        if (g.accumulate || g.kbatch > 1) return pick(std::integral_constant<int, 2>{}, e);
        return pick(std::integral_constant<int, 0>{}, e);
    };
    hipLaunchKernelGGL((edge ? pick_mode(std::true_type{}) : pick_mode(std::false_type{})), dim3((unsigned)tiles),
                       dim3(kThreads), 0, stream, g, tm, tn);
    return hipGetLastError();
}

}  // namespace

hipError_t gemm_f32(const GemmDesc& g, hipStream_t stream) { return gemm_any(g, false, stream); }
hipError_t gemm_f64(const GemmDesc& g, hipStream_t stream) { return gemm_any(g, true, stream); }

}  // namespace rot
