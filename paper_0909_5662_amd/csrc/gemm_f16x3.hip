// FP32 rotation on FP16 pairs.  The FP32 matrix instructions run at 1/16 of
// the FP16 ones' rate, so a product of FP32 operands taken as three FP16
// products (hi*hi + hi*lo + lo*hi, FP32 accumulation) has over five times the
// FP32 peak to work with.  A scaled pair holds a value in its range to 2^-23
// of itself, one unit of FP32's last place (split2_f16); the dropped lo*lo term
// is below 2^-22 of a product and averages 2^-25; the sum is rounded three
// times per 16 k where the FP32 instructions round eight times, which more
// than makes up for both.  Measured against 64 bits (relative Frobenius error,
// Gaussian operators; FP32 kernels -> pairs): 1024 states 1.28e-6 -> 8.0e-7,
// 403: 8.0e-7 -> 5.1e-7, 256: 4.4e-7 -> 3.2e-7, 128: 2.6e-7 -> 2.1e-7, 64:
// 2.1e-7 -> 1.8e-7.
// Time of the two stages and all passes around them, 64 operators of 1024
// states: 8.02 -> 2.79 ms; 65 of 403 (kept 391): 1.31 -> 0.27 ms.
//
// Scaling.  U's columns and each operator are brought to a largest entry in
// [2^14, 2^15) by exact powers of two (eu[beta], eo[b]).  |T| of the scaled
// operands is below 2^15 times the largest row sum of |O_b|, so stage 1's
// epilogue multiplies by 2^-t with that sum below 2^t before it splits T; stage
// 2's undoes every scale.  FP16's range leaves entries from 2^-2 on, 2^-16 of an
// operand's largest entry or 2^-17 of T's bound (Gaussian operators of 1024
// states: T at 2^-7; by m max|O| instead of the row sum it was at 2^-10, and large
// operators had blocks of T below it by chance), at full precision; the pair of
// a smaller one is off by up to 2^-25 whatever its size.
//
// Range.  Where such entries are many, in a part of an operand that some result
// is made of alone, that result would be less exact than FP32's: columns of an
// operator that are small beside others which U leaves out, states that U
// hardly reaches, blocks of different size.  So the entries themselves are
// counted where they are made: an operator is skipped by these kernels, and
// computed by the FP32 kernels that follow (which leave the others alone), when
//   - it holds an infinity or NaN, or its rows' largest entries differ by more
//     than 2^12, or non-zero entries below 2^-2 make up a quarter of 16 entries
//     of a row or of 64 of a column (split pass);
//   - the same is true of U: then every operator is (split pass: 3 of 8 entries
//     of a column, or a quarter of a row's 32 in its half of a wave), as where
//     U's columns are short or mostly scattered zeros (kPairColumn);
//   - in a 32 x 32 block of T they are half of a lane's 16 or a whole row of 32,
//     or an eighth of the block (stage 1, t_out_of_range).
// Scattered small entries of a Gaussian operand (6e-5 of O and U, 1e-3 of T at
// 1024 states) stay far below these counts.  Zeros count for nothing: they are
// exact.  Blocks of the results of accepted operators against the FP32 kernels'
// error: columns of operators that U leaves out, states that U hardly reaches,
// sectors, in order and mixed, and tails of U, from 2^0 to 2^-16 of the rest, at
// most 0.93 times it (160 states); sectors, sites, rows, columns and sparsity
// drawn at random (64 to 330 states, d 1 to 8, 25 500 blocks), at most 1.3e-7
// more (sparse operators between short sectors).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>
#include <vector>

#include "buffer_rsrc.h"
#include "lds_slice.h"
#include "rot_internal.h"
#include "split_slab.h"

namespace rot {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
// four floats at any 4-byte boundary: global_load_dwordx4 needs no more
typedef f32x4 f32x4u __attribute__((aligned(4)));

// FP16 carries 11 significant bits to BF16's 8, in a range of 2^30 instead of
// FP32's: its operands are scaled by powers of two first (|x| < 2^15), so
// hi + lo holds x to 2^-23 of itself (FP32's last bit) or 2^-40 of the
// operand's largest entry, whichever is larger.
// One conversion per pair and one back per value: the compiler would otherwise
// convert each value a second time for its remainder, in the epilogue that
// nothing overlaps (200 operators of 512 states, stage 1: 0.73 -> 0.62 ms).
__device__ inline u32x2 split2_f16(float a, float b) {
    uint32_t h = __builtin_bit_cast(uint32_t, f16x2{(_Float16)a, (_Float16)b});
    asm("" : "+v"(h));
    const f16x2 x = __builtin_bit_cast(f16x2, h);
    const f16x2 l = {(_Float16)fmaf((float)x[0], -1.0f, a), (_Float16)fmaf((float)x[1], -1.0f, b)};
    return u32x2{h, __builtin_bit_cast(uint32_t, l)};
}

// What the split pass finds in U (cleared by the scale pass).
struct UState {
    // low half: entries that are not zero; high half (signed): groups of eight of a
    // column with five and more of them less those with one to four (one addition
    // for both: 1024 workgroups add to it)
    unsigned long long filled_runs;
    int bad;  // leaves the pairs' range
};

// Rotation products with one A for every operator (U1 or U2) and one B per
// operator: the operators' B rows, each padded to whole blocks of 32, are laid
// end to end, and a tile takes 8 consecutive blocks (256 columns) whatever
// operator they belong to, so only the last tile of the launch and each
// operator's last block hold padding (403 columns: 3 % where 256-wide tiles
// per operator computed 21 %).  Tiles have 64 bi rows (64 to 256);
// the last M tile shrinks to the multiple of 64 that covers the rest of M.
// K may be cut into parts of `part_slabs` slabs, whose products go to their
// own partial results (c_ps apart) to be added in a fixed order.
struct FlatDesc {
    int M, N, K, batch;         // C_b (M x N) = A (M x K) B_b^T
    const uint16_t *a_hi, *a_lo;  // slab layout, M rows
    const uint16_t *b_hi, *b_lo;  // slab layout, n32 rows per operator, b_bs elements apart
    int64_t b_bs;
    int n32;                    // N rounded up to 32
    int tiles_m, tiles_n, parts, part_slabs;
    // plain epilogue: C_b(row, col) 2^-(op_e[b] + row_e[row] + col_e[col]) at
    // c + part*c_ps + b*c_bs + row*ldc + col
    float* c;
    int64_t ldc, c_bs, c_ps;
    const int *op_e, *row_e, *col_e;  // row_e: readable up to the last tile's rows
    // split-transposed epilogue: C_b(beta*d + s, i) 2^-t_e[b] -> T_b(beta, i*d + s),
    // slab layout with t_rows rows per operator, t_bs elements apart
    uint16_t *t_hi, *t_lo;
    int d, t_rows;
    int64_t t_bs;
    const int* t_e;
    int* skip;                  // operators left to the FP32 kernels: kSkipSplit, kSkipStage1
    int* any;                   // raised with the first of them
    const UState* u;            // stage 1: what the split pass found in U
    uint32_t u_least;           // entries that U needs
    // symmetric output (M == N, plain epilogue): tiles below the diagonal of
    // all their operators are left out, entries on or above it are also stored
    // transposed
    int upper;
};

// Bits of skip[b]: what the split pass found, and stage 1 (whose tiles read
// the first while others set the second).
constexpr int kSkipSplit = 1, kSkipStage1 = 2;

// U's columns hold at least this many entries on average (three quarters of
// shorter ones, 64 at least), mostly five and more of eight neighbours, or the
// FP32 instructions' sums, which round once per entry or two of them (two k)
// where these kernels round three times per 16 k, are the more exact ones: 128
// states with 1 / 16 / 64 / 128 / 256 of 512 entries per column, scattered, 0 /
// 0.85e-7 / 1.6e-7 / 2.3e-7 / 3.2e-7 against 0.4e-7 / 1.7e-7 / 2.4e-7 / 2.8e-7 /
// 2.9e-7; 74 of 369 in a row, sparse operators, 0.8e-7 against 1.9e-7.  Zeros of
// an operator do not matter: with such a U diagonal ones, permutations and ones
// of 1 entry in 20 have 0.61 to 1.01 times the FP32 kernels' error from 64 states
// on.
constexpr int kPairColumn = 128, kPairShortColumn = 64;

// Entries of a pair operand below this are off by more than 2^-23 of themselves.
constexpr float kPairLeast = 0.25f;

__device__ inline bool pair_small(float x) {
    return (__float_as_uint(x) & 0x7fffffffu) - 1u < __float_as_uint(kPairLeast) - 1u;
}

// The range of a 32 x 32 block of T (a column per lane, in lanes `valid`; rows
// 8 q + 4 h + e).  The epilogue's pairs are watched without telling zeros from
// small entries, one bit per entry; where they could be too many the blocks are
// looked at entry by entry (a comparison, a count and two ballot words per entry
// of all blocks made stage 1 of 65 operators of 403 states 10 % slower, this
// does by 3 %).
struct TWatch {
    uint32_t below = 0;  // bit 8 e + 7 - q
    __device__ inline void add(int q, uint32_t h01, uint32_t h23) {
        const f16x2 c = {(_Float16)(-kPairLeast * kPairLeast), (_Float16)(-kPairLeast * kPairLeast)};
        auto sign = [&](uint32_t h) {  // set where |h| < kPairLeast
            const f16x2 x = __builtin_bit_cast(f16x2, h);
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(x, x, c));
        };
        const uint32_t four = __builtin_amdgcn_perm(sign(h23), sign(h01), 0x07050301u) >> q, at = 0x80808080u >> q;
        below = (four & at) | (below & ~at);
    }
    // The bits of a block's first `rows` rows.
    __device__ static inline uint32_t inside(int rows, int lane) {
        const int left = rows - 4 * (lane >> 5);
        uint32_t in = 0;
#pragma unroll
        for (int v = 0; v < 16; v++) in |= 8 * (v >> 2) + (v & 3) < left ? 128u << 8 * (v & 3) >> (v >> 2) : 0u;
        return in;
    }
    __device__ static inline uint32_t filled(const f32x16& t) {
        uint32_t f = 0;
#pragma unroll
        for (int v = 0; v < 16; v++) f |= t[v] != 0.f ? 128u << 8 * (v & 3) >> (v >> 2) : 0u;
        return f;
    }
};

// x of the lane 8, 4, 2 or 1 further in the same 16 lanes (cyclically): sums and
// the like over these, which a swap of neighbouring sixteens completes to 32.
constexpr int kRor8 = 0x128, kRor4 = 0x124, kRor2 = 0x122, kRor1 = 0x121;
template <int CTRL>
__device__ inline uint32_t lane_dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, false);
}

// Whether one of BI blocks on the same columns is to be looked at: half a column
// (16 entries of a block) with four below, two in a quarter of the half columns,
// or a whole row.
template <int BI>
__device__ __attribute__((always_inline)) inline bool t_suspect(const TWatch (&w)[BI], uint64_t valid, int lane) {
    const bool in = (valid >> lane) & 1;
    int most = 0;
    uint32_t rows = 0;  // bits set in all lanes of a half wave: rows
#pragma unroll
    for (int i = 0; i < BI; i++) most = max(most, __builtin_popcount(w[i].below));
#pragma unroll
    for (int i = 0; i < BI; i += 2) {
        uint32_t r = w[i].below;  // the high half of each byte
        if (i + 1 < BI) r |= w[i + 1 < BI ? i + 1 : i].below >> 4;
        uint32_t x = in ? r : ~0u;
        x &= lane_dpp<kRor8>(x);
        x &= lane_dpp<kRor4>(x);
        x &= lane_dpp<kRor2>(x);
        x &= lane_dpp<kRor1>(x);
        const auto y = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        rows |= y[0] & y[1];
    }
    const uint64_t four = __builtin_amdgcn_ballot_w64(most >= 4) & valid;
    const uint64_t two = __builtin_amdgcn_ballot_w64(most >= 2) & valid;
    return (four | __builtin_amdgcn_ballot_w64(rows != 0)) != 0 ||
           4 * __builtin_popcountll(two) >= __builtin_popcountll(valid);
}

// Per bit over the 32 lanes of each half wave: `left` ored, and the count as
// ones, twos and "four or more".
struct RowBits {
    uint32_t left, one, two, four;
    __device__ inline void add(const RowBits& o) {
        const uint32_t carry = one & o.one;
        left |= o.left;
        four |= o.four | (two & o.two) | (carry & (two ^ o.two));
        two ^= o.two ^ carry;
        one ^= o.one;
    }
    template <int CTRL>
    __device__ inline void step() {
        add(RowBits{lane_dpp<CTRL>(left), lane_dpp<CTRL>(one), lane_dpp<CTRL>(two), lane_dpp<CTRL>(four)});
    }
    __device__ inline void reduce() {
        step<kRor8>();
        step<kRor4>();
        step<kRor2>();
        step<kRor1>();
        const auto l = __builtin_amdgcn_permlane16_swap(left, left, false, false);
        const auto o = __builtin_amdgcn_permlane16_swap(one, one, false, false);
        const auto t = __builtin_amdgcn_permlane16_swap(two, two, false, false);
        const auto f = __builtin_amdgcn_permlane16_swap(four, four, false, false);
        *this = RowBits{l[0], o[0], t[0], f[0]};
        add(RowBits{l[1], o[1], t[1], f[1]});
    }
};

// Whether too much of one of the blocks is below and not zero (filled: the
// entries in T that are not).  t_suspect passes no such block: what it passes
// has fewer than 94 entries below of 1024.
template <int BI>
__device__ __attribute__((always_inline)) inline bool t_out_of_range(const TWatch (&w)[BI], const uint32_t (&filled)[BI]) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < BI; i += 2) {
        // rows: two blocks' bits together
        const int j = i + 1 < BI ? i + 1 : i;
        const uint32_t f = filled[i] | (j > i ? filled[j] >> 4 : 0u), b = w[i].below | (j > i ? w[j].below >> 4 : 0u);
        RowBits r{f & ~b, f, 0, 0};
        r.reduce();
        bad |= (r.four & ~r.left) != 0;
    }
#pragma unroll
    for (int i = 0; i < BI; i++) {
        const int f = __builtin_popcount(filled[i]), n = __builtin_popcount(filled[i] & w[i].below);
        bad |= n >= 4 && 2 * n >= f;
        int sum = n << 16 | f;  // over the wave
        sum += (int)lane_dpp<kRor8>((uint32_t)sum);
        sum += (int)lane_dpp<kRor4>((uint32_t)sum);
        sum += (int)lane_dpp<kRor2>((uint32_t)sum);
        sum += (int)lane_dpp<kRor1>((uint32_t)sum);
        const int all = __builtin_amdgcn_readlane(sum, 0) + __builtin_amdgcn_readlane(sum, 16) +
                        __builtin_amdgcn_readlane(sum, 32) + __builtin_amdgcn_readlane(sum, 48);
        const int small = all >> 16, in = all & 0xffff;
        bad |= (small >= 8 && 8 * small >= in) || (small >= 2 && small == in);
    }
    return __builtin_amdgcn_ballot_w64(bad) != 0;
}

__device__ inline f32x16 mfma_f16(f16x8 a, f16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

constexpr int kFlatRing = 6;                         // LDS stages of A
constexpr int kFlatArr = 256 * kSlabK;               // elements of A_hi (or A_lo) in a stage
constexpr int kFlatLds = kFlatRing * 2 * kFlatArr;   // elements

// One tile of (64 BI) x 256 as 2 x 4 waves of (32 BI) x 64, by
// gemm_bf16x3_db_kernel's scheme: A through the LDS ring, B fragments straight
// into three register sets two slabs ahead.  A stage always holds 256 rows
// (those past the tile are copied and not read), so every wave issues the
// same number of loads and the waits stay immediate.
// DS: d of the transposed epilogue if it is 4 or 2, else 0.
template <int BI, bool EPI_T, int DS>
__device__ __attribute__((always_inline)) inline void flat_tile(const FlatDesc& g, uint16_t* lds, int m0, int nt,
                                                                int part) {
    constexpr int BJ = 2, S = kFlatRing, ARR = kFlatArr, STAGE = 2 * ARR;
    constexpr int LA = 2, LB = 2 * BJ;
    constexpr int WAIT_A0 = (S - 2) * LA + 2 * LB;
    constexpr int WAIT_A = (S - 3) * LA + (S - 2) * LB;
    constexpr int WAIT_B = 2 * (LA + LB), WAIT_B0 = LA + 2 * LB;
    static_assert(WAIT_A0 <= 63 && WAIT_A <= 63 && WAIT_B <= 63, "vmcnt range");
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int h = lane >> 5, c = lane & 31;
    const bool u_bad = EPI_T && (g.u->bad || (int)(g.u->filled_runs >> 32) <= 0 ||
                                 (uint32_t)g.u->filled_runs < g.u_least);
    if (u_bad || *g.any) {
        // nothing to do where all operators are skipped (64 of 1024 states, all
        // skipped: 10.3 ms with these products and the 64-wide FP32 tiles, 8.4
        // without and with the 128-wide ones; 7.96 on the FP32 kernels alone).
        // Stage 1 looks at the split pass's bits only, which no tile changes, so
        // that all waves decide alike; when U is not for the pairs it marks the
        // operators.
        const int bpo = g.n32 >> 5, first = nt * 8 / bpo, last = min(nt * 8 + 7, bpo * g.batch - 1) / bpo;
        if (u_bad) {
            for (int b = first + tid; b <= last; b += 512) atomicOr(&g.skip[b], kSkipStage1);
            if (tid == 0) atomicOr(g.any, 1);
            return;
        }
        bool all = true;
        for (int b = first; b <= last; b++) all &= (g.skip[b] & (EPI_T ? kSkipSplit : ~0)) != 0;
        if (all) return;
    }
    const int st0 = part * g.part_slabs;
    const int nk = min(g.part_slabs, (int)n_slabs(g.K) - st0);

    const __amdgpu_buffer_rsrc_t ra[2] = {operand_rsrc(g.a_hi, g.M, g.K), operand_rsrc(g.a_lo, g.M, g.K)};
    const int b_bytes = (int)(uint32_t)(g.batch * g.b_bs * 2);
    const __amdgpu_buffer_rsrc_t rb[2] = {
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.b_hi), (short)0, b_bytes, kBufferFlags),
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.b_lo), (short)0, b_bytes, kBufferFlags)};
    const uint32_t a_slab = (uint32_t)g.M * kSlabK * 2, b_slab = (uint32_t)g.n32 * kSlabK * 2;
    const uint32_t a_off = (uint32_t)((m0 + wave * 32) * kSlabK * 2 + lane * 16) + (uint32_t)st0 * a_slab;
    const int fslot = (h ^ ((c >> 3) & 1)) * 8;
    // this wave's column blocks: operator and block inside it (blocks past the
    // last operator repeat its last one and are not stored)
    const int bpo = g.n32 >> 5, nblk = bpo * g.batch;
    int op[BJ], cb[BJ];
    uint32_t b_off[BJ];
    bool live[BJ];
#pragma unroll
    for (int j = 0; j < BJ; j++) {
        const int x = nt * 8 + wn * BJ + j;
        live[j] = x < nblk;
        const int y = min(x, nblk - 1);
        op[j] = y / bpo;
        cb[j] = y - op[j] * bpo;
        b_off[j] = (uint32_t)(op[j] * g.b_bs * 2) + (uint32_t)(((cb[j] * 32 + c) * kSlabK + fslot) * 2) +
                   (uint32_t)st0 * b_slab;
    }

    auto issue_a = [&](int st) __attribute__((always_inline)) {
        uint16_t* base = lds + (st % S) * STAGE + wave * 512;
#pragma unroll
        for (int j = 0; j < 2; j++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                ra[j], (__attribute__((address_space(3))) void*)(base + j * ARR), 16, a_off + (uint32_t)st * a_slab,
                0, 0, 0);
    };
    struct BSet {
        f16x8 bh[BJ], bl[BJ];
    };
    auto issue_b = [&](BSet& o, int st) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < BJ; j++) {
            const uint32_t off = b_off[j] + (uint32_t)st * b_slab;
            o.bh[j] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rb[0], off, 0, 0));
            o.bl[j] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(rb[1], off, 0, 0));
        }
    };

    f32x16 acc[BI][BJ];
#pragma unroll
    for (int i = 0; i < BI; i++)
#pragma unroll
        for (int j = 0; j < BJ; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

    f16x8 ah[BI], al[BI];
    auto read_a = [&](int i, int st) __attribute__((always_inline)) {
        const uint16_t* sb = lds + (st % S) * STAGE;
        const int ra_ = (wm * 32 * BI + i * 32 + c) * kSlabK + fslot;
        ah[i] = *reinterpret_cast<const f16x8*>(sb + ra_);
        al[i] = *reinterpret_cast<const f16x8*>(sb + ARR + ra_);
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        compiler_fence();
        __builtin_amdgcn_s_barrier();
        compiler_fence();
    };

    // the wait counts assume exactly this issue order
    BSet bs[3];
#pragma unroll
    for (int st = 0; st <= S - 2; st++) {
        issue_a(st);
        compiler_fence();
    }
    issue_b(bs[0], 0);
    compiler_fence();
    issue_b(bs[1], 1);
    compiler_fence();
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(WAIT_A0));
    barrier();
#pragma unroll
    for (int i = 0; i < BI; i++) read_a(i, 0);

#define FLAT_STEP(T_, CUR, NB, WA, WB)                                                                    \
    do {                                                                                                  \
        const int t_ = (T_);                                                                              \
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(WA));                                                        \
        barrier();                                                                                        \
        issue_a(t_ + S - 1);                                                                              \
        compiler_fence();                                                                                 \
        issue_b(NB, t_ + 2);                                                                              \
        compiler_fence();                                                                                 \
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(WB));                                                        \
        compiler_fence();                                                                                 \
        _Pragma("unroll") for (int i = 0; i < BI; i++) {                                                  \
            _Pragma("unroll") for (int k = 0; k < BJ; k++) acc[i][k] =                                    \
                mfma_f16(al[i], (CUR).bh[k], acc[i][k]);                                                   \
            _Pragma("unroll") for (int k = 0; k < BJ; k++) acc[i][k] =                                    \
                mfma_f16(ah[i], (CUR).bl[k], acc[i][k]);                                                   \
            _Pragma("unroll") for (int k = 0; k < BJ; k++) acc[i][k] =                                    \
                mfma_f16(ah[i], (CUR).bh[k], acc[i][k]);                                                   \
            read_a(i, t_ + 1);                                                                            \
        }                                                                                                 \
        compiler_fence();                                                                                 \
    } while (0)
    constexpr int WA0 = (S - 3) * LA + 2 * LB;
    constexpr int WA1 = (S - 3) * LA + 3 * LB;
    constexpr int WA2 = (S - 3) * LA + 4 * LB;
    FLAT_STEP(0, bs[0], bs[2], WA0, WAIT_B0);
    FLAT_STEP(1, bs[1], bs[0], WA1, WAIT_B);
    FLAT_STEP(2, bs[2], bs[1], WA2, WAIT_B);
    int t = 3;
    for (; t + 3 <= nk; t += 3) {
        FLAT_STEP(t, bs[0], bs[2], WAIT_A, WAIT_B);
        FLAT_STEP(t + 1, bs[1], bs[0], WAIT_A, WAIT_B);
        FLAT_STEP(t + 2, bs[2], bs[1], WAIT_A, WAIT_B);
    }
    // the last one or two steps wait for every earlier load (their own B loads
    // are never used, and the compiler may drop them)
    if (t < nk) FLAT_STEP(t, bs[0], bs[2], 0, 0);
    if (t + 1 < nk) FLAT_STEP(t + 1, bs[1], bs[0], 0, 0);
#undef FLAT_STEP
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_waitcnt(kLgkmcnt0);

    const int row0w = m0 + wm * 32 * BI;
#pragma unroll
    for (int k = 0; k < BJ; k++) {
        const int col = cb[k] * 32 + c;
        // (stage 1: other waves may be raising it; one value for the wave)
        if (!live[k] || __builtin_amdgcn_readfirstlane(g.skip[op[k]])) continue;
        const uint64_t valid = __builtin_amdgcn_ballot_w64(col < g.N);
        const float t_scale = EPI_T ? ldexpf(1.0f, -g.t_e[op[k]]) : 1.0f;
        TWatch watch[BI];
        auto judge = [&]() __attribute__((always_inline)) {
            bool suspect = false;
            if (row0w + 32 * BI > g.M)
#pragma unroll
                for (int i = 0; i < BI; i++) {
                    const int rows = g.M - row0w - 32 * i;
                    watch[i].below &= TWatch::inside(rows, lane);
                    // a block cut off at M may be out of range with fewer entries below
                    const uint64_t one = __builtin_amdgcn_ballot_w64(watch[i].below != 0) & valid;
                    suspect |= rows > 0 && rows < 32 && 12 * __builtin_popcountll(one) >= __builtin_popcountll(valid);
                }
            if (!t_suspect(watch, valid, lane) && !suspect) return;
            uint32_t filled[BI];
#pragma unroll
            for (int i = 0; i < BI; i++)
                filled[i] = (valid >> lane) & 1
                                ? TWatch::filled(acc[i][k]) & TWatch::inside(g.M - row0w - 32 * i, lane)
                                : 0u;
            if (t_out_of_range(watch, filled) && lane == 0) {
                atomicOr(&g.skip[op[k]], kSkipStage1);
                atomicOr(g.any, 1);
            }
        };
        if (EPI_T && DS == 2) {
            // (33 operators of 500 states, kept 480, two states: single stores
            // 120 us, exchanged 78 us for stage 1)
            // rows row0 .. row0 + 3 are two beta of two states: lanes of two
            // neighbouring columns exchange halves, so that each stores four
            // k of one beta (a column past N holds zeros: k padding)
            uint16_t* th = g.t_hi + op[k] * g.t_bs;
            uint16_t* tl = g.t_lo + op[k] * g.t_bs;
            const bool odd = c & 1, in = col < g.N, store = col - (odd ? 1 : 0) < g.N;
#pragma unroll
            for (int i = 0; i < BI; i++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = row0w + i * 32 + 8 * q + 4 * h;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = in ? acc[i][k][4 * q + e] * t_scale : 0.f;
                    const u32x2 p0 = split2_f16(v[0], v[1]), p1 = split2_f16(v[2], v[3]);
                    watch[i].add(q, p0[0], p1[0]);
                    const uint32_t rh = __shfl_xor(odd ? p0[0] : p1[0], 1), rl = __shfl_xor(odd ? p0[1] : p1[1], 1);
                    const int beta = (row0 >> 1) + (odd ? 1 : 0);
                    if (store && beta * 2 < g.M) {
                        const int64_t off = slab_off(beta, (int64_t)(col & ~1) * 2, g.t_rows);
                        *reinterpret_cast<u32x2*>(th + off) = odd ? u32x2{rh, p1[0]} : u32x2{p0[0], rh};
                        *reinterpret_cast<u32x2*>(tl + off) = odd ? u32x2{rl, p1[1]} : u32x2{p0[1], rl};
                    }
                }
            judge();
            continue;
        }
        if (!EPI_T && col >= g.N) continue;
        if (EPI_T) {
            uint16_t* th = g.t_hi + op[k] * g.t_bs;
            uint16_t* tl = g.t_lo + op[k] * g.t_bs;
#pragma unroll
            for (int i = 0; i < BI; i++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = row0w + i * 32 + 8 * q + 4 * h;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = acc[i][k][4 * q + e] * t_scale;
                    const u32x2 p0 = split2_f16(v[0], v[1]), p1 = split2_f16(v[2], v[3]);
                    const u32x2 hv = {p0[0], p1[0]}, lv = {p0[1], p1[1]};
                    watch[i].add(q, hv[0], hv[1]);
                    if (col >= g.N) continue;
                    if (DS == 4) {
                        if (row0 < g.M) {
                            const int64_t off = slab_off(row0 >> 2, (int64_t)col * 4, g.t_rows);
                            *reinterpret_cast<u32x2*>(th + off) = hv;
                            *reinterpret_cast<u32x2*>(tl + off) = lv;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int row = row0 + e;
                            if (row < g.M) {
                                const int64_t off = slab_off(row / g.d, (int64_t)col * g.d + row % g.d, g.t_rows);
                                th[off] = (uint16_t)(hv[e >> 1] >> (16 * (e & 1)));
                                tl[off] = (uint16_t)(lv[e >> 1] >> (16 * (e & 1)));
                            }
                        }
                    }
                }
            judge();
        } else if (g.upper) {
            float* cp = g.c + part * g.c_ps + op[k] * g.c_bs;
            const int e0 = -(g.op_e[op[k]] + g.col_e[col]);
#pragma unroll
            for (int i = 0; i < BI; i++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = row0w + i * 32 + 8 * q + 4 * h;
                    if (row0 > col) continue;
                    const i32x4 er = *reinterpret_cast<const i32x4*>(g.row_e + row0);
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = ldexpf(acc[i][k][4 * q + e], e0 - er[e]);
                    float* mirror = cp + (int64_t)col * g.ldc + row0;
                    if (row0 + 3 <= col) {
                        *reinterpret_cast<f32x4u*>(mirror) = v;
#pragma unroll
                        for (int e = 0; e < 4; e++) cp[(int64_t)(row0 + e) * g.ldc + col] = v[e];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (row0 + e <= col) {
                                mirror[e] = v[e];
                                cp[(int64_t)(row0 + e) * g.ldc + col] = v[e];
                            }
                    }
                }
        } else {
            float* cp = g.c + part * g.c_ps + op[k] * g.c_bs + col;
            const int e0 = -(g.op_e[op[k]] + g.col_e[col]);
#pragma unroll
            for (int i = 0; i < BI; i++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row0 = row0w + i * 32 + 8 * q + 4 * h;
                    const i32x4 er = *reinterpret_cast<const i32x4*>(g.row_e + row0);
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        if (row0 + e < g.M) cp[(int64_t)(row0 + e) * g.ldc] = ldexpf(acc[i][k][4 * q + e], e0 - er[e]);
                }
        }
    }
}

template <int BI, bool EPI_T, int DS>
__global__ __launch_bounds__(512, 1) void gemm_flat_kernel(FlatDesc g) {
    __shared__ __attribute__((aligned(1024))) uint16_t lds[kFlatLds];
    const int lin = xcd_linear_id();
    const int mt = lin % g.tiles_m, r = lin / g.tiles_m, nt = r % g.tiles_n, part = r / g.tiles_n;
    const int m0 = mt * 64 * BI;
    if (!EPI_T && g.upper) {
        // the tile's 8 blocks: their largest column is one operator's last
        // block's if the tile crosses an operator's end, else the last one's
        const int bpo = g.n32 >> 5, first = nt * 8, last = min(first + 7, bpo * g.batch - 1);
        const int top = first / bpo == last / bpo ? last % bpo : bpo - 1;
        if (m0 > top * 32 + 31) return;
    }
    // M tiles fastest: neighbouring workgroups share the B panel
    const int rest = min(BI, (g.M - m0 + 63) / 64);
    if (rest == BI) flat_tile<BI, EPI_T, DS>(g, lds, m0, nt, part);
    else if (BI > 3 && rest == 3) flat_tile<BI < 3 ? BI : 3, EPI_T, DS>(g, lds, m0, nt, part);
    else if (BI > 2 && rest == 2) flat_tile<BI < 2 ? BI : 2, EPI_T, DS>(g, lds, m0, nt, part);
    else flat_tile<1, EPI_T, DS>(g, lds, m0, nt, part);
}

// One tile of a list of products (a plan's): rows m0 .. of 64 bi rows, column
// tile nt.
struct FlatTile {
    int piece, m0, nt, bi;
};

// Tiles of many products in one launch, longest first (flat_list): the last
// round of one product's tiles is filled by the next one's.
template <bool EPI_T, int DS>
__global__ __launch_bounds__(512, 1) void gemm_flat_list_kernel(const FlatDesc* tab, const FlatTile* list) {
    __shared__ __attribute__((aligned(1024))) uint16_t lds[kFlatLds];
    const FlatTile t = list[blockIdx.x];
    const FlatDesc g = tab[t.piece];
    switch (t.bi) {
        case 4: flat_tile<4, EPI_T, DS>(g, lds, t.m0, t.nt, 0); break;
        case 3: flat_tile<3, EPI_T, DS>(g, lds, t.m0, t.nt, 0); break;
        case 2: flat_tile<2, EPI_T, DS>(g, lds, t.m0, t.nt, 0); break;
        default: flat_tile<1, EPI_T, DS>(g, lds, t.m0, t.nt, 0); break;
    }
}

constexpr int kF16MaxSite = 8;          // a split block holds 16 j of all site states
constexpr int kF16RowSpread = 12;       // log2 of the accepted spread of row maxima
constexpr int kPrepRows = 256;          // rows of U per partial column maximum
constexpr int kPrepORows = 32;          // rows of O per partial maximum
constexpr uint32_t kInfBits = 0x7f800000u;

// A workgroup of the passes over a list of groups.
struct PairBlock {
    int piece, blk;
};

// Launch-time sizes and pointers of the scale pass.
struct F16Scale {
    const float* U;
    int rows, mp, d;
    int64_t ldu;
    const float* O;
    int m, nb;
    int64_t ldo, stride_o;
    uint32_t* upart;   // [chunk][mp]: largest |U| of a column in kPrepRows rows (bits)
    uint32_t* ublk;    // [U block of the scale pass]: largest |U|
    uint32_t* opart;   // [b][row block][3]: largest |O|, smallest non-zero row maximum, largest row sum of |O|
    int* eu;           // [mp]
    int n_ublk;
    int m32, mp32;     // rows of O_b's and T_b's layouts
    int *eo, *et;      // [nb]: exponents of O_b less T_b's, and of T_b
    int* skip;         // [nb], cleared by the scale pass
    UState* u;         // cleared by the scale pass when it works on U
    int* any;          // raised when an operator is skipped (behind skip; plans: one per chunk)
    uint16_t *u1h, *u1l, *u2h, *u2l;
    uint16_t *oh, *ol;
    int64_t o_bs;
    uint16_t *th, *tl;
    int64_t t_bs;
    int u_blocks;      // workgroups that work on U (0: done by an earlier chunk)
    int o_blocks;      // and on O
    // Blocked with a site (f16_site): U2 is made of Up (packed) instead of U,
    // and both of the d site states listed in sel (4 bits each) out of d_all;
    // the passes' first half of workgroups on U takes U, the second Up, with
    // partial maxima and exponents of its own
    const float* Up;
    int d_all;
    uint32_t sel;
    uint32_t* upart2;
    int* eu2;
};

inline __host__ __device__ int div_up(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

__device__ inline uint32_t abs_bits(float x) { return __float_as_uint(x) & 0x7fffffffu; }
__device__ inline uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ inline uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Power of two that brings a largest magnitude (bits) into [2^14, 2^15).
__device__ inline int scale_exp(uint32_t bits) {
    if (bits == 0 || bits >= kInfBits) return 0;
    return 14 - ilogbf(__uint_as_float(bits));
}

// Power of two that the scaled operator's row sums stay below: by the largest of
// them (bits), or where that overflows by the largest entry (bits) and m.
__device__ inline int t_exp(uint32_t mx, uint32_t most, int m) {
    if (mx == 0 || mx >= kInfBits) return 0;
    if (most >= kInfBits) return 15 + 32 - __builtin_clz(m);
    return scale_exp(mx) + ilogbf(__uint_as_float(most)) + 1;
}

// The eight values of all lanes, each reduced over the wave: eight lanes end with
// each of them (10 exchanges; one by one it would be 48).
template <typename T, typename F>
__device__ inline T row_of_eight(const T (&v)[8], int lane, F f) {
    T a[4], b[2], c;
#pragma unroll
    for (int k = 0; k < 4; k++) a[k] = f(lane & 32 ? v[k + 4] : v[k], __shfl_xor(lane & 32 ? v[k] : v[k + 4], 32));
#pragma unroll
    for (int k = 0; k < 2; k++) b[k] = f(lane & 16 ? a[k + 2] : a[k], __shfl_xor(lane & 16 ? a[k] : a[k + 2], 16));
    c = f(lane & 8 ? b[1] : b[0], __shfl_xor(lane & 8 ? b[0] : b[1], 8));
#pragma unroll
    for (int s = 4; s; s >>= 1) c = f(c, __shfl_xor(c, s));
    return c;
}

// Partial maxima of |U| per column (of the listed site states) and of |O| per
// operator, and of all of U per workgroup.  Bound by the one read of O and U.
template <bool SITE>
__device__ inline void f16_scale_block(const F16Scale& g, int blk) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ uint32_t red[4][64], red2[SITE ? 4 : 1][64];
    if (blk < g.u_blocks) {
        if (blk == 0 && tid == 0) *g.u = UState{0, 0};
        const int cb = div_up(g.mp, 64), half = g.u_blocks / 2;
        const bool up = SITE && blk >= half;
        const int x = up ? blk - half : blk;
        const float* U = up ? g.Up : g.U;
        const int64_t ldu = up ? g.mp : g.ldu;
        const int c = (x % cb) * 64 + lane, r0 = (x / cb) * kPrepRows;
        const int r1 = min(r0 + kPrepRows, SITE ? g.m * g.d_all : g.rows);
        uint32_t mx = 0, all = 0, listed = 0;
        if (SITE)
            for (int k = 0; k < g.d; k++) listed |= 1u << ((g.sel >> (4 * k)) & 15);
        if (c < g.mp) {
#pragma unroll 16
            for (int r = r0 + wave; r < r1; r += 4) {
                const uint32_t v = abs_bits(U[(int64_t)r * ldu + c]);
                mx = umax32(mx, !SITE || (listed >> (r % g.d_all)) & 1 ? v : 0u);
                if (SITE) all = umax32(all, v);
            }
        }
        red[wave][lane] = mx;
        if (SITE) red2[wave][lane] = all;
        __syncthreads();
        if (wave == 0) {
            mx = umax32(umax32(red[0][lane], red[1][lane]), umax32(red[2][lane], red[3][lane]));
            if (c < g.mp) (up ? g.upart2 : g.upart)[(int64_t)(x / cb) * g.mp + c] = mx;
            if (SITE)
                mx = umax32(umax32(red2[0][lane], red2[1][lane]), umax32(red2[2][lane], red2[3][lane]));
#pragma unroll
            for (int s = 32; s; s >>= 1) mx = umax32(mx, __shfl_xor(mx, s));
            if (lane == 0) g.ublk[blk] = mx;
        }
        return;
    }
    blk -= g.u_blocks;
    const int rb = div_up(g.m, kPrepORows);
    const int b = blk / rb, i0 = (blk % rb) * kPrepORows;
    if (i0 == 0 && tid == 0) g.skip[b] = 0;
    const float* src = g.O + (int64_t)b * g.stride_o;
    uint32_t mx = 0, mn = 0xffffffffu, most = 0;
    // eight rows per wave, their loads in flight together (rows past the last
    // repeat it)
    constexpr int RW = kPrepORows / 4;
    const int r0 = i0 + wave * RW;
    if (r0 < g.m) {
        uint32_t x[RW];
        float sum[RW];
#pragma unroll
        for (int k = 0; k < RW; k++) {
            x[k] = 0;
            sum[k] = 0.f;
        }
        const int m4 = g.m & ~3;
#pragma unroll 2
        for (int j = lane * 4; j < m4; j += 256)
#pragma unroll
            for (int k = 0; k < RW; k++) {
                const f32x4u v = *reinterpret_cast<const f32x4u*>(src + (int64_t)min(r0 + k, g.m - 1) * g.ldo + j);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    x[k] = umax32(x[k], abs_bits(v[e]));
                    sum[k] += fabsf(v[e]);
                }
            }
        if (m4 + lane < g.m)
#pragma unroll
            for (int k = 0; k < RW; k++) {
                const float v = src[(int64_t)min(r0 + k, g.m - 1) * g.ldo + m4 + lane];
                x[k] = umax32(x[k], abs_bits(v));
                sum[k] += fabsf(v);
            }
        // eight lanes to each row, then one value for all
        static_assert(RW == 8, "rows of a wave");
        const uint32_t row = row_of_eight(x, lane, [](uint32_t a, uint32_t b) { return umax32(a, b); });
        mx = row;
        mn = row ? row : mn;
        most = abs_bits(row_of_eight(sum, lane, [](float a, float b) { return a + b; }));
#pragma unroll
        for (int s = 32; s >= 8; s >>= 1) {
            mx = umax32(mx, __shfl_xor(mx, s));
            mn = umin32(mn, __shfl_xor(mn, s));
            most = umax32(most, __shfl_xor(most, s));
        }
    }
    if (lane == 0) {
        red[0][wave] = mx;
        red[1][wave] = mn;
        red[2][wave] = most;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t* o = g.opart + 3 * ((int64_t)b * rb + i0 / kPrepORows);
        o[0] = umax32(umax32(red[0][0], red[0][1]), umax32(red[0][2], red[0][3]));
        o[1] = umin32(umin32(red[1][0], red[1][1]), umin32(red[1][2], red[1][3]));
        o[2] = umax32(umax32(red[2][0], red[2][1]), umax32(red[2][2], red[2][3]));
    }
}

template <bool SITE>
__global__ __launch_bounds__(256) void f16_scale_kernel(F16Scale g) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *g.any = 0;
    f16_scale_block<SITE>(g, blockIdx.x);
}

// The same over a list of groups (a plan's); the first workgroup clears the
// flag that the split pass raises for a skipped operator.
__global__ __launch_bounds__(256) void f16_scale_list_kernel(const F16Scale* tab, const PairBlock* list, int* any) {
    const PairBlock b = list[blockIdx.x];
    const F16Scale g = tab[b.piece];
    if (blockIdx.x == 0 && threadIdx.x == 0) *any = 0;
    f16_scale_block<false>(g, b.blk);
}

// U, O and T's K padding into the slab layout:
//   U1 (d*mp rows, K = m):   element (beta*d + s, j) = U[j*d+s][beta] 2^eu[beta]
//   U2 (mp rows, K = m*d):   element (alpha, r)      = U[r][alpha] 2^eu[alpha]
//   O_b (m32 rows, K = m):   element (i, j)          = O_b[i][j] 2^eo[b]
// A workgroup on U takes 16 j (16 d rows) x 64 columns through LDS: one slab
// of U1's rows and d slabs of U2's, both written in whole 16-byte chunks,
// chunk after chunk.  One on O takes a 64 x 64 block (split_o_kernel's
// scheme).  The first block of each operator records eo[b]; each raises skip[b]
// (on U: u->bad) where its entries are out of range.
// With a site, the first half of the workgroups on U writes U1 from U and the
// second U2 from Up.
template <int DMAX, bool SITE>
__device__ inline void f16_split_block(const F16Scale& g, int blk) {
    static_assert(DMAX <= kF16MaxSite, "tile size");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ __attribute__((aligned(16))) float tile[DMAX <= 4 ? 64 * 68 : 16 * DMAX * 65];
    __shared__ int s_e[64];
    __shared__ uint32_t s_mx[4][64];
    const int u_chunks = div_up(SITE ? g.m * g.d_all : g.rows, kPrepRows);
    auto store8 = [&](uint16_t* hi, uint16_t* lo, const float (&v)[8]) {
        const u32x2 p0 = split2_f16(v[0], v[1]), p1 = split2_f16(v[2], v[3]);
        const u32x2 p2 = split2_f16(v[4], v[5]), p3 = split2_f16(v[6], v[7]);
        *reinterpret_cast<u32x4*>(hi) = u32x4{p0[0], p1[0], p2[0], p3[0]};
        *reinterpret_cast<u32x4*>(lo) = u32x4{p0[1], p1[1], p2[1], p3[1]};
    };
    if (blk < g.u_blocks) {
        const bool up = SITE && blk >= g.u_blocks / 2;
        if (up) blk -= g.u_blocks / 2;
        const float* U = up ? g.Up : g.U;
        const int64_t ldu = up ? g.mp : g.ldu;
        const uint32_t* upart = up ? g.upart2 : g.upart;
        const int cb = div_up(g.mp, 64), d = g.d;
        const int a0 = (blk % cb) * 64, q = blk / cb, r0 = q * 16 * d, nr = 16 * d;
        const int a = a0 + lane;
        // loads first (clamped addresses, all in flight together), then LDS
        const int ac = min(a, g.mp - 1);
        uint32_t mx = 0;
#pragma unroll 4
        for (int x = wave; x < u_chunks; x += 4) mx = umax32(mx, upart[(int64_t)x * g.mp + ac]);
        float v[DMAX * 4];
#pragma unroll
        for (int k = 0; k < DMAX * 4; k++) {
            int64_t row = min(r0 + wave + 4 * k, g.rows - 1);
            if (SITE) {
                const int j = (int)row / d, t = (int)row - j * d;
                row = (int64_t)j * g.d_all + ((g.sel >> (4 * t)) & 15);
            }
            v[k] = U[row * ldu + ac];
        }
        s_mx[wave][lane] = mx;
#pragma unroll
        for (int k = 0; k < DMAX * 4; k++)
            if (wave + 4 * k < nr) tile[(wave + 4 * k) * 65 + lane] = r0 + wave + 4 * k < g.rows ? v[k] : 0.f;
        __syncthreads();
        if (wave == 0) {
            mx = umax32(umax32(s_mx[0][lane], s_mx[1][lane]), umax32(s_mx[2][lane], s_mx[3][lane]));
            s_e[lane] = scale_exp(mx);
            if (q == 0 && a < g.mp) (up ? g.eu2 : g.eu)[a] = scale_exp(mx);
        }
        __syncthreads();
        const int na = min(64, g.mp - a0);
        // entries below the pairs' range: three of a thread's eight, or a
        // quarter of a row's 32 among the wave's (two rows take turns in it);
        // and how full the eights are
        bool u_bad = false;
        int filled = 0, runs = 0;
        auto check = [&](const float (&v)[8]) {
            int small = 0, n = 0;
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const bool s = pair_small(v[k]);
                small += s;
                n += v[k] != 0.f;
                u_bad |= __builtin_popcountll(__ballot(s)) >= 8;
            }
            u_bad |= small >= 3;
            filled += n;
            runs += n >= 5 ? 1 : n ? -1 : 0;
        };
        // U1: rows a*d + s of slab q, chunk (row, slot)
        const int64_t rows1 = (int64_t)d * g.mp;
        for (int x = up ? na * d * 2 : tid; x < na * d * 2; x += 256) {
            const int row = x >> 1, slot = x & 1, al = row / d, s = row - al * d;
            const int64_t gr = (int64_t)a0 * d + row;
            const int half = slot ^ (int)((gr >> 3) & 1), e = s_e[al];
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = ldexpf(tile[((half * 8 + k) * d + s) * 65 + al], e);
            check(v);
            const int64_t off = (int64_t)q * rows1 * kSlabK + gr * kSlabK + slot * 8;
            store8(g.u1h + off, g.u1l + off, v);
        }
        // U2: rows a of slabs q*d .. q*d + d - 1
        const int64_t ns2 = n_slabs(g.rows);
        for (int x = SITE && !up ? na * d * 2 : tid; x < na * d * 2; x += 256) {
            const int sl = x / (na * 2), y = x - sl * (na * 2), al = y >> 1, slot = y & 1;
            const int64_t sq = (int64_t)q * d + sl;
            if (sq >= ns2) break;
            const int half = slot ^ (((a0 + al) >> 3) & 1), e = s_e[al];
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = ldexpf(tile[(sl * 16 + half * 8 + k) * 65 + al], e);
            if (SITE) check(v);
            const int64_t off = sq * (int64_t)g.mp * kSlabK + (int64_t)(a0 + al) * kSlabK + slot * 8;
            store8(g.u2h + off, g.u2l + off, v);
        }
        if (__any(u_bad) && lane == 0) atomicOr(&g.u->bad, 1);
#pragma unroll
        for (int s = 32; s; s >>= 1) {
            filled += __shfl_xor(filled, s);
            runs += __shfl_xor(runs, s);
        }
        if (lane == 0) {
            s_mx[wave][0] = (uint32_t)filled;
            s_mx[wave][1] = (uint32_t)runs;
        }
        __syncthreads();
        if (tid == 0) {
            const uint32_t n = s_mx[0][0] + s_mx[1][0] + s_mx[2][0] + s_mx[3][0];
            const uint32_t r = s_mx[0][1] + s_mx[1][1] + s_mx[2][1] + s_mx[3][1];
            atomicAdd(&g.u->filled_runs, (unsigned long long)r << 32 | n);
        }
        return;
    }
    blk -= g.u_blocks;
    if (blk < g.o_blocks) {
        const int tb = div_up(g.m, 64);
        const int b = blk / (tb * tb), t = blk % (tb * tb), i0 = (t / tb) * 64, j0 = (t % tb) * 64;
        const float* src = g.O + (int64_t)b * g.stride_o;
        if (j0 + 64 <= g.m) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int r = (tid >> 4) + 16 * k, c4 = (tid & 15) * 4, i = i0 + r;
                // rows past the last repeat it (they are not written)
                *reinterpret_cast<f32x4*>(&tile[r * 68 + c4]) =
                    *reinterpret_cast<const f32x4u*>(src + (int64_t)min(i, g.m - 1) * g.ldo + j0 + c4);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const int i = i0 + wave + 4 * k, j = j0 + lane;
                tile[(wave + 4 * k) * 68 + lane] = (i < g.m && j < g.m) ? src[(int64_t)i * g.ldo + j] : 0.f;
            }
        }
        if (wave == 0) {
            const int rb = div_up(g.m, kPrepORows);
            const uint32_t* p = g.opart + 3 * (int64_t)b * rb;
            uint32_t mx = 0, mn = 0xffffffffu, most = 0;
            for (int x = lane; x < rb; x += 64) {
                mx = umax32(mx, p[3 * x]);
                mn = umin32(mn, p[3 * x + 1]);
                most = umax32(most, p[3 * x + 2]);
            }
            for (int s = 32; s; s >>= 1) {
                mx = umax32(mx, __shfl_xor(mx, s));
                mn = umin32(mn, __shfl_xor(mn, s));
                most = umax32(most, __shfl_xor(most, s));
            }
            if (lane == 0) s_e[0] = scale_exp(mx);
            if (t == 0) {
                bool bad = mx >= kInfBits ||
                           (mx && ilogbf(__uint_as_float(mx)) - ilogbf(__uint_as_float(mn)) > kF16RowSpread);
                for (int x = lane; x < g.n_ublk; x += 64) bad |= g.ublk[x] >= kInfBits;
                bad = __any(bad);
                if (lane == 0) {
                    g.et[b] = t_exp(mx, most, g.m);
                    g.eo[b] = scale_exp(mx) - t_exp(mx, most, g.m);
                    if (bad) {
                        atomicOr(&g.skip[b], kSkipSplit);
                        atomicOr(g.any, 1);
                    }
                }
            }
        }
        __syncthreads();
        const int e = s_e[0];
        const int64_t nslab = n_slabs(g.m);
        int small = 0;
        bool bad = false;
#pragma unroll
        for (int x = 0; x < 2; x++) {
            const int ch = tid + 256 * x;  // slab q, k half, row
            const int q = ch >> 7, half = (ch >> 6) & 1, row = ch & 63;
            const int i = i0 + row;
            const int64_t sq = j0 / kSlabK + q;
            if (i >= g.m || sq >= nslab) continue;
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) {
                v[k] = ldexpf(tile[row * 68 + q * kSlabK + half * 8 + k], e);
                const bool s = pair_small(v[k]);
                small += s;
                bad |= __builtin_popcountll(__ballot(s)) >= 16;  // of a column's 64 rows
            }
            const int64_t off = (int64_t)b * g.o_bs + sq * (int64_t)g.m32 * kSlabK + (int64_t)i * kSlabK +
                                (half ^ ((i >> 3) & 1)) * 8;
            store8(g.oh + off, g.ol + off, v);
        }
        if (__any(bad || small >= 4) && lane == 0) {
            atomicOr(&g.skip[b], kSkipSplit);
            atomicOr(g.any, 1);
        }
        return;
    }
    // T's last slab (stage 1 writes only k < m*d): zeros, 16 bytes per chunk
    blk -= g.o_blocks;
    const int tb = div_up((int64_t)g.mp * 2, 256);
    const int b = blk / tb, x = (blk % tb) * 256 + tid;
    if (x >= g.mp * 2) return;
    const int64_t off = (int64_t)b * g.t_bs + (n_slabs(g.rows) - 1) * (int64_t)g.mp32 * kSlabK + (int64_t)x * 8;
    *reinterpret_cast<u32x4*>(g.th + off) = u32x4{0, 0, 0, 0};
    *reinterpret_cast<u32x4*>(g.tl + off) = u32x4{0, 0, 0, 0};
}

template <int DMAX, bool SITE>
__global__ __launch_bounds__(256) void f16_split_kernel(F16Scale g) {
    f16_split_block<DMAX, SITE>(g, blockIdx.x);
}

template <int DMAX>
__global__ __launch_bounds__(256) void f16_split_list_kernel(const F16Scale* tab, const PairBlock* list) {
    const PairBlock b = list[blockIdx.x];
    const F16Scale g = tab[b.piece];
    f16_split_block<DMAX, false>(g, b.blk);
}

// us per slab of a tile of 64 bi rows with the chip full (1024-state batches
// of 64 operators, stage 2), and around its K loop.
constexpr double kFlatCost[5] = {0, 0.66, 0.74, 0.96, 1.22};
constexpr double kFlatAround = 5;

// Rows per tile (64 bi) and K parts of a flat product.
struct FlatCfg {
    int bi, parts, part_slabs;
};

// The choice with the least estimated time: tiles go to 256 CUs one per CU
// (the ring fills the LDS), so a launch takes whole rounds of its tile's
// time; smaller tiles cost more per row and K parts cost a pass over the
// partial results, and pay where the tiles are too few to fill the chip
// (512 states, 48 operators, stage 2: 256-row tiles 0.145 ms, 192: 0.20,
// 128: 0.20; 256 states, 20 operators, stage 1: 25.0 against 18.3 us for
// 128 rows).  At least min_parts.  out_bytes: bytes of the whole result, read and written once more per part.
FlatCfg flat_cfg(int M, int blocks, int slabs, int min_parts, int max_parts, double out_bytes) {
    const double* cost = kFlatCost;
    const double around = kFlatAround;
    FlatCfg best{4, 1, slabs};
    double best_t = 1e30;
    const int tn = div_up(blocks, 8);
    for (int bi = 4; bi >= 1; bi--)
        for (int parts = min_parts; parts <= max_parts; parts++) {
            const int ps = div_up(slabs, parts);
            if (parts > min_parts && (ps < 8 || (int64_t)ps * (parts - 1) >= slabs - 2)) break;
            const int full = M / (64 * bi), rest = div_up(M - full * 64 * bi, 64);
            const double tf = cost[bi] * ps + around, tr = rest ? cost[rest] * ps + around : 0;
            const double tiles = (double)(full + (rest > 0)) * tn * parts;
            const double busy = (full * tf + tr) * tn * parts / 256;
            // whole rounds when all tiles are alike, about half a tile of tail otherwise
            double t = full ? (rest ? std::max(tf, busy + 0.4 * tf) : std::ceil(tiles / 256) * tf) : std::ceil(tiles / 256) * tr;
            if (tiles <= 256) t = full ? tf : tr;
            if (parts > 1) t += 4 + (parts + 1) * out_bytes / 4e6;
            if (t < best_t * 0.97) {
                best_t = t;
                best = {bi, parts, ps};
            }
        }
    return best;
}

constexpr int kF16MaxParts = 8;

template <bool EPI_T, int DS>
hipError_t launch_flat(FlatDesc g, const FlatCfg& c, hipStream_t s) {
    g.parts = c.parts;
    g.part_slabs = c.part_slabs;
    g.tiles_m = div_up(g.M, 64 * c.bi);
    g.tiles_n = div_up((int64_t)g.batch * (g.n32 / 32), 8);
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n * g.parts;
    if (tiles > 0x7fffffff || n_slabs(g.K) - (int64_t)(g.parts - 1) * g.part_slabs < 3) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(512);
    switch (c.bi) {
        case 1: hipLaunchKernelGGL((gemm_flat_kernel<1, EPI_T, DS>), grid, block, 0, s, g); break;
        case 2: hipLaunchKernelGGL((gemm_flat_kernel<2, EPI_T, DS>), grid, block, 0, s, g); break;
        case 3: hipLaunchKernelGGL((gemm_flat_kernel<3, EPI_T, DS>), grid, block, 0, s, g); break;
        default: hipLaunchKernelGGL((gemm_flat_kernel<4, EPI_T, DS>), grid, block, 0, s, g); break;
    }
    return hipGetLastError();
}

struct F16Layout {
    int m32, mp32;
    size_t u1, u2;              // bytes of one array (hi or lo)
    size_t t_op, o_op;          // one operator's
    size_t t32;                 // one operator's T of the FP32 kernels
    size_t part_u, ublk, eu;    // scale pass: partial column maxima, block maxima, exponents
    size_t u_state;
    size_t shared;
};

F16Layout f16_layout(const rot_problem& p, int d_all = 0) {
    F16Layout L;
    const int64_t md = (int64_t)p.m * p.d, all = d_all ? (int64_t)p.m * d_all : md;
    L.m32 = div_up(p.m, 32) * 32;
    L.mp32 = div_up(p.mp, 32) * 32;
    L.u1 = al256((size_t)(n_slabs(p.m) * p.d * p.mp * kSlabK * 2));
    L.u2 = al256((size_t)(n_slabs(md) * p.mp * kSlabK * 2));
    L.o_op = (size_t)(n_slabs(p.m) * L.m32 * kSlabK * 2);
    L.t_op = (size_t)(n_slabs(md) * L.mp32 * kSlabK * 2);
    L.t32 = al256((size_t)all * p.ldu * 4);
    const size_t chunks = div_up(all, kPrepRows);
    L.part_u = al256(chunks * p.mp * 4);
    L.ublk = al256((d_all ? 2 : 1) * chunks * div_up(p.mp, 64) * 4);
    L.eu = al256((size_t)(p.mp + 256) * 4);  // read in groups of four up to a tile's last row
    L.u_state = al256(sizeof(UState));
    L.shared = L.u_state + 2 * L.u1 + 2 * L.u2 + (d_all ? 2 : 1) * (L.part_u + L.eu) + L.ublk;
    return L;
}

size_t f16_t_bytes(const F16Layout& L, int ops) { return std::max(2 * al256(ops * L.t_op), ops * L.t32); }
size_t f16_scale_bytes(const rot_problem& p, int ops) {
    return al256((size_t)ops * (div_up(p.m, kPrepORows) * 12 + 12) + 4);
}
// Stage 2 of `ops` operators of the group.  The K parts are those of the
// whole group, so that results do not depend on the chunks.  Symmetric output
// computes the tiles on or above the diagonal, a little over half of them:
// the choice is made for that many operators.
FlatCfg f16_stage2_cfg(const rot_problem& p, int ops, bool symmetric) {
    const int slabs = (int)n_slabs((int64_t)p.m * p.d), bpo = div_up(p.mp, 32);
    auto tiled = [&](int n) { return symmetric ? (n * 5 + 7) / 8 : n; };
    // where the FP32 kernels split K, sums must not get longer than theirs (3
    // roundings per 16 k against 8)
    int kp;
    int least = symmetric ? 1 : (stage2_parts(p, p.n_ops, &kp) * 3 + 7) / 8;
    while (least > 1 && slabs - div_up(slabs, least) * (least - 1) < 3) least--;
    const int parts = flat_cfg(p.mp, tiled(p.n_ops) * bpo, slabs, least, kF16MaxParts, 4.0 * p.n_ops * p.mp * p.mp).parts;
    return flat_cfg(p.mp, tiled(ops) * bpo, slabs, parts, parts, 0);
}
// The split O, and later (stage 1 done) stage 2's partial results.
size_t f16_o_bytes(const rot_problem& p, const F16Layout& L, int ops, int parts) {
    return std::max(2 * al256(ops * L.o_op), parts > 1 ? al256((size_t)parts * ops * p.mp * p.mp * 4) : 0);
}

// Operators b0 .. b0 + nb - 1 of p (leading dimensions resolved) laid out in a
// workspace: the scale and split passes' table (block counts left out), T's
// place (pairs, and later the FP32 kernels' intermediates) and O's (pairs, and
// later stage 2's partial results).
struct F16Bound {
    F16Scale g;
    char *T, *O;
};
F16Bound f16_bind(const rot_problem& p, const F16Layout& L, int b0, int nb, int parts, void* ws) {
    char* base = static_cast<char*>(ws);
    auto take = [&](size_t bytes) {
        char* q = base;
        base += bytes;
        return q;
    };
    F16Bound r{};
    F16Scale& g = r.g;
    g.U = static_cast<const float*>(p.U);
    g.rows = p.m * p.d;
    g.mp = p.mp;
    g.d = p.d;
    g.ldu = p.ldu;
    g.O = static_cast<const float*>(p.O) + (int64_t)b0 * p.stride_o;
    g.m = p.m;
    g.nb = nb;
    g.m32 = L.m32;
    g.mp32 = L.mp32;
    g.ldo = p.ldo;
    g.stride_o = p.stride_o;
    g.u1h = reinterpret_cast<uint16_t*>(take(L.u1));
    g.u1l = reinterpret_cast<uint16_t*>(take(L.u1));
    g.u2h = reinterpret_cast<uint16_t*>(take(L.u2));
    g.u2l = reinterpret_cast<uint16_t*>(take(L.u2));
    g.upart = reinterpret_cast<uint32_t*>(take(L.part_u));
    g.ublk = reinterpret_cast<uint32_t*>(take(L.ublk));
    g.eu = reinterpret_cast<int*>(take(L.eu));
    g.u = reinterpret_cast<UState*>(take(L.u_state));
    r.T = take(f16_t_bytes(L, nb));
    g.th = reinterpret_cast<uint16_t*>(r.T);
    g.tl = reinterpret_cast<uint16_t*>(r.T + al256(nb * L.t_op));
    g.t_bs = (int64_t)(L.t_op / 2);
    r.O = take(f16_o_bytes(p, L, nb, parts));
    g.oh = reinterpret_cast<uint16_t*>(r.O);
    g.ol = reinterpret_cast<uint16_t*>(r.O + al256(nb * L.o_op));
    g.o_bs = (int64_t)(L.o_op / 2);
    g.opart = reinterpret_cast<uint32_t*>(base);
    g.eo = reinterpret_cast<int*>(g.opart + 3 * (size_t)nb * div_up(p.m, kPrepORows));
    g.et = g.eo + nb;
    g.skip = g.et + nb;
    g.any = g.skip + nb;
    g.n_ublk = div_up(p.mp, 64) * div_up(g.rows, kPrepRows);
    return r;
}

// Workgroups of the two passes: on U (with_u), on O and on T's padding.
void scale_blocks(F16Scale& g, bool with_u) {
    g.u_blocks = with_u ? g.n_ublk : 0;
    g.o_blocks = g.nb * div_up(g.m, kPrepORows);
}
int split_blocks(F16Scale& g, bool with_u) {
    const int tb = div_up(g.m, 64);
    g.u_blocks = with_u ? (g.Up ? 2 : 1) * div_up(g.mp, 64) * div_up(g.m, kSlabK) : 0;
    g.o_blocks = g.nb * tb * tb;
    return g.u_blocks + g.o_blocks + (g.rows % kSlabK ? g.nb * div_up((int64_t)g.mp * 2, 256) : 0);
}

// Stage 1, transposed: C(beta*d + s, i) = sum_j U1(beta*d + s, j) O_b(i, j).
FlatDesc f16_stage1(const F16Scale& g) {
    FlatDesc a{};
    a.M = g.d * g.mp;
    a.N = g.m;
    a.K = g.m;
    a.batch = g.nb;
    a.a_hi = g.u1h;
    a.a_lo = g.u1l;
    a.b_hi = g.oh;
    a.b_lo = g.ol;
    a.b_bs = g.o_bs;
    a.n32 = g.m32;
    a.t_hi = g.th;
    a.t_lo = g.tl;
    a.d = g.d;
    a.t_rows = g.mp32;
    a.t_bs = g.t_bs;
    a.t_e = g.et;
    a.skip = g.skip;
    a.any = g.any;
    a.u = g.u;
    // both halves of a site's split count
    const int column = std::min(kPairColumn, std::max(kPairShortColumn, g.rows / 4 * 3));
    a.u_least = (uint32_t)((int64_t)column * g.mp * (g.Up ? 2 : 1));
    a.parts = 1;
    a.part_slabs = (int)n_slabs(a.K);
    return a;
}

// Stage 2: out_b = U2 T_b^T.
FlatDesc f16_stage2(const F16Scale& g, float* c, int64_t ldc, int64_t c_bs) {
    FlatDesc b{};
    b.M = g.mp;
    b.N = g.mp;
    b.K = g.rows;
    b.batch = g.nb;
    b.a_hi = g.u2h;
    b.a_lo = g.u2l;
    b.b_hi = g.th;
    b.b_lo = g.tl;
    b.b_bs = g.t_bs;
    b.n32 = g.mp32;
    b.c = c;
    b.ldc = ldc;
    b.c_bs = c_bs;
    b.op_e = g.eo;
    b.row_e = g.eu;
    b.col_e = g.eu;
    b.skip = g.skip;
    b.any = g.any;
    b.parts = 1;
    b.part_slabs = (int)n_slabs(b.K);
    return b;
}

// Tiles of many products, longest first.  Each product takes the tallest
// tiles that stay below a time limit; the limit is the one whose tiles,
// handed out in this order to 256 CUs, end first by the estimate of flat_cfg
// (a step's 16 groups of 128 to 1024 states: the 1024-state tiles of stage 2
// alone last as long as the mean CU's share).
struct FlatProduct {
    int M, blocks, slabs;
};
std::vector<FlatTile> flat_list(const std::vector<FlatProduct>& prods) {
    struct Run {
        double t;
        int piece, bi, m0, rows, cols;  // rows of tiles from m0 on, 64 bi each
    };
    auto tile_us = [](int bi, int slabs) { return kFlatCost[bi] * slabs + kFlatAround; };
    std::vector<double> limits;
    for (const FlatProduct& p : prods)
        for (int bi = 1; bi <= 4; bi++) limits.push_back(tile_us(bi, p.slabs));
    std::sort(limits.begin(), limits.end(), std::greater<double>());
    limits.erase(std::unique(limits.begin(), limits.end()), limits.end());
    if (limits.size() > 32) limits.resize(32);
    auto runs_for = [&](double limit) {
        std::vector<Run> runs;
        for (int i = 0; i < (int)prods.size(); i++) {
            const FlatProduct& p = prods[i];
            int bi = 4;
            while (bi > 1 && (tile_us(bi, p.slabs) > limit || 64 * (bi - 1) >= p.M)) bi--;
            const int full = p.M / (64 * bi), rest = div_up(p.M - full * 64 * bi, 64), cols = div_up(p.blocks, 8);
            if (full) runs.push_back({tile_us(bi, p.slabs), i, bi, 0, full, cols});
            if (rest) runs.push_back({tile_us(rest, p.slabs), i, rest, full * 64 * bi, 1, cols});
        }
        std::stable_sort(runs.begin(), runs.end(), [](const Run& a, const Run& b) { return a.t > b.t; });
        return runs;
    };
    std::vector<Run> best;
    double best_t = 1e300;
    for (double limit : limits) {
        std::vector<Run> runs = runs_for(limit);
        std::priority_queue<double, std::vector<double>, std::greater<double>> cu(std::greater<double>(),
                                                                                  std::vector<double>(256, 0.0));
        double end = 0, all = 0;  // latest CU, whole rounds given to every CU
        for (const Run& r : runs) {
            const int64_t n = (int64_t)r.rows * r.cols, rounds = std::max<int64_t>(0, n / 256 - 1);
            all += rounds * r.t;
            for (int64_t x = rounds * 256; x < n; x++) {
                const double t = cu.top() + r.t;
                cu.pop();
                cu.push(t);
                end = std::max(end, t);
            }
        }
        end += all;
        if (end < best_t * 0.97) {
            best_t = end;
            best = std::move(runs);
        }
    }
    // Inside a run (alike tiles), M tiles fastest, in one stretch per XCD:
    // workgroup w runs on XCD w % 8, and neighbours share panels in its L2.
    std::vector<FlatTile> list;
    for (const Run& r : best) {
        const int n = r.rows * r.cols, w0 = (int)list.size();
        list.resize(w0 + n);
        int x = 0;
        for (int xcd = 0; xcd < 8; xcd++)
            for (int w = (xcd - w0 % 8 + 8) % 8; w < n; w += 8, x++)
                list[w0 + w] = {r.piece, r.m0 + (x % r.rows) * 64 * r.bi, x / r.rows, r.bi};
    }
    return list;
}

}  // namespace

// Whether `ops` operators of a group can run on FP16 pairs together: below 64
// states the tiles are mostly padding; U's split takes d up to 8; 32-bit
// offsets bound the operand arrays.
bool f16_shape_supported(const rot_problem& p, int ops) {
    if (p.d > kF16MaxSite || p.m < 64 || p.mp < 64) return false;
    const F16Layout L = f16_layout(p);
    if (std::max(L.u1, L.u2) >= ((size_t)1 << 31) - 256 * kSlabK * 2) return false;
    return std::max(L.o_op, L.t_op) * ops < (size_t)1 << 31;
}

// Whether a group runs on FP16 pairs, `ops` operators at a time.  The passes
// over U and O and the launches for skipped operators cost about 30 us, which
// pays from about 4 GFLOP on (back to back, FP32 kernels against pairs: 80
// operators of 128 states, 2.7 GFLOP, 52 / 52 us, 200 of them 97 / 78; 3 of
// 403, 3.0 GFLOP, 59 / 59; 2 of 512, 4.3 GFLOP, 56 / 56, 4 of them 94 / 75).
bool f16_rotate_applies(const rot_problem& p, int ops) {
    return f16_shape_supported(p, ops) && 2.0 * p.m * p.d * p.mp * ((double)p.m + p.mp) * p.n_ops >= kPairsLeastFlop;
}

size_t f16_group_workspace(const rot_problem& p, int ops, bool symmetric) {
    const F16Layout L = f16_layout(p);
    const int parts = f16_stage2_cfg(p, ops, symmetric).parts;
    return L.shared + f16_t_bytes(L, ops) + f16_o_bytes(p, L, ops, parts) + f16_scale_bytes(p, ops);
}

namespace {
// The passes and both stages of operators b0 .. b0 + nb - 1 of p, bound in r.
hipError_t run_pairs(const rot_problem& p, const F16Bound& r, int b0, int nb, bool with_u, bool symmetric,
                     const FlatCfg& c2, hipStream_t stream) {
    const F16Scale& g = r.g;
    const bool site = g.Up != nullptr;
    const dim3 block(256);
    hipError_t e = prof_timed("scale_f16x3", stream, [&] {
        F16Scale q = g;
        scale_blocks(q, with_u);
        const dim3 grid((unsigned)(q.u_blocks + q.o_blocks));
        if (site)
            hipLaunchKernelGGL(f16_scale_kernel<true>, grid, block, 0, stream, q);
        else
            hipLaunchKernelGGL(f16_scale_kernel<false>, grid, block, 0, stream, q);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    e = prof_timed("split_f16x3", stream, [&] {
        F16Scale q = g;
        const dim3 grid((unsigned)split_blocks(q, with_u));
        if (site && p.d <= 4)
            hipLaunchKernelGGL((f16_split_kernel<4, true>), grid, block, 0, stream, q);
        else if (site)
            hipLaunchKernelGGL((f16_split_kernel<kF16MaxSite, true>), grid, block, 0, stream, q);
        else if (p.d <= 4)
            hipLaunchKernelGGL((f16_split_kernel<4, false>), grid, block, 0, stream, q);
        else
            hipLaunchKernelGGL((f16_split_kernel<kF16MaxSite, false>), grid, block, 0, stream, q);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    const FlatDesc a = f16_stage1(g);
    const FlatCfg c1 = flat_cfg(a.M, nb * (g.m32 / 32), (int)n_slabs(p.m), 1, 1, 0);
    e = prof_timed("stage1_f16x3", stream, [&] {
        return p.d == 4   ? launch_flat<true, 4>(a, c1, stream)
               : p.d == 2 ? launch_flat<true, 2>(a, c1, stream)
                          : launch_flat<true, 0>(a, c1, stream);
    });
    if (e != hipSuccess) return e;
    float* out = static_cast<float*>(p.out) + (int64_t)b0 * p.stride_out;
    FlatDesc b = c2.parts > 1 ? f16_stage2(g, reinterpret_cast<float*>(r.O), p.mp, (int64_t)p.mp * p.mp)
                              : f16_stage2(g, out, p.ldout, p.stride_out);
    if (g.Up) b.row_e = g.eu2;
    b.c_ps = (int64_t)nb * p.mp * p.mp;
    b.upper = symmetric;
    e = prof_timed(symmetric ? "stage2sym_f16x3" : "stage2_f16x3", stream,
                   [&] { return launch_flat<false, 0>(b, c2, stream); });
    if (e == hipSuccess && c2.parts > 1)
        e = prof_timed("stage2_sum", stream, [&] {
            return sum_parts_2d(out, p.ldout, p.stride_out, r.O, p.mp, p.mp, nb, c2.parts, b.c_ps, false, stream);
        });
    if (e != hipSuccess) return e;
    return hipSuccess;
}

// Operators b0 .. of a site group: the flags, then the pairs and, over them,
// the FP32 kernels' intermediates.
F16Bound f16_site_bind(const rot_problem& p, const F16Site& x, const F16Layout& L, int b0, int nb, int parts,
                       void* ws, char** T32) {
    char* base = static_cast<char*>(ws);
    int* skip = reinterpret_cast<int*>(base);
    base += al256((size_t)(nb + 1) * 4);
    *T32 = base;
    F16Scale extra{};
    extra.upart2 = reinterpret_cast<uint32_t*>(base);
    base += L.part_u;
    extra.eu2 = reinterpret_cast<int*>(base);
    base += L.eu;
    F16Bound r = f16_bind(p, L, b0, nb, parts, base);
    r.g.skip = skip;
    r.g.any = skip + nb;
    r.g.Up = x.Up;
    r.g.d_all = x.d_all;
    r.g.sel = x.sel;
    r.g.upart2 = extra.upart2;
    r.g.eu2 = extra.eu2;
    r.g.n_ublk = 2 * div_up(p.mp, 64) * div_up((int64_t)p.m * x.d_all, kPrepRows);
    return r;
}
}  // namespace

// Operators b0 .. b0 + nb - 1 of p (leading dimensions resolved) through FP16
// pairs; `fallback` enqueues the FP32 kernels for the operators they skip
// (T: FP32 intermediates, slot_elems apart; skip: their flags, and behind them
// one that is set if any is).
hipError_t rotate_f16(const rot_problem& p, int b0, int nb, void* ws, bool symmetric,
                      const std::function<hipError_t(void* T, int64_t slot_elems, const int* skip)>& fallback,
                      hipStream_t stream) {
    const F16Layout L = f16_layout(p);
    const FlatCfg c2 = f16_stage2_cfg(p, nb, symmetric);
    const F16Bound r = f16_bind(p, L, b0, nb, c2.parts, ws);
    const hipError_t e = run_pairs(p, r, b0, nb, b0 == 0, symmetric, c2, stream);
    return e == hipSuccess ? fallback(r.T, (int64_t)(L.t32 / 4), r.g.skip) : e;
}

// Block operators times a site operator, out_b = U'^T (X_b U_r): stage 2's A
// is the mixed Up instead of U, and only the site states t that Up has rows
// for (S's non-zero columns; p.d of them, x.sel) enter either stage.  An
// annihilator has two of the Hubbard site's four: half the products.  33
// operators of 500 states, kept 480: 635 us for all four on the FP32 kernels,
// 172 us for two on pairs (stage 1 78, stage 2 57, the passes 29).
size_t f16_site_workspace(const rot_problem& p, const F16Site& x, int ops) {
    const F16Layout L = f16_layout(p, x.d_all);
    const int parts = f16_stage2_cfg(p, ops, false).parts;
    return al256((size_t)(ops + 1) * 4) + std::max(L.shared + 2 * al256(ops * L.t_op) + f16_o_bytes(p, L, ops, parts) +
                                                 f16_scale_bytes(p, ops),
                                             ops * L.t32);
}
hipError_t rotate_f16_site(const rot_problem& p, const F16Site& x, int b0, int nb, void* ws,
                           const std::function<hipError_t(void* T, int64_t slot_elems, const int* skip)>& fallback,
                           hipStream_t stream) {
    F16Layout L = f16_layout(p, x.d_all);
    const int64_t t32 = (int64_t)(L.t32 / 4);
    L.t32 = 0;  // laid over everything instead of beside T's pairs
    const FlatCfg c2 = f16_stage2_cfg(p, nb, false);
    char* T32;
    const F16Bound r = f16_site_bind(p, x, L, b0, nb, c2.parts, ws, &T32);
    const hipError_t e = run_pairs(p, r, b0, nb, true, false, c2, stream);
    return e == hipSuccess ? fallback(T32, t32, r.g.skip) : e;
}

// ------------------------------------------------------------------ plans --
// A chunk of a plan: operators of several groups ("pieces") through one
// launch per pass and stage, from tables and lists in device memory.  Stage 2
// is not split over K: the plan's FP32 kernels do not either, and the tiles
// of all groups together fill the chip.  One execution, FP32 kernels before
// -> pairs (rate of the products in brackets, TFLOP/s): 16 groups of 128 to
// 1024 states, 8 operators each, 230 GFLOP, 2427 -> 738 us (95 -> 312); 8 of
// 1000 states 1372 -> 397 us; 50 GFLOP in 7 groups of 101 to 900 states, 3
// operators each, 826 -> 229 us.

size_t pair_piece_workspace(const rot_problem& p, int ops) {
    const F16Layout L = f16_layout(p);
    return L.shared + f16_t_bytes(L, ops) + f16_o_bytes(p, L, ops, 1) + f16_scale_bytes(p, ops);
}

// The FP32 kernels' flag and intermediate of operator b0 + k of a piece.
void pair_fallback(const rot_problem& p, const PairPiece& x, int k, const int** only, const float** T) {
    const F16Layout L = f16_layout(p);
    const F16Bound r = f16_bind(p, L, x.b0, x.nb, 1, x.ws);
    *only = r.g.skip + k;
    *T = reinterpret_cast<const float*>(r.T + k * L.t32);
}

namespace {
struct PairTables {
    F16Scale *scale, *split;
    FlatDesc *s1, *s2;
};
PairTables pair_tables_at(void* mem, int n) {
    PairTables t;
    t.s1 = static_cast<FlatDesc*>(mem);
    t.s2 = t.s1 + n;
    t.scale = reinterpret_cast<F16Scale*>(t.s2 + n);
    t.split = t.scale + n;
    return t;
}
static_assert(sizeof(FlatDesc) % 8 == 0 && sizeof(F16Scale) % 8 == 0, "table alignment");
}  // namespace

size_t pair_table_bytes(int n) { return (size_t)n * 2 * (sizeof(F16Scale) + sizeof(FlatDesc)); }

// The tables of a chunk's pieces (host memory of pair_table_bytes); `any` is
// the chunk's device flag.
void pair_fill_tables(const rot_problem* groups, const std::vector<PairPiece>& pieces, int* any, void* mem) {
    const PairTables t = pair_tables_at(mem, (int)pieces.size());
    for (size_t i = 0; i < pieces.size(); i++) {
        const PairPiece& x = pieces[i];
        const rot_problem& p = groups[x.group];
        F16Scale g = f16_bind(p, f16_layout(p), x.b0, x.nb, 1, x.ws).g;
        g.any = any;
        t.s1[i] = f16_stage1(g);
        t.s2[i] = f16_stage2(g, static_cast<float*>(p.out) + (int64_t)x.b0 * p.stride_out, p.ldout, p.stride_out);
        scale_blocks(g, true);
        t.scale[i] = g;
        split_blocks(g, true);
        t.split[i] = g;
    }
}

// Lists of a chunk, and one device allocation for the tables (first), the
// lists and the flag.
hipError_t pair_build(const rot_problem* groups, const std::vector<PairPiece>& pieces, PairChunk* c) {
    const int n = (int)pieces.size();
    std::vector<char> host(pair_table_bytes(n));
    pair_fill_tables(groups, pieces, nullptr, host.data());
    const PairTables t = pair_tables_at(host.data(), n);
    std::vector<PairBlock> scale, split;
    std::vector<FlatProduct> p1, p2;
    c->n_pieces = n;
    c->d_max = 0;
    c->same_d = groups[pieces[0].group].d;
    for (int i = 0; i < n; i++) {
        const F16Scale& a = t.scale[i];
        for (int x = 0; x < a.u_blocks + a.o_blocks; x++) scale.push_back({i, x});
        F16Scale b = t.split[i];
        const int nb = split_blocks(b, true);
        for (int x = 0; x < nb; x++) split.push_back({i, x});
        p1.push_back({t.s1[i].M, t.s1[i].batch * (t.s1[i].n32 / 32), (int)n_slabs(t.s1[i].K)});
        p2.push_back({t.s2[i].M, t.s2[i].batch * (t.s2[i].n32 / 32), (int)n_slabs(t.s2[i].K)});
        c->d_max = std::max(c->d_max, a.d);
        if (a.d != c->same_d) c->same_d = 0;
    }
    const std::vector<FlatTile> l1 = flat_list(p1), l2 = flat_list(p2);
    const size_t bytes[6] = {al256(host.size()), al256(scale.size() * sizeof(PairBlock)),
                             al256(split.size() * sizeof(PairBlock)), al256(l1.size() * sizeof(FlatTile)),
                             al256(l2.size() * sizeof(FlatTile)), 256};
    size_t total = 0;
    for (size_t x : bytes) total += x;
    hipError_t e = hipMalloc(&c->mem, total);
    if (e != hipSuccess) return e;
    char* at = static_cast<char*>(c->mem);
    c->scale = at += bytes[0];
    c->split = at += bytes[1];
    c->tiles1 = at += bytes[2];
    c->tiles2 = at += bytes[3];
    c->any = reinterpret_cast<int*>(at += bytes[4]);
    c->n_scale = (int)scale.size();
    c->n_split = (int)split.size();
    c->n_tiles1 = (int)l1.size();
    c->n_tiles2 = (int)l2.size();
    pair_fill_tables(groups, pieces, c->any, host.data());
    auto up = [&](void* dst, const void* src, size_t b) {
        if (e == hipSuccess) e = hipMemcpy(dst, src, b, hipMemcpyHostToDevice);
    };
    up(c->mem, host.data(), host.size());
    up(c->scale, scale.data(), scale.size() * sizeof(PairBlock));
    up(c->split, split.data(), split.size() * sizeof(PairBlock));
    up(c->tiles1, l1.data(), l1.size() * sizeof(FlatTile));
    up(c->tiles2, l2.data(), l2.size() * sizeof(FlatTile));
    return e;
}

// Enqueue a chunk's passes and stages; `timed` files each under the profiler.
hipError_t pair_issue(const PairChunk& c, hipStream_t s, bool timed) {
    const PairTables t = pair_tables_at(c.mem, c.n_pieces);
    auto run = [&](const char* name, const std::function<void()>& launch) {
        auto f = [&] {
            launch();
            return hipGetLastError();
        };
        return timed ? prof_timed(name, s, f) : f();
    };
    hipError_t e = run("scale_f16x3", [&] {
        hipLaunchKernelGGL(f16_scale_list_kernel, dim3((unsigned)c.n_scale), dim3(256), 0, s, t.scale,
                           static_cast<const PairBlock*>(c.scale), c.any);
    });
    if (e != hipSuccess) return e;
    e = run("split_f16x3", [&] {
        const dim3 grid((unsigned)c.n_split), block(256);
        const PairBlock* list = static_cast<const PairBlock*>(c.split);
        if (c.d_max <= 4)
            hipLaunchKernelGGL(f16_split_list_kernel<4>, grid, block, 0, s, t.split, list);
        else
            hipLaunchKernelGGL(f16_split_list_kernel<kF16MaxSite>, grid, block, 0, s, t.split, list);
    });
    if (e != hipSuccess) return e;
    e = run("plan_stage1_f16x3", [&] {
        const dim3 grid((unsigned)c.n_tiles1), block(512);
        const FlatTile* list = static_cast<const FlatTile*>(c.tiles1);
        if (c.same_d == 4)
            hipLaunchKernelGGL((gemm_flat_list_kernel<true, 4>), grid, block, 0, s, t.s1, list);
        else if (c.same_d == 2)
            hipLaunchKernelGGL((gemm_flat_list_kernel<true, 2>), grid, block, 0, s, t.s1, list);
        else
            hipLaunchKernelGGL((gemm_flat_list_kernel<true, 0>), grid, block, 0, s, t.s1, list);
    });
    if (e != hipSuccess) return e;
    return run("plan_stage2_f16x3", [&] {
        hipLaunchKernelGGL((gemm_flat_list_kernel<false, 0>), dim3((unsigned)c.n_tiles2), dim3(512), 0, s, t.s2,
                           static_cast<const FlatTile*>(c.tiles2));
    });
}

}  // namespace rot
