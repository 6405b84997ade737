// The system's reduced density matrix per quantum-number sector, its
// eigenbasis, and the choice of the kept states (Sec. 2: Eq. (2), step 4,
// Eq. (3)), all in FP64.
//
// rho_k = psi_k psi_k^T is formed tile by tile into a zero-padded n_pad x n_pad
// matrix (n_pad a multiple of 64) and diagonalised by two-sided block Jacobi:
// the matrix is cut into 32-wide blocks; in each round the blocks are paired
// by the circle method and every pair's 64 x 64 principal submatrix is swept
// once by scalar Jacobi in LDS (one workgroup per pair, the 32 disjoint rotations
// of a step applied together): all its index pairs in the first round of a
// sweep, those between its two blocks in the others.
//
// A round is one launch.  A pair's workgroup first brings its own 32 x 32 block
// between the two blocks up to date with the rotations of the round before
// (Q1^T X Q2 of the last full matrix) and then sweeps; beside it, on the CUs
// that the few pairs leave idle, the last round's rotations are applied to the
// whole matrix (into a second copy) and to the eigenvectors (V_{:,P} <- V_{:,P}
// Q), so neither is on the path from round to round.  Everything a round leaves
// behind alternates between two buffers.  Padded rows and columns are exactly
// zero and never rotate, so they stay decoupled.  A sector is finished after a
// full cycle of rounds without any rotation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "rot_internal.h"

namespace rot {

namespace {

constexpr int kBlk = 32;        // Jacobi block edge
constexpr int kPair = 64;       // two blocks
constexpr int kLs = kPair + 1;  // LDS row stride (doubles)
constexpr int kMaxSweeps = 80;
constexpr int kFirstCheck = 6, kCheckEvery = 3;  // sweeps after which the host asks whether all sectors are done
constexpr int kSortMax = 4096;  // largest sector (states)

struct DmSector {
    int n, r, npad, nb;
    const double* psi;
    int64_t ld_psi;
    double* w;
    double* V;
    int64_t ld_v;
    int64_t a_off;   // doubles, into a copy of the working matrix and the eigenvector matrix
    int64_t q_off;   // doubles, into a round's pair submatrices or rotations (nb/2 blocks of 64 x 64)
    int64_t w_off;   // doubles, into the concatenated sorted eigenvalues
    int64_t d_off;   // doubles, into the diagonals
    int flag_off;    // ints, into a round's per-pair rotation flags
    int pad;
};

struct DmState {
    double floor;  // |a_pq| <= floor of the scaled rho counts as zero
    int quiet[2];  // consecutive rounds without a rotation, before the last one of each parity
    int exponent;  // rho is swept scaled by 2^-exponent (trace in [1, 2))
    int pad;
};

struct DmItem {
    int sec, a, b, kind;
};

enum : int { kItemPair = 0, kItemA = 1, kItemV = 2 };

// The buffers of one call; index 1 of a pair starts `..._round` elements on.
struct DmBuffers {
    double *A, *V, *S, *Q, *diag;
    DmState* st;
    int* flags;
    int64_t a_round, q_round;
    int f_round;
};

// Round t of the circle method for nb players (nb even): player 0 is fixed,
// players 1..nb-1 sit on a circle turned by t; pair k is (0, c_0) for k = 0
// and (c_k, c_{nb-1-k}) otherwise, with c_j = 1 + (j + t) mod (nb - 1).  Over
// nb - 1 consecutive rounds every two players meet once.  Returns i < j.
__host__ __device__ inline void circle_pair(int nb, int t, int k, int& i, int& j) {
    const int m = nb - 1;
    t %= m;
    int a, b;
    if (k == 0) {
        a = 0;
        b = 1 + t;
    } else {
        a = 1 + (k + t) % m;
        b = 1 + (m - k + t) % m;
    }
    i = a < b ? a : b;
    j = a < b ? b : a;
}

// Pair (and which half of it, 0 or 1) that holds block b in round t.
__device__ inline void circle_where(int nb, int t, int b, int& k, int& half) {
    const int m = nb - 1;
    if (b == 0) {
        k = half = 0;
        return;
    }
    int j = b - 1 - t;
    if (j < 0) j += m;
    k = j <= m / 2 ? j : m - j;
    int i0, i1;
    circle_pair(nb, t, k, i0, i1);
    half = b == i1;
}

// Global row of local index l (0..63) of the pair of blocks (I, J).
__device__ inline int pair_row(int I, int J, int l) { return l < kBlk ? I * kBlk + l : J * kBlk + (l - kBlk); }

// ---------------------------------------------------------------------------
// rho tile (ti, tj), ti <= tj, of sector it.sec: rho[x][y] = sum_k psi[x][k] psi[y][k]
// over 64 x 64 outputs, one 32 x 32 quarter per wave on v_mfma_f64_16x16x4f64
// (lane l: A(l%16, l/16), B(l/16, l%16); element v of the result is row
// 4 v + l/16, column l%16); written to both (ti, tj) and its mirror.  The
// eigenvector matrix is set to the identity on the same tiles.  K in slices of
// 16 through two LDS buffers, the next slice in registers: with one workgroup
// per CU the loads' latency is the bound (60 sectors of up to 246 states: one
// buffer and vector arithmetic 80 us, now 25).
__global__ __launch_bounds__(256) void dm_rho_kernel(const DmSector* __restrict__ secs,
                                                     const DmItem* __restrict__ items, double* __restrict__ A,
                                                     double* __restrict__ Vw) {
    const DmItem it = items[blockIdx.x];
    const DmSector s = secs[it.sec];
    const int ti = it.a, tj = it.b;
    constexpr int kRow = 18;  // LDS row of a slice (doubles): 16 rows' reads spread over the banks
    __shared__ double pa[2][kPair * kRow], pb[2][kPair * kRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 4, c = lane & 15;
    const int wr = 32 * (wave >> 1), wc = 32 * (wave & 1);
    const int kk = tid & 15, row = tid >> 4;
    double va[4], vb[4];
    auto load = [&](int k0) {
        const int gk = k0 + kk;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int gi = ti * kPair + row + 16 * j, gj = tj * kPair + row + 16 * j;
            va[j] = (gk < s.r && gi < s.n) ? s.psi[(int64_t)gi * s.ld_psi + gk] : 0.0;
            vb[j] = (gk < s.r && gj < s.n) ? s.psi[(int64_t)gj * s.ld_psi + gk] : 0.0;
        }
    };
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    f64x4 acc[2][2];
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int q = 0; q < 2; q++) acc[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
    load(0);
    for (int k0 = 0, cur = 0; k0 < s.r; k0 += 16, cur ^= 1) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            pa[cur][(row + 16 * j) * kRow + kk] = va[j];
            pb[cur][(row + 16 * j) * kRow + kk] = vb[j];
        }
        __syncthreads();
        if (k0 + 16 < s.r) load(k0 + 16);
#pragma unroll
        for (int k4 = 0; k4 < 16; k4 += 4) {
            double x[2], y[2];
#pragma unroll
            for (int p = 0; p < 2; p++) {
                x[p] = pa[cur][(wr + 16 * p + c) * kRow + k4 + h];
                y[p] = pb[cur][(wc + 16 * p + c) * kRow + k4 + h];
            }
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int q = 0; q < 2; q++) acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[p], y[q], acc[p][q], 0, 0, 0);
        }
    }
    double* a = A + s.a_off;
    double* v = Vw + s.a_off;
    const int64_t np = s.npad;
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int q = 0; q < 2; q++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int64_t r0 = ti * kPair + wr + 16 * p + 4 * e + h, c0 = tj * kPair + wc + 16 * q + c;
                a[r0 * np + c0] = acc[p][q][e];
                v[r0 * np + c0] = r0 == c0 ? 1.0 : 0.0;
                if (ti != tj) {
                    a[c0 * np + r0] = acc[p][q][e];
                    v[c0 * np + r0] = 0.0;
                }
            }
}

// Per sector: the threshold 2^-52 tr(rho) (trace summed in a fixed order) and
// cleared convergence counters.
__global__ __launch_bounds__(256) void dm_prep_kernel(const DmSector* __restrict__ secs,
                                                      const double* __restrict__ A, DmState* __restrict__ st) {
    const DmSector s = secs[blockIdx.x];
    __shared__ double red[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < s.n; i += 256) acc += A[s.a_off + (int64_t)i * s.npad + i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        DmState x;
        x.exponent = red[0] > 0.0 && red[0] < INFINITY ? ilogb(red[0]) : 0;
        x.floor = ldexp(red[0], -52 - x.exponent);
        x.quiet[0] = x.quiet[1] = 0;
        x.pad = 0;
        st[blockIdx.x] = x;
    }
}

// ---------------------------------------------------------------------------
// One Jacobi sweep over the 64 x 64 principal submatrix S of a pair of blocks,
// in steps of 32 disjoint rotations.  The 64 indices sit in 32 slots of a top
// and a bottom one; a step rotates every slot's pair, then the indices move to
// the next step's slots:
//   full sweep (63 steps, circle order): top of slot 0 stays, the other 63
//     indices turn one place: top k <- top k+1, top 31 <- bottom 31,
//     bottom 0 <- top 1, bottom k <- bottom k-1;
//   cross sweep (32 steps, the pairs between the two blocks): tops stay,
//     bottom k <- bottom k+1 cyclically.
// Both return every index to its first slot at the end.
//
// Rotation (p, q) zeroes a_pq of J^T S J, J = [[c, s], [-s, c]] on rows and
// columns (p, q): with d = a_qq - a_pp, t = s / c = 2 a_pq / (d + sign(d)
// sqrt(d^2 + 4 a_pq^2)) (|t| <= 1).
//
// A full step is bound by its chain of LDS round trips and dependent FP64
// operations, so it has one barrier: each of the 496 two-slot blocks is
// rotated by one thread, and the 32 blocks that hold the next step's a_pq
// belong to the lanes of one wave, which go on from the updated entry to the
// next rotation (the diagonal lives apart, double-buffered, written by those
// lanes only).  S is held as its upper triangle.  A cross step holds S in
// registers (dm_sweep_cross).  The accumulated Q never touches the LDS: four
// waves hold 8 slots of every row each in registers and hand one value per
// neighbour and step on.
// Time of a step, and of 60 sectors of up to 246 states (4 096 in all, 13
// sweeps): two barriers and Q in the LDS 1.1 us, 7.1 ms; one barrier, Q in
// registers 0.5 us, 3.5 ms; cross steps in registers and short rotation chains
// 0.37 us (cross) and 0.6 us (full), 2.7 ms.  A cross step is now bound by the
// issue of FP64 instructions (890 cycles; 560 for the wave of the rotations
// alone, 700 without the other waves of S, 770 without those of Q); a round's
// other 13 us are the launch, the loads and two 64-deep products before the
// sweep and the stores after it.
constexpr int kQWaves = 4;
constexpr int kSWaves = 9;
constexpr int kPairThreads = 64 * (kQWaves + kSWaves);
constexpr int kParamWave = 7;   // shares its SIMD with the fewest others
constexpr int kCross = 32;      // steps
constexpr int kFull = kPair - 1;

struct DmBlocks {
    // blocks (kx, ky), kx <= ky, by thread of the 8 plain S waves, then those of
    // the next step's pairs by lane, for a full sweep; 255: none.  entry: which
    // of (top, top), (top, bottom), (bottom, top), (bottom, bottom) of (kx, ky)
    // is the next pair's a_pq.
    unsigned char x[512], y[512], nx[32], ny[32], entry[32];
};

constexpr DmBlocks dm_blocks() {
    DmBlocks b{};
    for (int k = 0; k < 32; k++) {
        // (top 0, top 1); (top 2, bottom 0); (top k+1, bottom k-1); (bottom 31, bottom 30)
        b.nx[k] = (unsigned char)(k == 0 ? 0 : k == 31 ? 30 : k - 1);
        b.ny[k] = (unsigned char)(k == 0 ? 1 : k == 31 ? 31 : k + 1);
        b.entry[k] = (unsigned char)(k == 0 ? 0 : k == 31 ? 3 : 2);
    }
    int n = 0;
    for (int ky = 0; ky < 32; ky++)
        for (int kx = 0; kx <= ky; kx++) {
            bool next = false;
            for (int k = 0; k < 32; k++) next = next || (b.nx[k] == kx && b.ny[k] == ky);
            if (next) continue;
            b.x[n] = (unsigned char)kx;
            b.y[n] = (unsigned char)ky;
            n++;
        }
    for (; n < 512; n++) b.x[n] = b.y[n] = 255;
    return b;
}

__constant__ DmBlocks kDmBlocks = dm_blocks();

// Index in the top (bottom) of slot k at step u.
__device__ inline int slot_index(bool full, int k, bool bottom, int u) {
    if (!full) return bottom ? 32 + ((k + u) & 31) : k;
    if (k == 0 && !bottom) return 0;
    const int j = (bottom ? (k == 0 ? 0 : 63 - k) : k) + u;
    return 1 + (j >= 63 ? j - 63 : j);
}

__device__ inline int su(unsigned a, unsigned b) { return (int)(__umul24(min(a, b), kLs) + max(a, b)); }

struct DmRot {
    double c, s;
};

// The rotation that zeroes apq, the diagonal entries after it and what is left
// of apq.  Only c^2 + s^2 = 1 has to hold to the last bit: t comes from single
// precision (apq and the diagonal's difference are above 2^-52 of a trace in
// [1, 2), or do not matter) and c = 1 / sqrt(1 + t^2) from that very t in
// double, by one third-order step from a single-precision start (an error of
// 2^-22 becomes 2^-66); the 2^-23 of apq that t's rounding leaves behind is
// kept, not dropped.  The chain through the next pair's entry sets the time of
// a step: 25 dependent FP64 operations with exact t, 9 so.
__device__ inline DmRot dm_rotation(double& app, double& aqq, double apq, double floor, double& left) {
    const double d = aqq - app;
    const float df = (float)d, af = (float)apq;
    const float den = fabsf(df) + __builtin_amdgcn_sqrtf(fmaf(df, df, 4.0f * af * af));
    const float tf = 2.0f * af * __builtin_amdgcn_rcpf(copysignf(den, df));
    const double t = (double)tf, x = fma(t, t, 1.0), y = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.0f));
    const double e = fma(-x, y * y, 1.0);
    const bool on = fabs(apq) > floor;
    DmRot r;
    r.c = on ? fma(y * e, fma(0.375, e, 0.5), y) : 1.0;
    r.s = on ? t * r.c : 0.0;
    const double g = fma(r.c, apq, -r.s * d), w = fma(r.c, apq, g);
    app = fma(-r.s, w, app);
    aqq = fma(r.s, w, aqq);
    left = fma(r.c, g, -r.s * r.s * apq);
    return r;
}

constexpr int kHalf = kBlk + 1;  // LDS row stride of 64 x 32 operands

struct DmPairLds {
    double S[kPair * kLs];                // before the sweep: X, then X Q2
    double L1[kPair * kHalf], R2[kPair * kHalf];  // Q1's and Q2's columns of the two blocks
    double2 rot[2][32];                   // (c, s) of a step's slots
    double D[2][kPair];                   // diagonal after a step's rotations, by index
    double hand[2][kQWaves][2][kPair];    // what the Q waves hand on, by row
    int any, work;
};

// The accumulated Q through a sweep: this wave's eight slots of row `lane`.
template <bool FULL>
__device__ __attribute__((always_inline)) inline void dm_sweep_q(DmPairLds& L, int wave, int lane, double (&qt)[8],
                                                                 double (&qb)[8]) {
    constexpr int NS = FULL ? kFull : kCross;
    for (int u = 0; u < NS; u++) {
        const int cur = u & 1;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const double2 r = L.rot[cur][8 * wave + j];
            const double a = qt[j], b = qb[j];
            qt[j] = fma(r.x, a, -r.y * b);
            qb[j] = fma(r.y, a, r.x * b);
        }
        // hand on to the neighbours, move the own ones
        L.hand[cur][wave][0][lane] = FULL ? qt[0] : qb[0];
        if (FULL) L.hand[cur][wave][1][lane] = qb[7];
        __syncthreads();
        const double up = L.hand[cur][(wave + 1) & 3][0][lane];
        if (FULL) {
            const double down = L.hand[cur][(wave + 3) & 3][1][lane];
            const double t0 = qt[0], t1 = qt[1], last = qb[7];
#pragma unroll
            for (int j = 0; j < 7; j++) qt[j] = qt[j + 1];
            qt[7] = wave == 3 ? last : up;
#pragma unroll
            for (int j = 7; j > 0; j--) qb[j] = qb[j - 1];
            qb[0] = down;
            if (wave == 0) {
                qt[0] = t0;
                qb[0] = t1;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 7; j++) qb[j] = qb[j + 1];
            qb[7] = up;
        }
    }
}

// Lane i's x from lane i + 1 (i - 1) of 64, cyclically.
template <int CTRL>
__device__ inline double dm_wave_rotate(double x) {
    const int64_t b = __builtin_bit_cast(int64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (int64_t)hi << 32 | lo);
}
__device__ inline double from_next(double x) { return dm_wave_rotate<0x134>(x); }
__device__ inline double from_prev(double x) { return dm_wave_rotate<0x13C>(x); }

// S through a cross sweep, in registers: the block between slots ky - m and ky
// (mod 32) is lane ky's, m = 1..16 spread two to a wave (lanes 32..63 repeat
// 0..31, which makes the wave's rotation one of 32; m = 16 holds every block
// twice, once transposed).  A step's moves of the bottoms then are: bottom x
// bottom to the lane before; top x bottom there too, from m + 1 to m; bottom x
// top from m to m + 1 in its lane.  Only what crosses from wave to wave goes
// through the LDS, one value each way.  The wave of m = 1, 2 sees every next
// a_pq first and goes on from its own rotations without the LDS.
struct DmCrossBlock {
    double tt, tb, bt, bb;
};
__device__ inline void dm_rotate_block(DmCrossBlock& x, double cx, double sx, double cy, double sy) {
    const double u1 = fma(cx, x.tt, -sx * x.bt), x1 = fma(sx, x.tt, cx * x.bt);
    const double v1 = fma(cx, x.tb, -sx * x.bb), y1 = fma(sx, x.tb, cx * x.bb);
    x.tt = fma(cy, u1, -sy * v1);
    x.tb = fma(sy, u1, cy * v1);
    x.bt = fma(cy, x1, -sy * y1);
    x.bb = fma(sy, x1, cy * y1);
}

constexpr int kCrossWaves = 8;

__device__ __attribute__((always_inline)) inline void dm_sweep_cross(DmPairLds& L, double floor, int wave, int lane) {
    const int w = wave == kParamWave ? 0 : wave < kParamWave ? wave - kQWaves + 1 : wave - kQWaves;
    if (w >= kCrossWaves) {
        for (int u = 0; u < kCross; u++) __syncthreads();
        return;
    }
    const int l = lane & 31, ma = 2 * w + 1, ka = (l - ma) & 31, kb = (l - ma - 1) & 31;
    // what waves hand on: bottom x top up to the next m, top x bottom down
    double(*up)[kCrossWaves][32] = reinterpret_cast<double(*)[kCrossWaves][32]>(L.L1);
    double(*down)[kCrossWaves][32] = reinterpret_cast<double(*)[kCrossWaves][32]>(L.R2);
    static_assert(2 * kCrossWaves * 32 <= kPair * kHalf, "handing on fits the operands' place");
    auto get = [&](int k) {
        return DmCrossBlock{L.S[su(k, l)], L.S[su(k, 32 + l)], L.S[su(32 + k, l)], L.S[su(32 + k, 32 + l)]};
    };
    DmCrossBlock a = get(ka), b = get(kb);
    if (w == 0) {
        __builtin_amdgcn_s_setprio(3);  // the step waits for this wave
        const double2 r0 = L.rot[0][l];
        double c = r0.x, sn = r0.y, app = L.D[0][l], aqq = L.D[0][32 + l];
        double left = L.S[su(l, 32 + l)], apq = 0.0;  // the pair's entry after its rotation, the next one's before
        for (int u = 0; u < kCross; u++) {
            const int cur = u & 1;
            const double c1 = from_prev(c), s1 = from_prev(sn), c2 = from_prev(c1), s2 = from_prev(s1);
            if (u) b.tb = down[cur][1][(l + 1) & 31];
            dm_rotate_block(a, c1, s1, c, sn);
            apq = from_next(a.tb);
            aqq = from_next(aqq);
            a.bb = from_next(a.bb);
            dm_rotate_block(b, c2, s2, c, sn);
            a.tb = from_next(b.tb);
            b.bb = from_next(b.bb);
            up[cur ^ 1][0][l] = b.bt;
            b.bt = a.bt;
            a.bt = left;
            if (u + 1 < kCross) {
                const DmRot r = dm_rotation(app, aqq, apq, floor, left);
                c = r.c;
                sn = r.s;
                L.rot[cur ^ 1][l] = double2{c, sn};
                if (sn != 0.0) L.any = 1;
            }
            __syncthreads();
        }
        b.tb = down[kCross & 1][1][(l + 1) & 31];
        __builtin_amdgcn_s_setprio(0);
        L.D[kCross & 1][l] = app;
        L.D[kCross & 1][32 + l] = aqq;
        L.S[su(l, 32 + l)] = apq;
    } else {
        const bool end = w == kCrossWaves - 1;
        const double* above = end ? &up[0][w][0] : &down[0][w + 1][0];
        const int at = end ? l ^ 16 : (l + 1) & 31;
        constexpr int kStep = kCrossWaves * 32;  // from one step's values to the other's
        for (int u = 0; u < kCross; u++) {
            const int cur = u & 1;
            const double2 ry = L.rot[cur][l], ra = L.rot[cur][ka], rb = L.rot[cur][kb];
            if (u) {
                a.bt = up[cur][w - 1][l];
                b.tb = above[cur * kStep + at];
            }
            dm_rotate_block(a, ra.x, ra.y, ry.x, ry.y);
            dm_rotate_block(b, rb.x, rb.y, ry.x, ry.y);
            // the end hands its own bottom x top over transposed
            up[cur ^ 1][w][l] = end ? a.bt : b.bt;
            down[cur ^ 1][w][l] = a.tb;
            a.bb = from_next(a.bb);
            a.tb = from_next(b.tb);
            b.bb = from_next(b.bb);
            b.bt = a.bt;
            __syncthreads();
        }
        a.bt = up[kCross & 1][w - 1][l];
        b.tb = above[(kCross & 1) * kStep + at];
    }
    auto put = [&](int k, const DmCrossBlock& x) {
        L.S[su(k, l)] = x.tt;
        L.S[su(k, 32 + l)] = x.tb;
        L.S[su(32 + k, l)] = x.bt;
        L.S[su(32 + k, 32 + l)] = x.bb;
    };
    if (lane < 32) {
        put(ka, a);
        if (w + 1 < kCrossWaves || l >= 16) put(kb, b);
    }
}

// S through a full sweep, in the LDS.
__device__ __attribute__((always_inline)) inline void dm_sweep_full(DmPairLds& L, double floor, int wave, int lane) {
    constexpr int NS = kFull;
    const bool param = wave == kParamWave;
    const int plain = (wave - kQWaves - (wave > kParamWave ? 1 : 0)) * 64 + lane;
    unsigned kx, ky, entry = 0;
    if (param) {
        kx = lane < 32 ? kDmBlocks.nx[lane] : 255;
        ky = lane < 32 ? kDmBlocks.ny[lane] : 255;
        entry = kDmBlocks.entry[lane & 31];
        __builtin_amdgcn_s_setprio(3);  // the step waits for this wave
    } else {
        kx = kDmBlocks.x[plain];
        ky = kDmBlocks.y[plain];
    }
    const bool live = kx < 32, diagonal = kx == ky;
    if (!live) kx = ky = 0;
    // this thread's indices, and (lanes of the next rotations) the next pair's,
    // carried from step to step
    unsigned px = slot_index(true, kx, false, 0), qx = slot_index(true, kx, true, 0);
    unsigned py = slot_index(true, ky, false, 0), qy = slot_index(true, ky, true, 0);
    unsigned p = slot_index(true, lane & 31, false, 1), q = slot_index(true, lane & 31, true, 1);
    auto advance = [](unsigned i) -> unsigned { return i == 0 ? 0 : i == 63 ? 1 : i + 1; };
    for (int u = 0; u < NS; u++) {
        const int cur = u & 1;
        if (live) {
            if (!diagonal) {
                const int iu = su(px, py), iv = su(px, qy), ix = su(qx, py), iy = su(qx, qy);
                const double2 rx = L.rot[cur][kx], ry = L.rot[cur][ky];
                double u0 = L.S[iu], v0 = L.S[iv], x0 = L.S[ix], y0 = L.S[iy];
                double app = 0.0, aqq = 0.0;
                if (param) {
                    app = L.D[cur][p];
                    aqq = L.D[cur][q];
                }
                if (rx.y != 0.0 || ry.y != 0.0) {
                    const double u1 = fma(rx.x, u0, -rx.y * x0), x1 = fma(rx.y, u0, rx.x * x0);
                    const double v1 = fma(rx.x, v0, -rx.y * y0), y1 = fma(rx.y, v0, rx.x * y0);
                    u0 = fma(ry.x, u1, -ry.y * v1);
                    v0 = fma(ry.y, u1, ry.x * v1);
                    x0 = fma(ry.x, x1, -ry.y * y1);
                    y0 = fma(ry.y, x1, ry.x * y1);
                    L.S[iu] = u0;
                    L.S[iv] = v0;
                    L.S[ix] = x0;
                    L.S[iy] = y0;
                }
                if (param) {
                    const double apq = entry & 2 ? (entry & 1 ? y0 : x0) : (entry & 1 ? v0 : u0);
                    DmRot r{1.0, 0.0};
                    if (u + 1 < NS) {
                        double left;
                        r = dm_rotation(app, aqq, apq, floor, left);
                        L.S[su(p, q)] = left;
                    }
                    L.rot[cur ^ 1][lane] = double2{r.c, r.s};
                    L.D[cur ^ 1][p] = app;
                    L.D[cur ^ 1][q] = aqq;
                    if (r.s != 0.0) L.any = 1;
                    p = advance(p);
                    q = advance(q);
                }
            }
            px = advance(px);
            qx = advance(qx);
            py = advance(py);
            qy = advance(qy);
        }
        __syncthreads();
    }
    if (param) __builtin_amdgcn_s_setprio(0);
}

typedef double dm_f64x4 __attribute__((ext_vector_type(4)));

// 16 x 16 block of op(L) R over K = 64 on v_mfma_f64_16x16x4f64, operands in LDS
// with row strides ls and rs: L at element (row, k) or, kTransL, (k, row).
// Lane l supplies A(row l%16, k l/16) and B(k l/16, col l%16); element v is row
// 4 v + l/16, column l%16.
template <bool kTransL>
__device__ inline dm_f64x4 mm16(const double* L, int ls, int row0, const double* R, int rs, int col0, int lane) {
    const int h = lane >> 4, c = lane & 15;
    dm_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k4 = 0; k4 < kPair / 4; k4++) {
        const int k = 4 * k4 + h;
        const double x = kTransL ? L[k * ls + row0 + c] : L[(row0 + c) * ls + k];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, R[k * rs + col0 + c], acc, 0, 0, 0);
    }
    return acc;
}

// A sector's place in launch `round`: its own round index a, and whether it
// takes part at all (sectors with fewer blocks than the largest sit out the
// rest of a sweep of max_rounds).
struct DmClock {
    int a, t, t_prev;  // t: round of its sweep, t_prev: that of round a - 1
    bool active;
};

__device__ inline DmClock dm_clock(int nb, int round, int max_rounds) {
    const int sweep = round / max_rounds, t = round - sweep * max_rounds;
    return {sweep * (nb - 1) + t, t, t ? t - 1 : nb - 2, t < nb - 1};
}

// Pair k in its sector's round ck.a.
__device__ inline void dm_pair(const DmSector& s, int sec, int k, const DmClock& ck, DmPairLds& L,
                               const DmBuffers& g) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cur = ck.a & 1, old = cur ^ 1;
    DmState* st = g.st + sec;
    int* flags = g.flags + s.flag_off;
    const int* flags_old = flags + old * g.f_round;
    int* flag = flags + cur * g.f_round + k;
    const int quiet = ck.a ? st->quiet[old] : 0;
    const bool done = quiet >= s.nb - 1;
    if (k == 0 && tid == 0) {
        int any = ck.a == 0;
        for (int x = 0; x < s.nb / 2 && ck.a && !done; x++) any |= flags_old[x];
        st->quiet[cur] = done ? quiet : any ? 0 : quiet + 1;
    }
    if (done) {
        if (tid == 0) *flag = 0;
        return;
    }
    const double floor = st->floor;
    const int expo = st->exponent;
    const bool full = ck.t == 0;
    int I, J;
    circle_pair(s.nb, ck.t, k, I, J);
    const int64_t np = s.npad;
    const double* Sold = g.S + old * g.q_round + s.q_off;
    if (tid == 0) L.any = L.work = 0;
    constexpr int kPer = (kPair * kPair + kPairThreads - 1) / kPairThreads;
    double sv[kPer];  // this thread's entries e = tid + kPairThreads j of S
    bool mixed = false;  // the block between I and J comes from a product
    int P1 = 0, P2 = 0, h1 = 0, h2 = 0;
    if (ck.a == 0) {
        const double* a = g.A + s.a_off;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = min(tid + kPairThreads * j, kPair * kPair - 1);
            sv[j] = a[(int64_t)pair_row(I, J, e >> 6) * np + pair_row(I, J, e & 63)];
        }
    } else {
        circle_where(s.nb, ck.t_prev, I, P1, h1);
        circle_where(s.nb, ck.t_prev, J, P2, h2);
        mixed = P1 != P2;
        const double *s1 = Sold + (int64_t)P1 * kPair * kPair, *s2 = Sold + (int64_t)P2 * kPair * kPair;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = min(tid + kPairThreads * j, kPair * kPair - 1), x = e >> 6, y = e & 63;
            sv[j] = !mixed              ? s1[e]
                    : y < kBlk          ? (x < kBlk ? s1[(kBlk * h1 + x) * kPair + kBlk * h1 + y] : 0.0)
                    : x < kBlk          ? 0.0
                                        : s2[(kBlk * (h2 - 1) + x) * kPair + kBlk * (h2 - 1) + y];
        }
    }
    double cross[4] = {0.0, 0.0, 0.0, 0.0};  // waves 0..3: 16 x 16 of the block between I and J
    if (mixed) {
        int I1, J1, I2, J2;
        circle_pair(s.nb, ck.t_prev, P1, I1, J1);
        circle_pair(s.nb, ck.t_prev, P2, I2, J2);
        const double* a = g.A + old * g.a_round + s.a_off;
        const double* q1 = g.Q + old * g.q_round + s.q_off + (int64_t)P1 * kPair * kPair;
        const double* q2 = g.Q + old * g.q_round + s.q_off + (int64_t)P2 * kPair * kPair;
        const int r1 = flags_old[P1], r2 = flags_old[P2];
        double xv[kPer], lv[kPer], rv[kPer];
        constexpr int kPerH = (kPair * kBlk + kPairThreads - 1) / kPairThreads;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = min(tid + kPairThreads * j, kPair * kPair - 1);
            xv[j] = a[(int64_t)pair_row(I1, J1, e >> 6) * np + pair_row(I2, J2, e & 63)];
        }
#pragma unroll
        for (int j = 0; j < kPerH; j++) {
            const int e = min(tid + kPairThreads * j, kPair * kBlk - 1), x = e >> 5, y = e & 31;
            lv[j] = r1 ? q1[x * kPair + kBlk * h1 + y] : x == kBlk * h1 + y ? 1.0 : 0.0;
            rv[j] = r2 ? q2[x * kPair + kBlk * h2 + y] : x == kBlk * h2 + y ? 1.0 : 0.0;
        }
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = tid + kPairThreads * j;
            if (e < kPair * kPair) L.S[(e >> 6) * kLs + (e & 63)] = xv[j];
        }
#pragma unroll
        for (int j = 0; j < kPerH; j++) {
            const int e = tid + kPairThreads * j;
            if (e < kPair * kBlk) {
                L.L1[(e >> 5) * kHalf + (e & 31)] = lv[j];
                L.R2[(e >> 5) * kHalf + (e & 31)] = rv[j];
            }
        }
        __syncthreads();
        dm_f64x4 z = {0.0, 0.0, 0.0, 0.0};
        const int zr = 16 * (wave >> 1), zc = 16 * (wave & 1), h = lane >> 4, c = lane & 15;
        if (wave < 8) z = mm16<false>(L.S, kLs, zr, L.R2, kHalf, zc, lane);
        __syncthreads();
        if (wave < 8)
#pragma unroll
            for (int v = 0; v < 4; v++) L.S[(zr + 4 * v + h) * kHalf + zc + c] = z[v];
        __syncthreads();
        if (wave < 4) {
            const dm_f64x4 y = mm16<true>(L.L1, kHalf, zr, L.S, kHalf, zc, lane);
#pragma unroll
            for (int v = 0; v < 4; v++) cross[v] = y[v];
        }
    }
    __syncthreads();
    {
        bool over = false;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = tid + kPairThreads * j, x = e >> 6, y = e & 63;
            const bool between = x < kBlk && y >= kBlk;
            if (e >= kPair * kPair || x > y || (mixed && between)) continue;
            const double v = ldexp(sv[j], -expo);
            L.S[x * kLs + y] = v;
            if (x != y && (full || between) && !(fabs(v) <= floor)) over = true;
        }
        if (mixed && wave < 4)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int x = 16 * (wave >> 1) + 4 * v + (lane >> 4), y = kBlk + 16 * (wave & 1) + (lane & 15);
                const double w = ldexp(cross[v], -expo);
                L.S[x * kLs + y] = w;
                if (!(fabs(w) <= floor)) over = true;
            }
        if (over) L.work = 1;
    }
    __syncthreads();
    double* Snew = g.S + cur * g.q_round + s.q_off + (int64_t)k * kPair * kPair;
    double* diag = g.diag + s.d_off;
    if (!L.work) {
        for (int e = tid; e < kPair * kPair; e += kPairThreads) {
            const int x = e >> 6, y = e & 63;
            const double v = ldexp(L.S[su(x, y)], expo);
            Snew[e] = v;
            if (x == y) diag[pair_row(I, J, x)] = v;
        }
        if (tid == 0) *flag = 0;
        return;
    }
    if (tid < 32) {
        const int p = slot_index(full, tid, false, 0), q = slot_index(full, tid, true, 0);
        double app = L.S[p * kLs + p], aqq = L.S[q * kLs + q];
        double left;
        const DmRot r = dm_rotation(app, aqq, L.S[su(p, q)], floor, left);
        L.S[su(p, q)] = left;
        L.rot[0][tid] = double2{r.c, r.s};
        L.D[0][p] = app;
        L.D[0][q] = aqq;
        if (r.s != 0.0) L.any = 1;
    }
    // Q's columns of this wave's slots, row `lane`
    double qt[8], qb[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        qt[j] = slot_index(full, 8 * (wave & 3) + j, false, 0) == lane ? 1.0 : 0.0;
        qb[j] = slot_index(full, 8 * (wave & 3) + j, true, 0) == lane ? 1.0 : 0.0;
    }
    __syncthreads();
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    if (full) {
        if (wv < kQWaves) dm_sweep_q<true>(L, wv, lane, qt, qb);
        else dm_sweep_full(L, floor, wv, lane);
    } else {
        if (wv < kQWaves) dm_sweep_q<false>(L, wv, lane, qt, qb);
        else dm_sweep_cross(L, floor, wv, lane);
        __syncthreads();
    }
    const int last = (full ? kFull : kCross) & 1;
    for (int e = tid; e < kPair * kPair; e += kPairThreads) {
        const int x = e >> 6, y = e & 63;
        const double v = ldexp(x == y ? L.D[last][x] : L.S[su(x, y)], expo);
        Snew[e] = v;
        if (x == y) diag[pair_row(I, J, x)] = v;
    }
    __syncthreads();
    // Q through the LDS, so that its rows are written whole
    if (wave < kQWaves)
#pragma unroll
        for (int j = 0; j < 8; j++) {
            L.S[lane * kLs + slot_index(full, 8 * wave + j, false, 0)] = qt[j];
            L.S[lane * kLs + slot_index(full, 8 * wave + j, true, 0)] = qb[j];
        }
    __syncthreads();
    double* qw = g.Q + cur * g.q_round + s.q_off + (int64_t)k * kPair * kPair;
    for (int e = tid; e < kPair * kPair; e += kPairThreads) qw[e] = L.S[(e >> 6) * kLs + (e & 63)];
    if (tid == 0) *flag = L.any;
}

struct DmApplyLds {
    double X[kPair * kLs], R[kPair * kLs];
};

// The rotations of a sector's last round on the block of pairs P1 <= P2 of its
// matrix, from the old copy to the new one: Q1^T X Q2 and its mirror, or the
// swept submatrix itself.
__device__ inline void dm_apply_a(const DmSector& s, int P1, int P2, const DmClock& ck, DmApplyLds& L,
                                  const DmBuffers& g) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 4, c = lane & 15;
    const int cur = ck.a & 1, old = cur ^ 1;
    const int64_t np = s.npad;
    const double* from = g.A + old * g.a_round + s.a_off;
    double* to = g.A + cur * g.a_round + s.a_off;
    const int64_t qp = s.q_off + old * g.q_round;
    int I1, J1, I2, J2;
    circle_pair(s.nb, ck.t_prev, P1, I1, J1);
    circle_pair(s.nb, ck.t_prev, P2, I2, J2);
    if (P1 == P2) {
        const double* sv = g.S + qp + (int64_t)P1 * kPair * kPair;
        for (int e = tid; e < kPair * kPair; e += kPairThreads)
            to[(int64_t)pair_row(I1, J1, e >> 6) * np + pair_row(I1, J1, e & 63)] = sv[e];
        return;
    }
    const int* rf = g.flags + old * g.f_round + s.flag_off;
    const int r1 = rf[P1], r2 = rf[P2];
    const double *q1 = g.Q + qp + (int64_t)P1 * kPair * kPair, *q2 = g.Q + qp + (int64_t)P2 * kPair * kPair;
    constexpr int kPer = (kPair * kPair + kPairThreads - 1) / kPairThreads;
    double xv[kPer], lv[kPer], rv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int e = min(tid + kPairThreads * j, kPair * kPair - 1), x = e >> 6, z = e & 63;
        xv[j] = from[(int64_t)pair_row(I1, J1, x) * np + pair_row(I2, J2, z)];
        lv[j] = r1 ? q1[e] : 0.0;
        rv[j] = r2 ? q2[e] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int e = tid + kPairThreads * j, x = e >> 6, z = e & 63;
        if (e >= kPair * kPair) continue;
        L.X[x * kLs + z] = xv[j];
        L.R[x * kLs + z] = rv[j];
    }
    __syncthreads();
    const int row0 = 16 * (w >> 1), col0 = 32 * (w & 1);  // eight waves of 16 x 32
    auto put = [&](const dm_f64x4 (&y)[2]) {
        __syncthreads();
        if (w < 8)
#pragma unroll
            for (int bj = 0; bj < 2; bj++)
#pragma unroll
                for (int v = 0; v < 4; v++) L.X[(row0 + 4 * v + h) * kLs + col0 + 16 * bj + c] = y[bj][v];
    };
    dm_f64x4 y[2];
    if (r2) {
        if (w < 8)
            for (int bj = 0; bj < 2; bj++) y[bj] = mm16<false>(L.X, kLs, row0, L.R, kLs, col0 + 16 * bj, lane);
        put(y);
        __syncthreads();
    }
    if (r1) {
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int e = tid + kPairThreads * j;
            if (e < kPair * kPair) L.R[(e >> 6) * kLs + (e & 63)] = lv[j];
        }
        __syncthreads();
        if (w < 8)
            for (int bj = 0; bj < 2; bj++) y[bj] = mm16<true>(L.R, kLs, row0, L.X, kLs, col0 + 16 * bj, lane);
        put(y);
        __syncthreads();
    }
    // the block and its mirror, both written along rows
    for (int e = tid; e < kPair * kPair; e += kPairThreads) {
        const int x = e >> 6, z = e & 63;
        to[(int64_t)pair_row(I1, J1, x) * np + pair_row(I2, J2, z)] = L.X[x * kLs + z];
        to[(int64_t)pair_row(I2, J2, x) * np + pair_row(I1, J1, z)] = L.X[z * kLs + x];
    }
}

// V_{R,P} <- V_{R,P} Q_P of the last round for one 64-row tile R.
__device__ inline void dm_apply_v(const DmSector& s, int tile, int P, const DmClock& ck, DmApplyLds& L,
                                  const DmBuffers& g) {
    const int old = (ck.a & 1) ^ 1;
    if (!g.flags[old * g.f_round + s.flag_off + P]) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 4, c = lane & 15;
    int I, J;
    circle_pair(s.nb, ck.t_prev, P, I, J);
    double* v = g.V + s.a_off;
    const double* qm = g.Q + old * g.q_round + s.q_off + (int64_t)P * kPair * kPair;
    const int64_t r0 = (int64_t)tile * kPair, np = s.npad;
    constexpr int kPer = (kPair * kPair + kPairThreads - 1) / kPairThreads;
    double xv[kPer], rv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int e = min(tid + kPairThreads * j, kPair * kPair - 1), x = e >> 6, z = e & 63;
        xv[j] = v[(r0 + x) * np + pair_row(I, J, z)];
        rv[j] = qm[e];
    }
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int e = tid + kPairThreads * j, x = e >> 6, z = e & 63;
        if (e >= kPair * kPair) continue;
        L.X[x * kLs + z] = xv[j];
        L.R[x * kLs + z] = rv[j];
    }
    __syncthreads();
    if (w >= 8) return;
    const int row0 = 16 * (w >> 1), col0 = 32 * (w & 1);
#pragma unroll
    for (int bj = 0; bj < 2; bj++) {
        const dm_f64x4 y = mm16<false>(L.X, kLs, row0, L.R, kLs, col0 + 16 * bj, lane);
        const int64_t col = pair_row(I, J, col0 + 16 * bj + c);
#pragma unroll
        for (int e = 0; e < 4; e++) v[(r0 + row0 + 4 * e + h) * np + col] = y[e];
    }
}

// One round of every sector: its pairs first (they decide the launch's time),
// then the last round's rotations on matrix and eigenvectors.
__global__ __launch_bounds__(kPairThreads) void dm_round_kernel(const DmSector* __restrict__ secs,
                                                                const DmItem* __restrict__ items, DmBuffers g,
                                                                int round, int max_rounds) {
    __shared__ __attribute__((aligned(16))) char lds[std::max(sizeof(DmPairLds), sizeof(DmApplyLds))];
    const DmItem it = items[blockIdx.x];
    const DmSector s = secs[it.sec];
    const DmClock ck = dm_clock(s.nb, round, max_rounds);
    if (!ck.active) return;
    if (it.kind == kItemPair) {
        dm_pair(s, it.sec, it.a, ck, *reinterpret_cast<DmPairLds*>(lds), g);
        return;
    }
    if (ck.a == 0 || g.st[it.sec].quiet[(ck.a & 1) ^ 1] >= s.nb - 1) return;
    DmApplyLds& L = *reinterpret_cast<DmApplyLds*>(lds);
    if (it.kind == kItemA) dm_apply_a(s, it.a, it.b, ck, L, g);
    else dm_apply_v(s, it.a, it.b, ck, L, g);
}

// Sectors that still rotate after launch `round` (the last of a sweep).
__global__ __launch_bounds__(256) void dm_count_kernel(const DmSector* __restrict__ secs,
                                                       const DmState* __restrict__ st,
                                                       const int* __restrict__ flags, int f_round, int n_sec,
                                                       int sweep, int* __restrict__ out) {
    __shared__ int red[256];
    int c = 0;
    for (int k = threadIdx.x; k < n_sec; k += 256) {
        const int nb = secs[k].nb, par = ((sweep + 1) * (nb - 1) - 1) & 1;
        const int* f = flags + par * f_round + secs[k].flag_off;
        int quiet = st[k].quiet[par], any = 0;
        for (int x = 0; x < nb / 2; x++) any |= f[x];
        if (quiet < nb - 1) quiet = any ? 0 : quiet + 1;
        c += quiet < nb - 1;
    }
    red[threadIdx.x] = c;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

// ---------------------------------------------------------------------------
// Per sector: the diagonal sorted descending (equal values by position, a
// bitonic network in LDS), written to w and to the concatenated list, with the
// positions it came from.
__device__ inline bool dm_before(double ka, int ia, double kb, int ib) {
    return ka > kb || (ka == kb && ia < ib);
}

__global__ __launch_bounds__(256) void dm_sort_kernel(const DmSector* __restrict__ secs,
                                                      const double* __restrict__ diag, double* __restrict__ wall,
                                                      int* __restrict__ order) {
    const DmSector s = secs[blockIdx.x];
    __shared__ double key[kSortMax];
    __shared__ int idx[kSortMax];
    const int tid = threadIdx.x;
    int p2 = 1;
    while (p2 < s.n) p2 <<= 1;
    for (int i = tid; i < p2; i += 256) {
        key[i] = i < s.n ? diag[s.d_off + i] + 0.0 : -INFINITY;
        idx[i] = i;
    }
    __syncthreads();
    for (int size = 2; size <= p2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < p2; i += 256) {
                const int j = i ^ stride;
                if (j <= i) continue;
                const bool up = (i & size) == 0;
                const bool sw = up ? dm_before(key[j], idx[j], key[i], idx[i])
                                   : dm_before(key[i], idx[i], key[j], idx[j]);
                if (sw) {
                    const double tk = key[i];
                    key[i] = key[j];
                    key[j] = tk;
                    const int tj = idx[i];
                    idx[i] = idx[j];
                    idx[j] = tj;
                }
            }
            __syncthreads();
        }
    }
    for (int k = tid; k < s.n; k += 256) {
        s.w[k] = key[k];
        wall[s.w_off + k] = key[k];
        // idx[k] < n for finite diagonals; the clamp keeps the reads in the
        // sector's block should a non-finite value reorder the padding
        order[s.w_off + k] = idx[k] < s.n ? idx[k] : k;
    }
}

// The eigenvector columns in descending order into the caller's V, kGatherRows
// rows of a sector per workgroup (one workgroup per sector: 104 us for 60
// sectors of up to 246 states, now 7).
constexpr int kGatherRows = 16;
__global__ __launch_bounds__(256) void dm_gather_kernel(const DmSector* __restrict__ secs,
                                                        const double* __restrict__ Vw, const int* __restrict__ order) {
    const DmSector s = secs[blockIdx.x];
    const int row0 = blockIdx.y * kGatherRows, rows = min(kGatherRows, s.n - row0);
    const double* v = Vw + s.a_off;
    for (int col = threadIdx.x & 63; col < s.n; col += 64) {
        const int src = order[s.w_off + col];
        for (int r = threadIdx.x >> 6; r < rows; r += 4)
            s.V[(int64_t)(row0 + r) * s.ld_v + col] = v[(int64_t)(row0 + r) * s.npad + src];
    }
}

// Eigenvalues as unsigned keys with the same order (negative zero counts as zero).
__device__ inline uint64_t dm_key(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x + 0.0);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// Number of leading entries of a descending list whose key is >= c.
__device__ inline int dm_count_ge(const double* w, int n, uint64_t c) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (dm_key(w[mid]) >= c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The m_keep largest eigenvalues over all sectors: the m_keep-th largest key T
// found eight bits at a time (a histogram of the keys that share T's higher
// bits; 64 counting passes, one per bit, took 70 us for 4 096 values, now
// 25), all entries above T kept, entries equal to T handed out in sector
// order; then the weight left out, per sector by one wave (strided lanes, then
// a fixed butterfly) and over sectors in sector order.
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

__device__ inline long long dm_wave_sum(long long x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__global__ __launch_bounds__(kSelThreads) void dm_select_kernel(const DmSector* __restrict__ secs, int n_sec,
                                                                const double* __restrict__ wall, int64_t m_keep,
                                                                int64_t total, int* __restrict__ above,
                                                                int* __restrict__ equal, double* __restrict__ part,
                                                                int32_t* __restrict__ kept,
                                                                double* __restrict__ eps) {
    __shared__ unsigned hist[256];
    __shared__ uint64_t s_T;
    __shared__ long long s_need;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (m_keep >= total || m_keep == 0) {
        for (int k = tid; k < n_sec; k += kSelThreads) kept[k] = m_keep == 0 ? 0 : secs[k].n;
    } else {
        if (tid == 0) {
            s_T = 0;
            s_need = m_keep;
        }
        for (int shift = 56; shift >= 0; shift -= 8) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            const uint64_t T = s_T;
            for (int64_t e = tid; e < (total + 63) / 64 * 64; e += kSelThreads) {
                const uint64_t key = e < total ? dm_key(wall[e]) : 0;
                const bool in = e < total && (shift == 56 || (key >> (shift + 8)) == (T >> (shift + 8)));
                const unsigned digit = (unsigned)(key >> shift) & 255;
                // the lanes that share the first one's digit add together
                const unsigned long long lanes = __ballot(in);
                if (lanes == 0) continue;
                const int lead = __builtin_ctzll(lanes);
                const bool same = in && digit == (unsigned)__shfl((int)digit, lead);
                const unsigned long long alike = __ballot(same);
                if (lane == lead) atomicAdd(&hist[digit], (unsigned)__popcll(alike));
                else if (in && !same) atomicAdd(&hist[digit], 1u);
            }
            __syncthreads();
            if (wave == 0) {
                // four digits per lane, from the largest down
                unsigned h[4], own = 0;
#pragma unroll
                for (int j = 0; j < 4; j++) own += h[j] = hist[255 - 4 * lane - j];
                long long upto = own;
                for (int o = 1; o < 64; o <<= 1) {
                    const long long x = __shfl_up(upto, o);
                    if (lane >= o) upto += x;
                }
                const long long need = s_need;
                long long before = upto - own;  // keys with larger digits than this lane's
                if (before < need && need <= upto) {
                    int j = 0;
                    while (j < 3 && before + h[j] < need) before += h[j++];
                    s_T = T | (uint64_t)(255 - 4 * lane - j) << shift;
                    s_need = need - before;
                }
            }
            __syncthreads();
        }
        const uint64_t T = s_T;
        for (int k = tid; k < n_sec; k += kSelThreads) {
            const double* w = wall + secs[k].w_off;
            const int ge = dm_count_ge(w, secs[k].n, T);
            const int gt = T == ~0ull ? 0 : dm_count_ge(w, secs[k].n, T + 1);
            above[k] = gt;
            equal[k] = ge - gt;
        }
        __syncthreads();
        if (wave == 0) {
            long long need = m_keep, sum = 0;
            for (int k = lane; k < n_sec; k += 64) sum += above[k];
            need -= dm_wave_sum(sum);
            for (int k0 = 0; k0 < n_sec; k0 += 64) {
                const int k = k0 + lane, eq = k < n_sec ? equal[k] : 0;
                long long upto = eq;
                for (int o = 1; o < 64; o <<= 1) {
                    const long long x = __shfl_up(upto, o);
                    if (lane >= o) upto += x;
                }
                const long long left = need - (upto - eq);
                if (k < n_sec) kept[k] = above[k] + (int)(left < 0 ? 0 : left < eq ? left : eq);
                need -= __shfl(upto, 63);
                if (need < 0) need = 0;
            }
        }
    }
    __syncthreads();
    for (int k = wave; k < n_sec; k += kSelWaves) {
        const double* w = wall + secs[k].w_off;
        double acc = 0.0;
        for (int i = kept[k] + lane; i < secs[k].n; i += 64) acc += w[i];
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
        if (lane == 0) part[k] = acc;
    }
    __syncthreads();
    if (wave == 0) {
        double acc = 0.0;
        for (int k0 = 0; k0 < n_sec; k0 += 64) {
            const double p = k0 + lane < n_sec ? part[k0 + lane] : 0.0;
            const int m = min(64, n_sec - k0);
            for (int i = 0; i < m; i++) acc += __shfl(p, i);
        }
        if (lane == 0) eps[0] = acc;
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct DmLayout {
    std::vector<DmSector> secs;
    std::vector<DmItem> rho_items, items;
    size_t off_secs, off_state, off_rho, off_items, off_flags, off_count, off_above, off_equal, off_part;
    size_t off_A, off_V, off_S, off_Q, off_D, off_W, off_order, total;
    int64_t a_round, q_round;  // doubles of one copy of the matrices, of one round's submatrices
    int f_round;               // flags of one round
    int n_pair, n_apply_v;     // items: the pairs, then V updates, then A updates
    int max_rounds;            // rounds per sweep: max over sectors of nb - 1
    int max_n;
};

DmLayout dm_layout(const rot_dm_sector* in, int n_sec) {
    DmLayout L;
    std::vector<DmItem> v_items, a_items;
    int64_t a_off = 0, q_off = 0, w_off = 0, d_off = 0;
    int flag_off = 0;
    L.max_rounds = 1;
    L.max_n = 0;
    for (int k = 0; k < n_sec; k++) {
        DmSector s{};
        s.n = in[k].n;
        s.r = in[k].r;
        s.npad = (s.n + kPair - 1) / kPair * kPair;
        s.nb = s.npad / kBlk;
        s.psi = in[k].psi;
        s.ld_psi = in[k].ld_psi;
        s.w = in[k].w;
        s.V = in[k].V;
        s.ld_v = in[k].ld_v;
        s.a_off = a_off;
        s.q_off = q_off;
        s.w_off = w_off;
        s.d_off = d_off;
        s.flag_off = flag_off;
        const int h = s.nb / 2, tiles = s.npad / kPair;
        a_off += (int64_t)s.npad * s.npad;
        q_off += (int64_t)h * kPair * kPair;
        w_off += s.n;
        d_off += s.npad;
        flag_off += h;
        L.max_rounds = std::max(L.max_rounds, s.nb - 1);
        L.max_n = std::max(L.max_n, s.n);
        for (int j = 0; j < tiles; j++)
            for (int i = 0; i <= j; i++) L.rho_items.push_back({k, i, j, 0});
        for (int p = 0; p < h; p++) L.items.push_back({k, p, 0, kItemPair});
        for (int p2 = 0; p2 < h; p2++)
            for (int p1 = 0; p1 <= p2; p1++) a_items.push_back({k, p1, p2, kItemA});
        for (int rt = 0; rt < tiles; rt++)
            for (int p = 0; p < h; p++) v_items.push_back({k, rt, p, kItemV});
        L.secs.push_back(s);
    }
    L.n_pair = (int)L.items.size();
    L.n_apply_v = (int)v_items.size();
    L.items.insert(L.items.end(), v_items.begin(), v_items.end());
    L.items.insert(L.items.end(), a_items.begin(), a_items.end());
    L.a_round = a_off;
    L.q_round = q_off;
    L.f_round = flag_off;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align256(bytes);
        return at;
    };
    L.off_secs = take(sizeof(DmSector) * n_sec);
    L.off_rho = take(sizeof(DmItem) * L.rho_items.size());
    L.off_items = take(sizeof(DmItem) * L.items.size());
    L.off_state = take(sizeof(DmState) * n_sec);
    L.off_flags = take(sizeof(int) * 2 * (size_t)flag_off);
    L.off_count = take(sizeof(int));
    L.off_above = take(sizeof(int) * n_sec);
    L.off_equal = take(sizeof(int) * n_sec);
    L.off_part = take(sizeof(double) * n_sec);
    L.off_A = take(sizeof(double) * 2 * (size_t)a_off);
    L.off_V = take(sizeof(double) * (size_t)a_off);
    L.off_S = take(sizeof(double) * 2 * (size_t)q_off);
    L.off_Q = take(sizeof(double) * 2 * (size_t)q_off);
    L.off_D = take(sizeof(double) * (size_t)d_off);
    L.off_W = take(sizeof(double) * (size_t)w_off);
    L.off_order = take(sizeof(int) * (size_t)w_off);
    L.total = o;
    return L;
}

}  // namespace

size_t density_workspace_bytes(const rot_dm_sector* sectors, int n_sectors) {
    return dm_layout(sectors, n_sectors).total;
}

hipError_t density_basis(const rot_dm_sector* sectors, int n_sec, int64_t m_keep, int32_t* kept, double* eps,
                         void* workspace, hipStream_t stream, bool* converged) {
    DmLayout L = dm_layout(sectors, n_sec);
    char* ws = static_cast<char*>(workspace);
    // host tables -> workspace head (one copy; the host buffer outlives it: the
    // first convergence check below synchronises the stream)
    std::vector<char> head(L.off_state, 0);
    std::memcpy(head.data() + L.off_secs, L.secs.data(), sizeof(DmSector) * n_sec);
    std::memcpy(head.data() + L.off_rho, L.rho_items.data(), sizeof(DmItem) * L.rho_items.size());
    std::memcpy(head.data() + L.off_items, L.items.data(), sizeof(DmItem) * L.items.size());
    hipError_t e = hipMemcpyAsync(ws, head.data(), head.size(), hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return e;
    const DmSector* secs = reinterpret_cast<const DmSector*>(ws + L.off_secs);
    const DmItem* rho_items = reinterpret_cast<const DmItem*>(ws + L.off_rho);
    const DmItem* items = reinterpret_cast<const DmItem*>(ws + L.off_items);
    int* count = reinterpret_cast<int*>(ws + L.off_count);
    double* W = reinterpret_cast<double*>(ws + L.off_W);
    DmBuffers g{};
    g.A = reinterpret_cast<double*>(ws + L.off_A);
    g.V = reinterpret_cast<double*>(ws + L.off_V);
    g.S = reinterpret_cast<double*>(ws + L.off_S);
    g.Q = reinterpret_cast<double*>(ws + L.off_Q);
    g.diag = reinterpret_cast<double*>(ws + L.off_D);
    g.st = reinterpret_cast<DmState*>(ws + L.off_state);
    g.flags = reinterpret_cast<int*>(ws + L.off_flags);
    g.a_round = L.a_round;
    g.q_round = L.q_round;
    g.f_round = L.f_round;

    e = prof_timed("dm_rho", stream, [&] {
        hipLaunchKernelGGL(dm_rho_kernel, dim3((unsigned)L.rho_items.size()), dim3(256), 0, stream, secs,
                           rho_items, g.A, g.V);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(dm_prep_kernel, dim3(n_sec), dim3(256), 0, stream, secs, (const double*)g.A, g.st);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    *converged = false;
    int round = 0;
    auto launch = [&](int first, int n) {
        return prof_timed("dm_jacobi_round", stream, [&] {
            hipLaunchKernelGGL(dm_round_kernel, dim3((unsigned)n), dim3(kPairThreads), 0, stream, secs, items + first, g,
                               round, L.max_rounds);
            return hipGetLastError();
        });
    };
    for (int sweep = 0; sweep < kMaxSweeps && !*converged; sweep++) {
        for (int r = 0; r < L.max_rounds; r++, round++) {
            e = launch(0, (int)L.items.size());
            if (e != hipSuccess) return e;
        }
        // asking costs 25 us of idle device, a sweep after the last one (its
        // workgroups find their sector done) 3 us a launch
        if (sweep + 1 < kMaxSweeps && (sweep + 1 < kFirstCheck || (sweep + 1 - kFirstCheck) % kCheckEvery)) continue;
        hipLaunchKernelGGL(dm_count_kernel, dim3(1), dim3(256), 0, stream, secs, (const DmState*)g.st,
                           (const int*)g.flags, L.f_round, n_sec, sweep, count);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        int host_count = -1;
        e = hipMemcpyAsync(&host_count, count, sizeof(int), hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return e;
        *converged = host_count == 0;
    }
    if (!*converged) {
        // the last round's rotations are still due on the eigenvectors
        e = launch(L.n_pair, L.n_apply_v);
        if (e != hipSuccess) return e;
    }
    int64_t total = 0;
    for (int k = 0; k < n_sec; k++) total += sectors[k].n;
    return prof_timed("dm_sort_select", stream, [&] {
        int* order = reinterpret_cast<int*>(ws + L.off_order);
        hipLaunchKernelGGL(dm_sort_kernel, dim3(n_sec), dim3(256), 0, stream, secs, (const double*)g.diag, W, order);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(dm_gather_kernel, dim3(n_sec, (unsigned)((L.max_n + kGatherRows - 1) / kGatherRows)), dim3(256),
                           0, stream, secs, (const double*)g.V, (const int*)order);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(dm_select_kernel, dim3(1), dim3(kSelThreads), 0, stream, secs, n_sec, (const double*)W, m_keep,
                           total, reinterpret_cast<int*>(ws + L.off_above), reinterpret_cast<int*>(ws + L.off_equal),
                           reinterpret_cast<double*>(ws + L.off_part), kept, eps);
        return hipGetLastError();
    });
}

}  // namespace rot
