// The superblock Hamiltonian applied to a state over quantum-number blocks
// (Eq. (9) and Eq. (10)): out = sum_l coef_l (O_B (x) O_a (x) O_a~ (x) O_B~) psi.
//
// The state is one dense block per system sector Q of [B a] (rows: site a
// state s slow, B state fast) paired with environment sector P = target - Q of
// [a~ B~] (columns: site a~ state t slow, B~ state fast).  Inside a block the
// rows split into segments (s, q) of B sector q = Q - qn(s) and the columns into
// segments (t, p).  A term maps source segment (s, q) x (t, p) to output
// segment (s', q + dB) x (t', p + dB~) with weight site_a[s'][s] site_at[t'][t]:
//   operator on B:  out_seg += w coef O_B(q' <- q) psi_seg        (K = dim q)
//   operator on B~: out_seg += w coef psi_seg O_B~(p' <- p)^T      (K = dim p)
//   site terms only: out_seg += w coef psi_seg
// The plan lists, per output segment and in term order, every contribution
// reaching it, and cuts the segment into square tiles; one wave computes one
// tile from the segment's list and writes it once, so the sum has a fixed order
// and needs no atomics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "rot_internal.h"

namespace rot {
namespace {

constexpr int kSbMaxSite = 16;

enum : int { kFromLeft = 0, kFromRight = 1, kCopy = 2 };

constexpr int kSbKs = 16;  // k per step

// A step of a segment's sum: 16 k of a product, or a scaled copy.  Offsets are
// those of the segment's first row and column and of the step's first k.
struct SbStep {
    double alpha;
    int64_t a_off;  // left: operator block (rows of the segment); right, copy: psi
    int64_t b_off;  // left: psi (columns of the segment); right: operator block (rows = segment columns)
    int lda, ldb;
    // kind; k below lo and from hi on count as zero (a last step of a longer
    // product starts 16 before its end, and lo cuts what the step before it
    // took); hi < 16: shorter products, nothing is read from hi on
    int kind, lo_hi;
};

struct SbTile {
    int64_t out_off, ldo;  // of the tile
    int r0, c0, rows, cols;
    int s_begin, s_end;
};

typedef double sb_f64x4 __attribute__((ext_vector_type(4)));
typedef double sb_f64x2 __attribute__((ext_vector_type(2)));
typedef sb_f64x2 sb_f64x2u __attribute__((aligned(8)));
typedef int sb_i32x4 __attribute__((ext_vector_type(4)));

// One step's operands of a wave: for a product, four consecutive k per lane of
// NB 16-row blocks of A and of B; for a copy, the psi entries of the lane's
// accumulator rows (those of blocks (0, j) in a[j], of (1, j) in b[j]).
template <int NB>
struct SbSet {
    sb_f64x4 a[NB], b[NB];
    double alpha;
    int kind, lo_hi;
};

__device__ inline int64_t sb_lane64(int lo, int hi, int l) {
    return (int64_t)(uint32_t)__builtin_amdgcn_readlane(lo, l) | (int64_t)__builtin_amdgcn_readlane(hi, l) << 32;
}

// C (16 NB x 16 NB at most) = sum of the segment's steps, one wave per tile.
// A state of 1024 + 1024 states has short segments and about 19 steps per tile,
// so the waves share nothing and meet at no barrier: operands go straight from
// the L2 to the registers of v_mfma_f64_16x16x4f64 in its own layout (lane l
// supplies A(l%16, k) and B(k, l%16), k = 4 (l/16) + j at instruction j, so that
// k-contiguous operands are read 32 bytes per lane; element v of the result is
// C(4 v + l/16, l%16)), and three register sets keep as many steps in flight.
// The plan lists the steps; 64 at a time are fetched, one per lane, and handed
// out by lane reads.  Rows and columns past the tile repeat its last one and are
// not stored.  Bound by the instructions around a step's four (NB = 2: sixteen)
// products.  Before, one 32 x 32 tile per workgroup through the LDS, 32 k per
// barrier; now, at 400 / 1024 / 2000 / 3500 states: 17.2 / 32.1 / 113 / 337 ->
// 10.8 / 25.0 / 95 / 229 us.  Not faster at 1024 states: loads through bounded
// descriptors instead of clamped addresses 26.9 us, turning k-contiguous
// operands through the wave's own LDS 37.0, 16 k per barrier with four steps in
// flight 29.4, tiles grouped by XCD 26.8.
template <int NB>
__global__ __launch_bounds__(256) void sb_tile_kernel(const SbTile* __restrict__ tiles, int n_tiles,
                                                      const SbStep* __restrict__ steps,
                                                      const double* __restrict__ left_blk,
                                                      const double* __restrict__ right_blk,
                                                      const double* __restrict__ psi, double* __restrict__ out) {
    const int t = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= n_tiles) return;
    const SbTile tl = tiles[t];
    const int lane = threadIdx.x & 63, h = lane >> 4, cl = lane & 15;
    int row[NB], col[NB];  // operand rows of this lane, inside the segment
#pragma unroll
    for (int i = 0; i < NB; i++) {
        row[i] = tl.r0 + min(16 * i + cl, tl.rows - 1);
        col[i] = tl.c0 + min(16 * i + cl, tl.cols - 1);
    }
    sb_f64x4 acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++) acc[i][j] = sb_f64x4{0.0, 0.0, 0.0, 0.0};
    // lane l's step: the l-th of the 64 from `base` on
    sb_i32x4 d0 = {0, 0, 0, 0}, d1 = {0, 0, 0, 0};
    int d8 = 0, d9 = 0;
    int base = tl.s_begin, next = tl.s_begin;
    auto fetch = [&]() __attribute__((always_inline)) {
        const int* p = reinterpret_cast<const int*>(steps + min(base + lane, tl.s_end - 1));
        d0 = sb_i32x4{p[0], p[1], p[2], p[3]};
        d1 = sb_i32x4{p[4], p[5], p[6], p[7]};
        d8 = p[8];
        d9 = p[9];
    };
    if (next < tl.s_end) fetch();
    auto load = [&](SbSet<NB>& s) __attribute__((always_inline)) {
        if (next >= tl.s_end) return;
        if (next - base == 64) {
            base += 64;
            fetch();
        }
        const int l = next - base;
        next++;
        s.alpha = __builtin_bit_cast(double, sb_lane64(d0[0], d0[1], l));
        const int64_t a_off = sb_lane64(d0[2], d0[3], l), b_off = sb_lane64(d1[0], d1[1], l);
        const int lda = __builtin_amdgcn_readlane(d1[2], l), ldb = __builtin_amdgcn_readlane(d1[3], l);
        s.kind = __builtin_amdgcn_readlane(d8, l);
        s.lo_hi = __builtin_amdgcn_readlane(d9, l);
        if (s.kind == kCopy) {
            const double* p = psi + a_off;
#pragma unroll
            for (int i = 0; i < NB; i++)
#pragma unroll
                for (int j = 0; j < NB; j++)
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int r = tl.r0 + min(16 * i + 4 * e + h, tl.rows - 1);
                        (i == 0 ? s.a[j] : s.b[j])[e] = p[(int64_t)r * lda + col[j]];
                    }
            return;
        }
        const bool left = s.kind == kFromLeft;
        const double *A = (left ? left_blk : psi) + a_off, *B = (left ? psi : right_blk) + b_off;
        const int hi = s.lo_hi >> 8;
        if (hi == kSbKs) {
            auto four = [&](const double* q) __attribute__((always_inline)) {
                const sb_f64x2 x = *reinterpret_cast<const sb_f64x2u*>(q), y = *reinterpret_cast<const sb_f64x2u*>(q + 2);
                return sb_f64x4{x[0], x[1], y[0], y[1]};
            };
#pragma unroll
            for (int i = 0; i < NB; i++) s.a[i] = four(A + (int64_t)row[i] * lda + 4 * h);
            if (left) {
                const double* q = B + (int64_t)(4 * h) * ldb;
#pragma unroll
                for (int e = 0; e < 4; e++)
#pragma unroll
                    for (int i = 0; i < NB; i++) s.b[i][e] = q[(int64_t)e * ldb + col[i]];
            } else {
#pragma unroll
                for (int i = 0; i < NB; i++) s.b[i] = four(B + (int64_t)col[i] * ldb + 4 * h);
            }
        } else {
            const int64_t bk = left ? ldb : 1, br = left ? 1 : ldb;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int k = min(4 * h + e, hi - 1);
#pragma unroll
                for (int i = 0; i < NB; i++) {
                    s.a[i][e] = A[(int64_t)row[i] * lda + k];
                    s.b[i][e] = B[k * bk + col[i] * br];
                }
            }
        }
    };
    auto run = [&](SbSet<NB>& s) __attribute__((always_inline)) {
        if (s.kind == kCopy) {
#pragma unroll
            for (int i = 0; i < NB; i++)
#pragma unroll
                for (int j = 0; j < NB; j++) acc[i][j] += s.alpha * (i == 0 ? s.a[j] : s.b[j]);
            return;
        }
        if (s.lo_hi != kSbKs << 8) {
            const int lo = s.lo_hi & 255, hi = s.lo_hi >> 8;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const bool in = 4 * h + e >= lo && 4 * h + e < hi;
#pragma unroll
                for (int i = 0; i < NB; i++) {
                    s.a[i][e] = in ? s.a[i][e] : 0.0;
                    s.b[i][e] = in ? s.b[i][e] : 0.0;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
            for (int i = 0; i < NB; i++)
#pragma unroll
                for (int j = 0; j < NB; j++)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.alpha * s.a[i][e], s.b[j][e], acc[i][j], 0, 0, 0);
    };
    SbSet<NB> s0, s1, s2;
    load(s0);
    load(s1);
    load(s2);
    for (int n = tl.s_end - tl.s_begin; n > 0; n -= 3) {
        run(s0);
        load(s0);
        if (n == 1) break;
        run(s1);
        load(s1);
        if (n == 2) break;
        run(s2);
        load(s2);
    }
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int r = 16 * i + 4 * v + h, c = 16 * j + cl;
                if (r < tl.rows && c < tl.cols) out[tl.out_off + r * tl.ldo + c] = acc[i][j][v];
            }
}

// 32 x 32 tiles read half as much and issue less per product, and pay once
// there are two waves of them for each SIMD (16 / 32 wide: 1024 states, 1076
// tiles, 25 / 34 us; 2000 states, 111 / 95; 3500 states, 6880 tiles, 314 / 229).
constexpr int64_t kSbWideTiles = 2048;

rot_status sberr(rot_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return set_error(s, buf);
}

using Qn = std::pair<int, int>;

// One segment of a system (or environment) sector: site state, block sector
// index and its first row (column) inside the sector.
struct Seg {
    int site, sec, start, dim;
};

struct Enlarged {
    std::map<Qn, std::vector<Seg>> segs;  // by sector numbers, segments in site order
    std::map<Qn, int> dim;
};

Enlarged enlarge(int d, const int32_t* site_qn, int n_sec, const rot_sector* sec) {
    Enlarged E;
    std::map<Qn, int> by_qn;
    for (int k = 0; k < n_sec; k++) by_qn[{sec[k].n_up, sec[k].n_dn}] = k;
    std::map<Qn, bool> seen;
    for (int k = 0; k < n_sec; k++)
        for (int s = 0; s < d; s++) seen[{sec[k].n_up + site_qn[2 * s], sec[k].n_dn + site_qn[2 * s + 1]}] = true;
    for (auto& kv : seen) {
        const Qn Q = kv.first;
        int start = 0;
        std::vector<Seg> v;
        for (int s = 0; s < d; s++) {
            auto it = by_qn.find({Q.first - site_qn[2 * s], Q.second - site_qn[2 * s + 1]});
            if (it == by_qn.end()) continue;
            v.push_back({s, it->second, start, sec[it->second].dim});
            start += sec[it->second].dim;
        }
        E.segs[Q] = v;
        E.dim[Q] = start;
    }
    return E;
}

struct Block {
    Qn Q;
    int rows, cols;
    int64_t offset;
};

std::vector<Block> psi_blocks(const rot_sb_problem* p, const Enlarged& sys, const Enlarged& env) {
    std::vector<Block> out;
    int64_t off = 0;
    for (auto& kv : sys.dim) {
        const Qn P{p->target[0] - kv.first.first, p->target[1] - kv.first.second};
        auto it = env.dim.find(P);
        if (it == env.dim.end()) continue;
        out.push_back({kv.first, kv.second, it->second, off});
        off += (int64_t)kv.second * it->second;
    }
    return out;
}

rot_status validate_sb(const rot_sb_problem* p) {
    if (!p) return sberr(ROT_ERR_INVALID_ARG, "null problem");
    if (p->d < 1 || p->d > kSbMaxSite || !p->site_qn) return sberr(ROT_ERR_INVALID_ARG, "need 1 <= d <= %d and site_qn", kSbMaxSite);
    for (int side = 0; side < 2; side++) {
        const int n = side ? p->n_right : p->n_left;
        const rot_sector* sec = side ? p->right : p->left;
        if (n < 1 || !sec) return sberr(ROT_ERR_INVALID_ARG, "%s block: need at least one sector", side ? "right" : "left");
        std::map<Qn, int> seen;
        for (int k = 0; k < n; k++) {
            if (sec[k].dim < 1) return sberr(ROT_ERR_INVALID_ARG, "%s sector %d: dim < 1", side ? "right" : "left", k);
            if (seen.count({sec[k].n_up, sec[k].n_dn}))
                return sberr(ROT_ERR_INVALID_ARG, "%s sector %d: repeated numbers", side ? "right" : "left", k);
            seen[{sec[k].n_up, sec[k].n_dn}] = k;
        }
        const int n_ops = side ? p->n_right_ops : p->n_left_ops;
        if (n_ops < 0) return sberr(ROT_ERR_INVALID_ARG, "negative operator count");
        if (n_ops > 0) {
            const int32_t* sh = side ? p->right_shift : p->left_shift;
            const int64_t* off = side ? p->right_off : p->left_off;
            const double* blk = side ? p->right_blk : p->left_blk;
            if (!sh || !off) return sberr(ROT_ERR_INVALID_ARG, "%s operators: null shift or offset table", side ? "right" : "left");
            bool any = false;
            for (int64_t e = 0; e < (int64_t)n_ops * n; e++) {
                if (off[e] < -1) return sberr(ROT_ERR_INVALID_ARG, "operator offset below -1");
                any = any || off[e] >= 0;
            }
            if (any && !blk) return sberr(ROT_ERR_INVALID_ARG, "%s operators: null block data", side ? "right" : "left");
        }
    }
    if (p->n_terms < 0 || (p->n_terms > 0 && !p->terms)) return sberr(ROT_ERR_INVALID_ARG, "null terms");
    for (int l = 0; l < p->n_terms; l++) {
        const rot_sb_term& t = p->terms[l];
        if (t.left_op < -1 || t.left_op >= p->n_left_ops || t.right_op < -1 || t.right_op >= p->n_right_ops)
            return sberr(ROT_ERR_INVALID_ARG, "term %d: operator index out of range", l);
        if (t.left_op >= 0 && t.right_op >= 0)
            return sberr(ROT_ERR_UNSUPPORTED, "term %d: operators on both blocks are not supported", l);
        int dn[2] = {0, 0};
        if (t.left_op >= 0) {
            dn[0] += p->left_shift[2 * t.left_op];
            dn[1] += p->left_shift[2 * t.left_op + 1];
        }
        if (t.right_op >= 0) {
            dn[0] += p->right_shift[2 * t.right_op];
            dn[1] += p->right_shift[2 * t.right_op + 1];
        }
        for (int w = 0; w < 2; w++) {
            const double* S = w ? t.site_at : t.site_a;
            if (!S) continue;
            bool have = false;
            int sh[2] = {0, 0};
            for (int a = 0; a < p->d; a++)
                for (int b = 0; b < p->d; b++) {
                    if (S[a * p->d + b] == 0.0) continue;
                    const int x = p->site_qn[2 * a] - p->site_qn[2 * b], y = p->site_qn[2 * a + 1] - p->site_qn[2 * b + 1];
                    if (have && (x != sh[0] || y != sh[1]))
                        return sberr(ROT_ERR_INVALID_ARG, "term %d: site matrix mixes particle-number shifts", l);
                    have = true;
                    sh[0] = x;
                    sh[1] = y;
                }
            dn[0] += sh[0];
            dn[1] += sh[1];
        }
        if (dn[0] != 0 || dn[1] != 0) return sberr(ROT_ERR_INVALID_ARG, "term %d: shifts do not add to zero", l);
    }
    return ROT_OK;
}

// Output segments (as one tile each) and their contributions, in block, segment
// and then term order (site states of the term's sums in ascending order).
void build_work(const rot_sb_problem* p, std::vector<SbTile>& segments, std::vector<SbStep>& st, double& flops,
                int64_t& total) {
    const Enlarged sys = enlarge(p->d, p->site_qn, p->n_left, p->left);
    const Enlarged env = enlarge(p->d, p->site_qn, p->n_right, p->right);
    const std::vector<Block> blocks = psi_blocks(p, sys, env);
    total = blocks.empty() ? 0 : blocks.back().offset + (int64_t)blocks.back().rows * blocks.back().cols;
    std::map<Qn, const Block*> block_of;
    for (const Block& b : blocks) block_of[b.Q] = &b;
    std::map<Qn, int> lsec, rsec;
    for (int k = 0; k < p->n_left; k++) lsec[{p->left[k].n_up, p->left[k].n_dn}] = k;
    for (int k = 0; k < p->n_right; k++) rsec[{p->right[k].n_up, p->right[k].n_dn}] = k;
    // first row (column) of segment (site state, block sector) inside an enlarged sector
    auto seg_start = [](const Enlarged& E, Qn Q, int site, int sec) {
        auto it = E.segs.find(Q);
        if (it == E.segs.end()) return -1;
        for (const Seg& g : it->second)
            if (g.site == site && g.sec == sec) return g.start;
        return -1;
    };
    const int d = p->d;
    const int32_t* qn = p->site_qn;
    flops = 0.0;
    for (const Block& ob : blocks) {
        const Qn P{p->target[0] - ob.Q.first, p->target[1] - ob.Q.second};
        for (const Seg& rs : sys.segs.at(ob.Q)) {
            const Qn qo{p->left[rs.sec].n_up, p->left[rs.sec].n_dn};
            for (const Seg& csg : env.segs.at(P)) {
                const Qn po{p->right[csg.sec].n_up, p->right[csg.sec].n_dn};
                SbTile tl{};
                tl.out_off = ob.offset + (int64_t)rs.start * ob.cols + csg.start;
                tl.ldo = ob.cols;
                tl.rows = rs.dim;
                tl.cols = csg.dim;
                tl.s_begin = (int)st.size();
                for (int l = 0; l < p->n_terms; l++) {
                    const rot_sb_term& t = p->terms[l];
                    const int lo = t.left_op, ro = t.right_op;
                    const Qn qs{qo.first - (lo >= 0 ? p->left_shift[2 * lo] : 0),
                                qo.second - (lo >= 0 ? p->left_shift[2 * lo + 1] : 0)};
                    const Qn ps{po.first - (ro >= 0 ? p->right_shift[2 * ro] : 0),
                                po.second - (ro >= 0 ? p->right_shift[2 * ro + 1] : 0)};
                    auto kq = lsec.find(qs);
                    auto kp = rsec.find(ps);
                    if (kq == lsec.end() || kp == rsec.end()) continue;
                    int64_t op_off = -1;
                    if (lo >= 0) op_off = p->left_off[(int64_t)lo * p->n_left + kq->second];
                    if (ro >= 0) op_off = p->right_off[(int64_t)ro * p->n_right + kp->second];
                    if ((lo >= 0 || ro >= 0) && op_off < 0) continue;
                    for (int sa = 0; sa < d; sa++) {
                        const double wa = t.site_a ? t.site_a[rs.site * d + sa] : (sa == rs.site ? 1.0 : 0.0);
                        if (wa == 0.0) continue;
                        for (int ta = 0; ta < d; ta++) {
                            const double wt = t.site_at ? t.site_at[csg.site * d + ta] : (ta == csg.site ? 1.0 : 0.0);
                            if (wt == 0.0) continue;
                            const Qn Qs{qs.first + qn[2 * sa], qs.second + qn[2 * sa + 1]};
                            const Qn Ps{ps.first + qn[2 * ta], ps.second + qn[2 * ta + 1]};
                            auto sb = block_of.find(Qs);
                            if (sb == block_of.end()) continue;
                            const Block& src = *sb->second;
                            const int rstart = seg_start(sys, Qs, sa, kq->second);
                            const int cstart = seg_start(env, Ps, ta, kp->second);
                            if (rstart < 0 || cstart < 0) continue;
                            SbStep c{};
                            int K = 1;
                            c.alpha = t.coef * wa * wt;
                            if (lo >= 0) {
                                K = p->left[kq->second].dim;
                                c.kind = kFromLeft;
                                c.a_off = op_off;
                                c.lda = K;
                                c.b_off = src.offset + (int64_t)rstart * src.cols + cstart;
                                c.ldb = src.cols;
                            } else if (ro >= 0) {
                                K = p->right[kp->second].dim;
                                c.kind = kFromRight;
                                c.a_off = src.offset + (int64_t)rstart * src.cols + cstart;
                                c.lda = src.cols;
                                c.b_off = op_off;
                                c.ldb = K;
                            } else {
                                c.kind = kCopy;
                                c.a_off = src.offset + (int64_t)rstart * src.cols + cstart;
                                c.lda = src.cols;
                            }
                            flops += 2.0 * tl.rows * tl.cols * K;
                            const int64_t bk = c.kind == kFromLeft ? c.ldb : 1;
                            for (int k0 = 0; k0 < K; k0 += kSbKs) {
                                SbStep x = c;
                                const int at = K - k0 >= kSbKs ? k0 : std::max(0, K - kSbKs);
                                x.a_off += c.kind == kCopy ? 0 : at;
                                x.b_off += at * bk;
                                x.lo_hi = (k0 - at) | std::min(K, kSbKs) << 8;
                                st.push_back(x);
                            }
                        }
                    }
                }
                tl.s_end = (int)st.size();
                segments.push_back(tl);
            }
        }
    }
}

}  // namespace
}  // namespace rot

struct rot_sb_plan_s {
    rot::SbTile* tiles = nullptr;
    rot::SbStep* steps = nullptr;
    int n_tiles = 0;
    int edge = 16;
    const double* left_blk = nullptr;
    const double* right_blk = nullptr;
    int64_t total = 0;
    double flops = 0.0;
};

using namespace rot;

extern "C" {

rot_status rot_sb_layout(const rot_sb_problem* p, int32_t capacity, int32_t* n_blocks, int32_t* qn, int32_t* rows,
                         int32_t* cols, int64_t* offset, int64_t* total) {
    const rot_status v = validate_sb(p);
    if (v != ROT_OK) return v;
    if (!n_blocks || !total) return sberr(ROT_ERR_INVALID_ARG, "null n_blocks or total");
    const Enlarged sys = enlarge(p->d, p->site_qn, p->n_left, p->left);
    const Enlarged env = enlarge(p->d, p->site_qn, p->n_right, p->right);
    const std::vector<Block> blocks = psi_blocks(p, sys, env);
    *n_blocks = (int32_t)blocks.size();
    *total = blocks.empty() ? 0 : blocks.back().offset + (int64_t)blocks.back().rows * blocks.back().cols;
    const int n = std::min<int>(std::max(capacity, 0), (int)blocks.size());
    for (int k = 0; k < n; k++) {
        if (qn) {
            qn[2 * k] = blocks[k].Q.first;
            qn[2 * k + 1] = blocks[k].Q.second;
        }
        if (rows) rows[k] = blocks[k].rows;
        if (cols) cols[k] = blocks[k].cols;
        if (offset) offset[k] = blocks[k].offset;
    }
    return ROT_OK;
}

rot_status rot_sb_plan_create(const rot_sb_problem* p, rot_sb_plan* plan) {
    rot::TraceRange trace_("rot_sb_plan_create");
    if (!plan) return sberr(ROT_ERR_INVALID_ARG, "null plan output");
    *plan = nullptr;
    const rot_status v = validate_sb(p);
    if (v != ROT_OK) return v;
    std::vector<SbTile> segments, tiles;
    std::vector<SbStep> steps;
    auto* P = new rot_sb_plan_s();
    build_work(p, segments, steps, P->flops, P->total);
    int64_t n32 = 0;
    for (const SbTile& g : segments) n32 += (int64_t)((g.rows + 31) / 32) * ((g.cols + 31) / 32);
    P->edge = n32 >= kSbWideTiles ? 32 : 16;
    // heaviest tiles first: all tiles do not fit on the chip at once, and the
    // ones dispatched last should be short
    std::vector<std::pair<int64_t, int>> order(segments.size());
    for (size_t i = 0; i < segments.size(); i++) order[i] = {segments[i].s_begin - segments[i].s_end, (int)i};
    std::stable_sort(order.begin(), order.end());
    for (const auto& o : order) {
        const SbTile& g = segments[o.second];
        for (int r0 = 0; r0 < g.rows; r0 += P->edge)
            for (int c0 = 0; c0 < g.cols; c0 += P->edge) {
                SbTile t = g;
                t.out_off += r0 * g.ldo + c0;
                t.r0 = r0;
                t.c0 = c0;
                t.rows = std::min(P->edge, g.rows - r0);
                t.cols = std::min(P->edge, g.cols - c0);
                tiles.push_back(t);
            }
    }
    P->n_tiles = (int)tiles.size();
    P->left_blk = p->left_blk;
    P->right_blk = p->right_blk;
    hipError_t e = hipSuccess;
    if (!tiles.empty()) {
        e = hipMalloc(&P->tiles, sizeof(SbTile) * tiles.size());
        if (e == hipSuccess) e = hipMalloc(&P->steps, sizeof(SbStep) * std::max<size_t>(steps.size(), 1));
        if (e == hipSuccess) e = hipMemcpy(P->tiles, tiles.data(), sizeof(SbTile) * tiles.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess && !steps.empty())
            e = hipMemcpy(P->steps, steps.data(), sizeof(SbStep) * steps.size(), hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        rot_sb_plan_destroy(P);
        return sberr(ROT_ERR_HIP, "rot_sb_plan_create: %s", hipGetErrorString(e));
    }
    *plan = P;
    return ROT_OK;
}

rot_status rot_sb_apply(rot_sb_plan plan, const double* psi, double* out, void* stream) {
    rot::TraceRange trace_("rot_sb_apply");
    if (!plan) return sberr(ROT_ERR_INVALID_ARG, "null plan");
    if (plan->total == 0) return ROT_OK;
    if (!psi || !out) return sberr(ROT_ERR_INVALID_ARG, "null psi or out");
    if (out < psi + plan->total && psi < out + plan->total) return sberr(ROT_ERR_INVALID_ARG, "out overlaps psi");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = prof_timed("sb_matvec", s, [&] {
        const dim3 grid((plan->n_tiles + 3) / 4), block(256);
        if (plan->edge == 32)
            hipLaunchKernelGGL(sb_tile_kernel<2>, grid, block, 0, s, plan->tiles, plan->n_tiles, plan->steps,
                               plan->left_blk, plan->right_blk, psi, out);
        else
            hipLaunchKernelGGL(sb_tile_kernel<1>, grid, block, 0, s, plan->tiles, plan->n_tiles, plan->steps,
                               plan->left_blk, plan->right_blk, psi, out);
        return hipGetLastError();
    });
    return e == hipSuccess ? ROT_OK : sberr(ROT_ERR_HIP, "rot_sb_apply: %s", hipGetErrorString(e));
}

double rot_sb_plan_flops(rot_sb_plan plan) { return plan ? plan->flops : 0.0; }

rot_status rot_sb_plan_destroy(rot_sb_plan plan) {
    if (!plan) return ROT_OK;
    if (plan->tiles) (void)hipFree(plan->tiles);
    if (plan->steps) (void)hipFree(plan->steps);
    delete plan;
    return ROT_OK;
}

}  // extern "C"
