// gfx950 kernels after the Lanczos loop (Sec. III, second phase): Jacobi on
// the tridiagonal T, Top-K selection, Ritz vectors, and the accuracy report
// of Sec. IV-D (residuals, orthogonality of the basis and of the Ritz
// vectors, mean pairwise angle).
#include <algorithm>
#include <cmath>

#include "lz_ooc.h"
#include "lz_spmv.h"

namespace lz {

constexpr int JMAX_SWEEPS = 60;
constexpr int JBLOCK = 1024;      // Jacobi workgroup: one round is a single parallel step

// ---------------------------------------------------------------- Jacobi
// Parallel cyclic Jacobi on one CU.  Each round applies half = me/2 disjoint
// rotations chosen by the round-robin tournament ordering (me = m rounded up
// to even; an odd m gets a zero dummy row and column that is never rotated);
// me-1 rounds make a sweep.  Rotation (Rutishauser): zeta = (t_qq - t_pp) /
// (2 t_pq), t = sgn(zeta)/(|zeta| + sqrt(1+zeta^2)), c = 1/sqrt(1+t^2),
// s = t c.  A rotation is skipped when |t_pq| is negligible (<= eps
// sqrt|t_pp t_qq| or <= eps^2 ||T||_F); the method stops at a sweep without
// rotations (counted, not run).
//
// What bounds it is the chain of me-1 rounds per sweep, each with one FP64
// rotation, two LDS round trips and barriers; the arithmetic is small.  So a
// round is arranged around that chain:
//   * T is stored by tournament slot, not by index: pair i is slots i (top)
//     and me-1-i (bottom), and after a round the contents of slot k move to
//     slot k-1 (slot 1 to me-1, slot 0 stays).  A thread owns one 2x2 block of
//     two pairs a < b for the whole solve: it reads the block and the two
//     rotations at fixed addresses and writes the four results to fixed
//     addresses of the other buffer, so no index table is looked up.
//   * The first wavefront holds the diagonal blocks.  While the others apply
//     round k it already computes the rotations of round k+1: the next pivot
//     of a pair is one element of one 2x2 block after round k (four products
//     of the old block with the two rotations), and the diagonal follows from
//     t_pp' = t_pp - t t_pq, t_qq' = t_qq + t t_pq.  A round then costs one
//     barrier.
//   * S' = S J stays in registers: a half wavefront holds a row, lane i the
//     columns of pair i, and the tournament's move is a lane shift (DPP).
//   * The rotation is two reciprocal square roots instead of three divisions
//     and two square roots: with d = t_qq - t_pp, r = 1/sqrt(d^2 + 4 t_pq^2),
//     c^2 = (1 + |d| r)/2, s c = |t_pq| r; the skip test compares squares.
//     Both need operands of bounded size, so T is scaled once by a power of
//     two (exactly) to a norm in [1, 2).
// Measured on MI355X, before (index tables, two barriers a round, the rotation
// in line) -> now: m = 16 96 -> 39 us, m = 48 480 -> 150 us, m = 64 863 -> 223 us
// (about 0.4 us a round).  One loop over the rounds for all three roles
// instead of a loop each kept 248 us at m = 48.
struct JacobiShared {
    double blk[2][(MMAX / 2) * (MMAX / 2 - 1) / 2 * 4 + 4];   // 2x2 blocks of pairs a < b; the last 4 take dropped writes
    double2 cs[2][MMAX / 2];       // (c, s) of every pair, top as p and bottom as q
    double dg[2][MMAX];            // diagonal after the round's rotation: [2i] top, [2i+1] bottom of pair i
    double dpre[MMAX];             // diagonal before it
    double theta[MMAX];
    int pend;
};

// 1/sqrt(h) to about an ulp: the hardware estimate and one third-order step.
__device__ __forceinline__ double rsqrt_refined(double h) {
    const double r = __builtin_amdgcn_rsq(h);
    const double e = fma(-(h * r), r, 1.0);
    return fma(r * e, fma(0.375, e, 0.5), r);
}

// The rotation of a pair (top p, bottom q; `flipped`: the top holds the larger
// index, which only matters for the sign where t_pp = t_qq).  The matrix is
// scaled to a norm in [1, 2), so the squares neither overflow nor, for a pivot
// that is not negligible, underflow.
__device__ __forceinline__ bool jacobi_negligible(double apq, double dd, double fro) {
    constexpr double eps = 1.1102230246251565e-16;
    return apq * apq <= eps * eps * fabs(dd) || fabs(apq) <= eps * eps * fro;
}
__device__ __forceinline__ bool jacobi_rotation(double app, double aqq, double apq, bool flipped, double fro,
                                                double2& cs, double& app2, double& aqq2) {
    const bool rot = !jacobi_negligible(apq, app * aqq, fro);
    const double d = aqq - app;
    const double r = rsqrt_refined(fma(d, d, 4.0 * (apq * apq)));
    const double c2 = fma(0.5 * fabs(d), r, 0.5);
    const double ci = rsqrt_refined(c2);
    const bool neg = d == 0.0 ? flipped != (apq < 0.0) : d < 0.0;
    const double s = ((neg ? -apq : apq) * r) * ci, t = s * ci;
    cs = rot ? make_double2(c2 * ci, s) : make_double2(1.0, 0.0);
    app2 = rot ? fma(-t, apq, app) : app;
    aqq2 = rot ? fma(t, apq, aqq) : aqq;
    return rot;
}

// Shifts by one lane of the wavefront (0 past its ends): lane i takes lane
// i + 1, lane i - 1.
__device__ __forceinline__ double lane_next(double x) { return dpp_move<0x130>(x); }
__device__ __forceinline__ double lane_prev(double x) { return dpp_move<0x138>(x); }

// A sweep of column rotations on the S rows of a wavefront: NS row pairs, lane
// hl of a half wavefront holding the top and bottom columns of pair hl.
constexpr int JS_ROWS = 5;           // row pairs per wavefront at most: 32 over at least 7 wavefronts
template <int NS>
__device__ __forceinline__ void jacobi_s_rounds(int rounds, int half, int hl, const JacobiShared& sh, int& buf,
                                                double (&top)[JS_ROWS], double (&bot)[JS_ROWS]) {
    const bool first = hl == 0, last = hl == half - 1, single = half == 1;
    const int hc = min(hl, half - 1);
    for (int round = 0; round < rounds; ++round) {
        const double2 cs = sh.cs[buf][hc];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const double tp = cs.x * top[q] - cs.y * bot[q], bt = cs.y * top[q] + cs.x * bot[q];
            // The tournament's move (none for a single pair).
            const double tn = lane_next(tp), bp = lane_prev(bt);
            top[q] = first ? tp : (last ? bt : tn);
            bot[q] = single ? bt : (first ? tn : bp);
        }
        buf ^= 1;
        __syncthreads();
    }
}

// Jacobi of the symmetric tridiagonal matrix diag[0..m), off[0..m-1): leaves
// the diagonal in sh.theta and S in Sout (row-major, stride MMAX); returns the
// sweep count, -1 past the limit.  Called by JBLOCK threads.
__device__ __forceinline__ int jacobi_core(int m, const double* diag, const double* off, JacobiShared& sh, double* Sout) {
    constexpr int DROP = (MMAX / 2) * (MMAX / 2 - 1) / 2 * 4;
    const int me = (m + 1) & ~1, half = me / 2;
    const int nblk = half * (half - 1) / 2;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // Norm and scale, by every wavefront for itself.
    const double dl = lane < m ? diag[lane] : 0.0, ol = lane + 1 < m ? off[lane] : 0.0;
    const double big = fmax(fabs(dl), fabs(ol));
    const int ex0 = __builtin_amdgcn_frexp_exp(wave_max(big));
    const double ds = ldexp(dl, -ex0), os = ldexp(ol, -ex0);
    const double fro0 = sqrt(wave_sum(ds * ds + 2.0 * os * os));
    const int ex = ex0 + __builtin_amdgcn_frexp_exp(fro0) - 1;
    const double fro = ldexp(fro0, ex0 - ex);
    auto diag_at = [&](int i) { return i < m ? ldexp(diag[i], -ex) : 0.0; };
    auto tri = [&](int i, int j) {
        return i < m && j < m && abs(i - j) == 1 ? ldexp(off[min(i, j)], -ex) : 0.0;
    };
    auto slot = [&](int pair, int e) { return e == 0 ? pair : me - 1 - pair; };
    auto moved = [&](int k) { return k == 0 ? 0 : (k == 1 ? me - 1 : k - 1); };
    auto block = [&](int a, int b) { return a * (2 * half - a - 1) / 2 + (b - a - 1); };
    // Where the element of slots u, v is stored after a round (DROP: in a
    // diagonal block, which the first wavefront holds).
    auto target = [&](int u, int v) {
        const int mu = moved(u), mv = moved(v);
        const int pu = mu < half ? mu : me - 1 - mu, eu = mu < half ? 0 : 1;
        const int pv = mv < half ? mv : me - 1 - mv, ev = mv < half ? 0 : 1;
        if (pu == pv) return DROP;
        return pu < pv ? block(pu, pv) * 4 + eu * 2 + ev : block(pv, pu) * 4 + ev * 2 + eu;
    };
    const int twaves = (nblk + 63) / 64;                   // wavefronts 1 .. twaves: blocks; the rest: rows of S
    const bool is_rot = wave == 0, is_blk = !is_rot && wave <= twaves;
    const int sw = wave - 1 - twaves, nsw = JBLOCK / 64 - 1 - twaves;

    // Per-role constants and state.
    int ba = 0, bb = 0, bi = 0, dst[4] = {DROP, DROP, DROP, DROP};     // block threads
    bool live = false;
    int pa = 0, ea = 0, pb = 0, eb = 0, top_src = 0, bot_src = 0, piv_dst = DROP, itop = 0, ibot = 0;   // rotations
    double app = 0.0, aqq = 0.0, apq = 0.0, pivot_left = 0.0;
    bool rot = false;
    double st_[JS_ROWS], sb_[JS_ROWS];                         // S rows: columns of the top and bottom of pair `lane`
    if (is_blk) {
        bi = tid - 64;
        live = bi < nblk;
        if (live) {
            int rest = bi;
            while (rest >= half - 1 - ba) rest -= half - 1 - ba++;
            bb = ba + 1 + rest;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int u = slot(ba, e >> 1), v = slot(bb, e & 1);
                dst[e] = target(u, v);
                sh.blk[0][bi * 4 + e] = tri(u, v);
            }
        }
    }
    if (is_rot) {
        live = lane < half;
        const int i = live ? lane : 0;
        if (half > 1) {
            const bool last = i == half - 1;
            pa = i == 0 ? 0 : i - 1;
            ea = i == 0 ? 0 : 1;
            pb = last ? half - 1 : i + 1;
            eb = i == 0 || !last ? 0 : 1;
            top_src = i == 0 ? 0 : (last ? 2 * (half - 1) + 1 : 2 * (i + 1));
            bot_src = i == 0 ? 2 : 2 * (i - 1) + 1;
        }
        piv_dst = live ? target(slot(i, 0), slot(i, 1)) : DROP;
        itop = i;
        ibot = me - 1 - i;
        app = diag_at(itop);
        aqq = diag_at(ibot);
        apq = tri(itop, ibot);
        double2 cs;
        double a2, q2;
        rot = jacobi_rotation(app, aqq, apq, itop > ibot, fro, cs, a2, q2);
        pivot_left = rot ? 0.0 : apq;
        if (live) {
            sh.cs[0][lane] = cs;
            sh.dg[0][2 * lane] = a2;
            sh.dg[0][2 * lane + 1] = q2;
            sh.dpre[2 * lane] = app;
            sh.dpre[2 * lane + 1] = aqq;
        }
        if (tid == 0) sh.pend = 0;
    }
    const int hl = lane & 31;                              // pair held by a lane of an S row
#pragma unroll
    for (int q = 0; q < JS_ROWS; ++q) {
        const int r = 2 * (sw + q * nsw) + (lane >> 5);
        st_[q] = r == hl ? 1.0 : 0.0;
        sb_[q] = r == me - 1 - hl ? 1.0 : 0.0;
    }
    const int nsets = sw < 0 ? 0 : (half - sw + nsw - 1) / nsw;   // half = me/2 row pairs in all
    const int b4 = half > 1 ? block(pa, pb) * 4 : 0;
    if (is_rot) __builtin_amdgcn_s_setprio(3);

    int buf = 0, sweeps = -1;
    __syncthreads();
    for (int sweep = 1; sweep <= JMAX_SWEEPS; ++sweep) {
        // A sweep rotates nothing exactly when every pair already passes the
        // skip test at its start (T does not change within such a sweep), so
        // that sweep is detected here instead of being run.  The layout at the
        // start of a sweep is the identity.
        bool pending = false;
        if (is_rot) {
            pending = live && rot && m > 1;      // (m = 1: the only pair is with the dummy row, which a NaN would rotate)
        } else if (is_blk && live) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double dd = sh.dpre[2 * ba + (e >> 1)] * sh.dpre[2 * bb + (e & 1)];
                pending |= !jacobi_negligible(sh.blk[buf][bi * 4 + e], dd, fro);
            }
        }
        if (pending) sh.pend = sweep;
        __syncthreads();
        if (sh.pend != sweep) {
            sweeps = sweep;
            break;
        }
        // Each role runs its own loop over the rounds (the branch is uniform
        // in a wavefront), so its addresses and registers stay put.
        const int rounds = me - 1;
        if (is_rot) {
            // Next round's rotations from this round's, the old blocks and the
            // rotated diagonal.
            for (int round = 0; round < rounds; ++round) {
                const int nx = buf ^ 1;
                if (half > 1) {
                    const double2 ca = sh.cs[buf][pa], cb = sh.cs[buf][pb];
                    const double2 t0 = *(const double2*)&sh.blk[buf][b4], t1 = *(const double2*)&sh.blk[buf][b4 + 2];
                    app = sh.dg[buf][top_src];
                    aqq = sh.dg[buf][bot_src];
                    if (live) sh.blk[nx][piv_dst] = pivot_left;
                    const double ra0 = ea == 0 ? ca.x : ca.y, ra1 = ea == 0 ? -ca.y : ca.x;
                    const double rb0 = eb == 0 ? cb.x : cb.y, rb1 = eb == 0 ? -cb.y : cb.x;
                    const double u0 = fma(ra0, t0.x, ra1 * t1.x), u1 = fma(ra0, t0.y, ra1 * t1.y);
                    apq = fma(rb0, u0, rb1 * u1);
                    itop = itop == 0 ? 0 : (itop == rounds ? 1 : itop + 1);
                    ibot = ibot == rounds ? 1 : ibot + 1;
                } else {
                    app = sh.dg[buf][0];
                    aqq = sh.dg[buf][1];
                    apq = pivot_left;
                }
                double2 cs;
                double a2, q2;
                rot = jacobi_rotation(app, aqq, apq, itop > ibot, fro, cs, a2, q2);
                pivot_left = rot ? 0.0 : apq;
                if (live) {
                    sh.cs[nx][lane] = cs;
                    *(double2*)&sh.dg[nx][2 * lane] = make_double2(a2, q2);
                    if (round == rounds - 1) *(double2*)&sh.dpre[2 * lane] = make_double2(app, aqq);
                }
                buf = nx;
                __syncthreads();
            }
        } else if (is_blk) {
            for (int round = 0; round < rounds; ++round) {
                const int nx = buf ^ 1;
                if (live) {
                    const double2 ca = sh.cs[buf][ba], cb = sh.cs[buf][bb];
                    const double2 t0 = *(const double2*)&sh.blk[buf][bi * 4],
                                  t1 = *(const double2*)&sh.blk[buf][bi * 4 + 2];
                    const double u00 = ca.x * t0.x - ca.y * t1.x, u01 = ca.x * t0.y - ca.y * t1.y;
                    const double u10 = ca.y * t0.x + ca.x * t1.x, u11 = ca.y * t0.y + ca.x * t1.y;
                    double* out = sh.blk[nx];
                    out[dst[0]] = cb.x * u00 - cb.y * u01;
                    out[dst[1]] = cb.y * u00 + cb.x * u01;
                    out[dst[2]] = cb.x * u10 - cb.y * u11;
                    out[dst[3]] = cb.y * u10 + cb.x * u11;
                }
                buf = nx;
                __syncthreads();
            }
        } else {
            switch (nsets) {
                case 0:
                    for (int round = 0; round < rounds; ++round) __syncthreads();
                    buf ^= rounds & 1;
                    break;
                case 1: jacobi_s_rounds<1>(rounds, half, hl, sh, buf, st_, sb_); break;
                case 2: jacobi_s_rounds<2>(rounds, half, hl, sh, buf, st_, sb_); break;
                case 3: jacobi_s_rounds<3>(rounds, half, hl, sh, buf, st_, sb_); break;
                case 4: jacobi_s_rounds<4>(rounds, half, hl, sh, buf, st_, sb_); break;
                default: jacobi_s_rounds<JS_ROWS>(rounds, half, hl, sh, buf, st_, sb_); break;
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);
    if (is_rot && live) {
        sh.theta[lane] = ldexp(app, ex);
        sh.theta[me - 1 - lane] = ldexp(aqq, ex);
    }
#pragma unroll
    for (int q = 0; q < JS_ROWS; ++q) {
        const int r = 2 * (sw + q * nsw) + (lane >> 5);
        if (q < nsets && r < m && hl < half) {
            Sout[r * MMAX + hl] = st_[q];
            if (me - 1 - hl < m) Sout[r * MMAX + me - 1 - hl] = sb_[q];
        }
    }
    __syncthreads();
    return sweeps;
}

// T from alpha_1..alpha_m and beta_2..beta_m, Jacobi, Top-K selection by
// modulus (ties: larger value, then lower index); writes the eigenvalues.
// A solve that completed fewer than m steps (breakdowns took some of the
// enqueued iterations) ends as `strict` says (STRICT_*).
__global__ __launch_bounds__(JBLOCK) void k_jacobi_select(State* st, double* out_vals, int strict) {
    __shared__ JacobiShared sh;
    if (st->status != 0) return;
    if (strict != STRICT_NO && st->j < st->m) {
        if (threadIdx.x == 0) st->status = strict == STRICT_PENDING ? 1 : -9;   // LZ_PENDING, LZ_ERR_RESTART_BUDGET
        return;
    }
    const int m = min(st->j, st->m);
    const int K = st->K;
    if (m < K) {
        if (threadIdx.x == 0) st->status = -8;
        return;
    }
    const int sweeps = jacobi_core(m, st->alpha, st->beta + 1, sh, st->S);
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        const double ti = sh.theta[i];
        st->theta[i] = ti;
        int rank = 0;
#pragma unroll 8
        for (int k = 0; k < m; ++k) {
            const double tk = sh.theta[k];
            rank += fabs(tk) > fabs(ti) || (fabs(tk) == fabs(ti) && (tk > ti || (tk == ti && k < i)));
        }
        if (rank < K) {
            st->sel[rank] = i;
            if (out_vals) out_vals[rank] = ti;
        }
    }
    if (threadIdx.x == 0) {
        st->sweeps = sweeps;
        if (sweeps < 0) st->status = -6;       // LZ_ERR_NOT_CONVERGED
    }
}

// Standalone tridiagonal eigensolve (component entry point).
__global__ __launch_bounds__(JBLOCK) void k_jacobi_only(const double* alpha, const double* offd, int m, State* st) {
    __shared__ JacobiShared sh;
    const int sweeps = jacobi_core(m, alpha, offd, sh, st->S);
    for (int i = threadIdx.x; i < m; i += blockDim.x) st->theta[i] = sh.theta[i];
    if (threadIdx.x == 0) {
        st->sweeps = sweeps;
        st->status = sweeps < 0 ? -6 : 0;
    }
}

// ------------------------------------------------------------ Ritz vectors
// Joins (norm, entry of largest modulus) over rows; the lowest original row
// wins among equal moduli.  NOROW marks "no row yet" (exact as a double and
// as an int64).
constexpr int64_t NOROW = int64_t(1) << 62;
struct ColStat {
    double nrm, mod, val;     // sum of squares; largest modulus and its value
    int64_t row;              // its original row
};
__device__ __forceinline__ void join(ColStat& a, double nrm, double mod, double val, int64_t row) {
    a.nrm += nrm;
    if (mod > a.mod || (mod == a.mod && row < a.row)) {
        a.mod = mod;
        a.val = val;
        a.row = row;
    }
}
// Over the lanes with the same lane % kb (a power of two), pairwise.
__device__ __forceinline__ void join_lanes(ColStat& a, int kb) {
    for (int o = kb; o < 64; o <<= 1) {
        const double nrm = __shfl_xor(a.nrm, o, 64), mod = __shfl_xor(a.mod, o, 64), val = __shfl_xor(a.val, o, 64);
        const int64_t row = __shfl_xor((long long)a.row, o, 64);
        join(a, nrm, mod, val, row);
    }
}

// Y[r][k] = sum_i scale_i V[r,i] S[i, sel_k]  (eigenvectors of the matrix are
// the Lanczos basis times those of T).  Y is row-major n x K (a K-wide row
// per matrix row, the layout the residual SpMM gathers), not normalised.
// And per Ritz column: norm and the entry of largest modulus (lowest original
// row on ties) -> ysc[k] = sign(that entry) / norm.
// A wavefront takes 64 rows on the FP64 matrix cores: lane l loads rows 4 (l %
// 16) .. + 3 of basis column 4 q + l/16 as one vector, product e of step q
// takes the e-th of them, and the result's 16 columns leave as one contiguous
// piece per row.  Bound by the basis' bytes and Y's.  The original row is
// looked up only where moduli tie and for the winners.  (One thread per row
// with K serial stores took 125 us at R-MAT 20, m = 48, K = 16, and a pass
// over Y for the column values 49 us; together 84 us.  R-MAT 25: 1.87 +
// 0.37 -> 1.45 ms.)
template <int P, int NB>
__global__ __launch_bounds__(BLOCK) void k_ritz(State* st, const typename Tr<P>::V* __restrict__ Vb, int64_t n,
                                                int64_t ld, double* __restrict__ Y, double* part) {
    using VT = typename Tr<P>::V;
    typedef VT V4 __attribute__((ext_vector_type(4)));
    typedef double d4 __attribute__((ext_vector_type(4)));
    constexpr int KC = NB * 16, KP = NB == 1 ? 16 : NB == 2 ? 32 : 64, U = P == 0 ? 4 : 6;
    __shared__ double Ss[MMAX][KC];
    __shared__ ColStat sw[WAVES][64];
    __shared__ int s_last;
    if (st->status != 0) return;
    const int m = min(st->j, st->m), K = st->K, G = gridDim.x;
    for (int idx = threadIdx.x; idx < MMAX * KC; idx += BLOCK) {
        const int i = idx / KC, k = idx % KC;
        Ss[i][k] = (i < m && k < K) ? st->S[i * MMAX + st->sel[k]] * st->scale[i] : 0.0;
    }
    __syncthreads();
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, cl = lane & 15, rg = lane >> 4;
    const int32_t* perm = st->perm;
    auto original = [&](int64_t r) { return perm ? (int64_t)perm[r] : r; };
    ColStat a[NB];
    int64_t best[NB];                              // row of the largest modulus so far, in the solve's order
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        a[b] = ColStat{0.0, -1.0, 0.0, NOROW};
        best[b] = -1;
    }
    // ld is a multiple of 64 past n, so whole vectors can be loaded.
    for (int64_t r0 = ((int64_t)blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(wv)) * 64; r0 < n;
         r0 += (int64_t)G * WAVES * 64) {
        d4 acc[4][NB];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[e][b] = d4{0.0, 0.0, 0.0, 0.0};
        const VT* x = Vb + r0 + cl * 4;
        for (int i0 = 0; i0 < m; i0 += 4 * U) {
            V4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *(const V4*)(x + (int64_t)min(i0 + u * 4 + rg, m - 1) * ld);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * 4 >= m) break;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const double s = Ss[i0 + u * 4 + rg][b * 16 + cl];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[e][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(to_d(VT(v[u][e])), s, acc[e][b], 0, 0, 0);
                }
            }
        }
        // Element t of lane l in acc[e]: row r0 + 4 (4 t + l/16) + e, column 16 b + l%16.
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t r = r0 + (t * 4 + rg) * 4 + e;
                if (r < n)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const int k = b * 16 + cl;
                        if (k < K) {
                            const double y = acc[e][b][t], mod = fabs(y);
                            Y[r * K + k] = y;
                            a[b].nrm += y * y;
                            if (mod > a[b].mod || (mod == a[b].mod && original(r) < original(best[b]))) {
                                a[b].mod = mod;
                                a[b].val = y;
                                best[b] = r;
                            }
                        }
                    }
            }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (best[b] >= 0) a[b].row = original(best[b]);
        join_lanes(a[b], 16);
        if (lane < 16) sw[wv][b * 16 + lane] = a[b];
    }
    __syncthreads();
    const int k = threadIdx.x % KP, g = threadIdx.x / KP, groups = BLOCK / KP;
    if ((int)threadIdx.x < K) {
        ColStat c = sw[0][k];
        for (int w = 1; w < WAVES; ++w) join(c, sw[w][k].nrm, sw[w][k].mod, sw[w][k].val, sw[w][k].row);
        double* pb = part + ((int64_t)blockIdx.x * 64 + k) * 4;
        st_dev(pb + 0, c.nrm);
        st_dev(pb + 1, c.mod);
        st_dev(pb + 2, c.val);
        st_dev(pb + 3, (double)c.row);
    }
    if (!last_block(&st->ticket[TK_RITZ], (uint32_t)G, &s_last)) return;
    // Thread (g, k) joins workgroups g, g + groups, ... of column k, four
    // loads in flight (past the end: the last one's, not joined).
    ColStat c{0.0, -1.0, 0.0, NOROW};
    if (k < K)
        for (int b = g; b < G; b += 4 * groups) {
            double v[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double* pb = part + ((int64_t)min(b + i * groups, G - 1) * 64 + k) * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[i][q] = ld_dev(pb + q);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + i * groups < G) join(c, v[i][0], v[i][1], v[i][2], (int64_t)v[i][3]);
        }
    join_lanes(c, KP);
    __syncthreads();
    if (lane < KP) sw[wv][lane] = c;
    __syncthreads();
    if ((int)threadIdx.x < K) {
        for (int w = 1; w < WAVES; ++w) join(c, sw[w][k].nrm, sw[w][k].mod, sw[w][k].val, sw[w][k].row);
        st->ysc[k] = (c.val < 0.0 ? -1.0 : 1.0) / sqrt(c.nrm);
    }
}

// Residual check (Sec. IV-D) in FP64 for all K Ritz pairs at once.
// First Z = A Y (stored matrix values upcast exactly) over the SpMV tiles:
// each wavefront stages its tile's col/val in LDS in row order (values in the
// storage precision, upcast when used); lane k of a group of KB2 lanes owns
// pair k and gathers K-wide rows of Y.  The tile's entries are split evenly
// over the 64/KB2 groups, whatever rows they belong to: a group keeps SPMM_U
// gathers in flight and closes a row where the column word carries its mark.
// (By rows, a group had at most the eight gathers of one row in flight, and a
// long row kept three of four groups waiting: R-MAT 20 K = 16 FP32 / FP64 558 /
// 686 -> 290 / 410 us, R-MAT 150k FP64 142 -> 50 us, R-MAT 23 K = 24 BF16 11.7 ->
// 7.9 ms, R-MAT 25 K = 8 FP32 18.7 -> 16.6 ms; ER 500k FP32, whose gathers all
// miss L2, 174 -> 172 us.)  Rows cut by a group's bounds are joined in group order,
// rows cut by tile bounds by their last piece as in the SpMV, the pieces added
// in tile order.
// Gathers per lane of 8 / 12 / 16 / 24: finish of R-MAT 20 FP32 0.99 / 0.98 /
// 1.03 / 1.02 ms, R-MAT 25 FP32 24.97 / 25.01 / 25.44 / 25.47 ms.
constexpr int SPMM_U = 12;
constexpr int SPMM_END = (int)0x80000000;      // mark of a row's last entry

// Adds the groups' values (lanes that differ in the group bits), fixed order.
__device__ __forceinline__ double group_sum(double v, int KB2) {
    for (int o = KB2; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The matrix arrays come in as kernel arguments (the caller's CSR and the
// relabelled copy), so their loads are global loads, as in the step SpMV.
template <int P>
__global__ __launch_bounds__(BLOCK) void k_spmm(State* st, const double* __restrict__ Y, double* __restrict__ Z,
                                                int64_t n, int64_t nnz, int64_t n_tiles, const int32_t* __restrict__ ob,
                                                uint32_t* tk, double* head, double* tail, int KB2,
                                                const int64_t* rp_a, const int32_t* col_a, const void* val_a,
                                                const int64_t* rp_b, const int32_t* col_b, const void* val_b,
                                                int64_t tb, int64_t te) {
    using VT = typename Tr<P>::V;
    __shared__ int scol_all[WAVES][TILE];
    __shared__ VT sval_all[WAVES][TILE];
    __shared__ uint16_t srow_all[WAVES][TILE];
    if (st->status != 0) return;
    const bool rl = st->reordered != 0;
    const int packing = rl ? st->packed : PACK_NONE;
    const int64_t* rp = rl ? rp_b : rp_a;
    const int32_t* col = rl ? col_b : col_a;
    const VT* val = (const VT*)(rl ? val_b : val_a);
    const int K = st->K;
    const int lane = threadIdx.x & 63;
    const int G = 64 / KB2, g = lane / KB2, k = lane % KB2;
    const bool act = k < K;
    int* scol = scol_all[threadIdx.x >> 6];
    VT* sval = sval_all[threadIdx.x >> 6];
    uint16_t* srow = srow_all[threadIdx.x >> 6];
    // Pieces of split row r (tail pieces in t1..t2-1, head piece in t2),
    // added group-strided in tile order; the whole row sum in every group.
    auto split_total_k = [&](int64_t t1, int64_t t2) {
        double z = 0.0;
        if (act)
            for (int64_t i = t1 + g; i < t2; i += G) z += ld_dev(&tail[i * KB2 + k]);
        z = group_sum(z, KB2);
        return act ? z + ld_dev(&head[t2 * KB2 + k]) : 0.0;
    };
    // Rows of tile t from its entries in row order, scol/sval[0..cnt).
    auto tile_body = [&](int64_t t, int* scol, const VT* sval, uint16_t* srow) {
        const int64_t r_lo = ob[t], r_hi = ob[t + 1];
        const int64_t t0 = t * TILE - r_lo;
        const int cnt = (int)(min<int64_t>((t + 1) * TILE, nnz + n) - r_hi - t0);
        const int64_t rb_lo = r_lo < n ? rp[r_lo] : 0, rb_hi = r_hi < n ? rp[r_hi] : 0,
                      re_hi = r_hi < n ? rp[r_hi + 1] : 0;
        const bool split_head = r_lo < r_hi && rb_lo < t0, split_tail = r_hi < n && rb_hi < t0 + cnt;
        // Mark every owned row's last entry; rows without entries are zero.
        for (int64_t base = r_lo; base < r_hi; base += 64) {
            const int64_t r = base + lane;
            bool empty = false;
            if (r < r_hi) {
                const int b = (int)(max(rp[r], t0) - t0), e = (int)(rp[r + 1] - t0);
                if (e > b) {
                    scol[e - 1] |= SPMM_END;
                    srow[e - 1] = (uint16_t)(r - r_lo);
                } else {
                    empty = !(split_head && r == r_lo);
                }
            }
            const uint64_t mask = __ballot(empty);
            if (mask)
                for (int i = g; i < 64; i += G)
                    if (((mask >> i) & 1) && act) Z[(base + i) * K + k] = 0.0;
        }
        wave_sync();
        // Group g takes entries [lo, hi).  The first row it closes may have
        // begun in an earlier group: its sum waits in first_z, that of the row
        // left open in acc.
        const int S = (cnt + G - 1) / G, lo = min(g * S, cnt), hi = min(lo + S, cnt);
        double acc = 0.0, first_z = 0.0;
        int first_row = -1;
        for (int p = lo; p < hi; p += SPMM_U) {
            int w[SPMM_U];
            double y[SPMM_U];
#pragma unroll
            for (int i = 0; i < SPMM_U; ++i) w[i] = scol[min(p + i, hi - 1)];
#pragma unroll
            for (int i = 0; i < SPMM_U; ++i) y[i] = act ? Y[(int64_t)(w[i] & ~SPMM_END) * K + k] : 0.0;
#pragma unroll
            for (int i = 0; i < SPMM_U; ++i) {
                if (p + i < hi) {
                    acc = fma(to_d(sval[p + i]), y[i], acc);
                    if (w[i] < 0) {
                        const int row = srow[p + i];
                        if (first_row < 0) {
                            first_row = row;
                            first_z = acc;
                        } else if (act) {
                            Z[(r_lo + row) * K + k] = acc;
                        }
                        acc = 0.0;
                    }
                }
            }
        }
        // Rows across the groups, in group order; every lane follows its pair.
        double carry = 0.0, head_z = 0.0;
        for (int gg = 0; gg < G; ++gg) {
            const int row = lane_value(first_row, gg * KB2);
            const double open = __shfl(acc, gg * KB2 + k, 64);
            if (row >= 0) {
                const double z = carry + __shfl(first_z, gg * KB2 + k, 64);
                if (split_head && row == 0)
                    head_z = z;
                else if (g == 0 && act)
                    Z[(r_lo + row) * K + k] = z;
                carry = open;
            } else {
                carry += open;
            }
        }
        if (!split_head && !split_tail) return;
        // Pieces of split rows: published together, tickets taken together.
        const int64_t h1 = split_head ? item_tile(rb_lo + r_lo, n_tiles) : 0;
        const int64_t t1 = split_tail ? item_tile(rb_hi + r_hi, n_tiles) : 0;
        const int64_t t2 = split_tail ? item_tile(re_hi + r_hi, n_tiles) : 0;
        if (g == 0 && act) {
            if (split_head) st_dev(&head[t * KB2 + k], head_z);
            if (split_tail) st_dev(&tail[t * KB2 + k], carry);
        }
        __builtin_amdgcn_s_waitcnt(0);
        uint32_t got = 0;
        if ((lane == 0 && split_head) || (lane == 1 && split_tail))
            got = __hip_atomic_fetch_add(lane == 0 ? &tk[t] : &tk[t2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (split_head && (uint32_t)lane_value((int)got, 0) == (uint32_t)(t - h1)) {
            if (lane == 0) __hip_atomic_store(&tk[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double z = split_total_k(h1, t);
            if (g == 0 && act) Z[r_lo * K + k] = z;
        }
        if (split_tail && (uint32_t)lane_value((int)got, 1) == (uint32_t)(t2 - t1)) {
            if (lane == 0) __hip_atomic_store(&tk[t2], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double z = split_total_k(t1, t2);
            if (g == 0 && act) Z[r_hi * K + k] = z;
        }
    };
    if (packing == PACK_GROUP) {
        // Group-sorted storage: the workgroup puts a group's entries back in
        // row order in its LDS, then each wavefront takes its tile.
        static_assert(WAVES == GROUP_TILES, "one wavefront per tile of a group");
        int* gcol = &scol_all[0][0];
        VT* gval = &sval_all[0][0];
        const int w = threadIdx.x >> 6;
        const int64_t n_groups = (n_tiles + GROUP_TILES - 1) / GROUP_TILES;
        const int64_t xcd = blockIdx.x & 7, nb8 = gridDim.x >> 3;
        const int64_t lo = n_groups * xcd / 8, hi = n_groups * (xcd + 1) / 8;
        for (int64_t gi = lo + (blockIdx.x >> 3); gi < hi; gi += nb8) {
            const int64_t tg = gi * GROUP_TILES, tend = min<int64_t>(tg + GROUP_TILES, n_tiles);
            const int64_t g0 = tg * TILE - ob[tg];
            const int64_t gend = tend >= n_tiles ? nnz : tend * TILE - ob[tend];
            for (int64_t i = threadIdx.x; i < gend - g0; i += BLOCK) {
                const uint32_t cw = (uint32_t)col[g0 + i];
                const int sl = (int)(cw & GROUP_SLOTMASK);
                gcol[sl] = (int)(cw >> GROUP_SLOTBITS);
                gval[sl] = val[g0 + i];
            }
            __syncthreads();
            const int64_t t = tg + w;
            if (t < n_tiles) {
                const int off = (int)(t * TILE - ob[t] - g0);
                tile_body(t, gcol + off, gval + off, &srow_all[0][0] + off);
            }
            __syncthreads();
        }
        return;
    }
    const TileRange tr = wave_tiles(tb, te);
    for (int64_t t = tr.first; t < tr.end; t += tr.stride) {
        const int64_t r_lo = ob[t], r_hi = ob[t + 1];
        const int64_t t0 = t * TILE - r_lo;
        const int cnt = (int)(min<int64_t>((t + 1) * TILE, nnz + n) - r_hi - t0);
        // A tile-sorted tile goes back to row order in LDS.
        for (int i = lane; i < cnt; i += 64) {
            const uint32_t cw = (uint32_t)col[t0 + i];
            const int sl = packing == PACK_TILE ? (int)(cw & PACK_SLOTMASK) : i;
            scol[sl] = packing == PACK_TILE ? (int)(cw >> PACK_SLOTBITS) : (int)cw;
            sval[sl] = val[t0 + i];
        }
        wave_sync();
        tile_body(t, scol, sval, srow);
        wave_sync();
    }
}

// -------------------------------------------------------- orthogonality
// Gram matrices on the FP64 matrix cores (v_mfma_f64_16x16x4f64), straight from
// global memory: lane l holds rows 4 (l/16) .. + 3 of column 16 b + l%16 of
// every column block b, so its four products per block pair take row 4 (l/16)
// + e in step e, the same rows for both operands, whatever their order in the
// sum.  Each element is loaded once; there is nothing to stage in LDS.  (The
// LDS-panel form took 117 us on the R-MAT 20 FP32 basis of 48 columns, 2.3 ms at
// R-MAT 25 with 32 columns; this one 73 us and 1.2 ms, 2.7 and 3.6 TB/s.)
// A workgroup adds its wavefronts' blocks in LDS and writes the upper block
// pairs to gpart[workgroup][pair][16 x 16]; k_gram_finish adds the workgroups.
typedef double d4 __attribute__((ext_vector_type(4)));

// acc of the block pairs -> gp[pair * 256 + i * 16 + j] (element e of lane l
// holds D[4e + l/16][l % 16]), wavefronts in order.
template <int NP>
__device__ __forceinline__ void gram_store(const d4 (&acc)[NP], double* gp) {
    __shared__ double sh[NP][256];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int w = 0; w < WAVES; ++w) {
        if (wv == w)
#pragma unroll
            for (int t = 0; t < NP; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double* d = &sh[t][(e * 4 + (lane >> 4)) * 16 + (lane & 15)];
                    *d = w == 0 ? acc[t][e] : *d + acc[t][e];
                }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < NP * 256; i += BLOCK) gp[i] = sh[i / 256][i % 256];
}

// Basis: X column-major with c <= 16 NB columns, column k scaled by scale[k].
template <class T, int NB>
__global__ __launch_bounds__(BLOCK) void k_gram(const State* st, const T* __restrict__ X, int64_t ldx, int64_t n,
                                                double* __restrict__ gpart) {
    constexpr int NP = NB * (NB + 1) / 2;
    typedef T T4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    if (st->status != 0) return;
    const int c = min(st->j, st->m);
    if (c < 1 || c > 16 * NB) return;
    const int lane = threadIdx.x & 63, cl = lane & 15, rg = lane >> 4;
    double sc[NB];
    const T* xb[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int k = b * 16 + cl;
        sc[b] = k < c ? st->scale[k] : 0.0;        // columns past c enter as zeros
        xb[b] = X + (int64_t)min(k, c - 1) * ldx + rg * 4;
    }
    d4 acc[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    const int64_t step = (int64_t)gridDim.x * WAVES * 32;
    for (int64_t r0 = ((int64_t)blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 32; r0 < n;
         r0 += step) {
        T4 v[2][NB];
        if (r0 + 32 <= n) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < NB; ++b) v[h][b] = *(const T4*)(xb[b] + r0 + h * 16);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int64_t r = r0 + h * 16 + rg * 4 + e;
                        v[h][b][e] = r < n ? xb[b][r0 + h * 16 + e] : T(0);
                    }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double x[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) x[b] = to_d(T(v[h][b][e])) * sc[b];
#pragma unroll
                for (int bi = 0, t = 0; bi < NB; ++bi)
#pragma unroll
                    for (int bj = bi; bj < NB; ++bj, ++t)
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[bi], x[bj], acc[t], 0, 0, 0);
            }
    }
    gram_store<NP>(acc, gpart + (int64_t)blockIdx.x * GRAM_SLOT);
}

// Unit Ritz vectors y_k = ysc_k Y[:,k] into the caller's column-major output
// in original row order and, with REPORT, in the same pass over Y and Z (both
// row-major, n x K) the residuals ||A y_k - theta_k y_k|| = ||ysc_k Z[:,k] -
// theta_k ysc_k Y[:,k]|| (Sec. IV-D) and the Gram matrix of the unit vectors.
// A wavefront takes 4 U rows on its own: lane l gathers columns 16 b + l%16 of
// rows l/16, l/16 + 4, ... (through the original-to-solve row map when the
// matrix was relabelled; the next rows' map entries are loaded ahead), which are
// the operands of the FP64 matrix cores, and the rows leave column-wise
// through LDS.  Bound by the bytes of Y, Z and the output.  Sums of squares go
// to rpart[workgroup * 64 + column].  (R-MAT 20, K = 16: output 99 us and
// residual with Gram 48 us as separate passes; together 86 us.  R-MAT 25, K
// = 8: 1.55 + 0.84 -> 2.02 ms.)
template <int NB, bool REPORT>
__global__ __launch_bounds__(BLOCK) void k_out(const State* st, const double* __restrict__ Y,
                                               const double* __restrict__ Z, int64_t n, double* __restrict__ out,
                                               double* __restrict__ gpart, double* __restrict__ rpart) {
    constexpr int NP = NB * (NB + 1) / 2, U = NB <= 2 ? 8 : 4, R = 4 * U;
    __shared__ double ys[WAVES][R][NB * 16 + 1];
    __shared__ double shr[WAVES][NB * 16];
    if (st->status != 0) return;
    const int K = st->K;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, cl = lane & 15, rg = lane >> 4;
    const int32_t* __restrict__ iperm = st->iperm;
    double ysc[NB], th[NB], racc[NB];
    int kc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int k = b * 16 + cl;
        const bool act = k < K;
        ysc[b] = act ? st->ysc[k] : 0.0;
        th[b] = REPORT && act ? st->theta[st->sel[k]] : 0.0;
        kc[b] = min(k, K - 1);
        racc[b] = 0.0;
    }
    d4 acc[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    const int64_t step = (int64_t)gridDim.x * WAVES * R;
    int64_t r0 = ((int64_t)blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(wv)) * R;
    int64_t src[U];
    auto rows = [&](int64_t base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = min(base + u * 4 + rg, n - 1);
            src[u] = iperm ? (int64_t)iperm[r] : r;
        }
    };
    rows(r0);
    for (; r0 < n; r0 += step) {
        double y[U][NB], z[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                y[u][b] = Y[src[u] * K + kc[b]];
                if (REPORT) z[u][b] = Z[src[u] * K + kc[b]];
            }
        rows(r0 + step);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = r0 + u * 4 + rg < n;
            double x[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const double v = ysc[b] * y[u][b];
                ys[wv][u * 4 + rg][b * 16 + cl] = v;
                x[b] = in ? v : 0.0;
                if (REPORT) {
                    const double d = in ? ysc[b] * z[u][b] - th[b] * v : 0.0;
                    racc[b] += d * d;
                }
            }
            if (REPORT)
#pragma unroll
                for (int bi = 0, t = 0; bi < NB; ++bi)
#pragma unroll
                    for (int bj = bi; bj < NB; ++bj, ++t)
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[bi], x[bj], acc[t], 0, 0, 0);
        }
        // The wavefront's own rows: its LDS accesses stay in order.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int row = lane % R;
        if (r0 + row < n)
            for (int k = lane / R; k < K; k += 64 / R) out[(int64_t)k * n + r0 + row] = ys[wv][row][k];
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (!REPORT) return;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        racc[b] = add_xor_rows<32>(add_xor_rows<16>(racc[b]));
        if (lane < 16) shr[wv][b * 16 + lane] = racc[b];
    }
    __syncthreads();
    gram_store<NP>(acc, gpart + (int64_t)blockIdx.x * GRAM_SLOT);
    if ((int)threadIdx.x < NB * 16) {
        double s = shr[0][threadIdx.x];
        for (int w = 1; w < WAVES; ++w) s += shr[w][threadIdx.x];
        rpart[(int64_t)blockIdx.x * 64 + threadIdx.x] = s;
    }
}

// Adds the workgroups' partials, one wavefront per value (lane-strided, then
// the wavefront sum: a fixed order): the upper entries of the basis' Gram
// matrix (gv workgroups), those of the Ritz vectors' and the residuals' sums
// of squares (gy workgroups; 0: basis only).  The last workgroup takes max
// |G - I| of both, the mean angle between Ritz vectors and the residuals.
__device__ __forceinline__ int gram_place(int i, int j, int nb) {
    const int bi = i >> 4, bj = j >> 4;
    return (bi * (2 * nb - bi + 1) / 2 + (bj - bi)) * 256 + (i & 15) * 16 + (j & 15);
}
// (i, j), i <= j, of the e-th upper entry of a c x c matrix, row by row.
__device__ __forceinline__ void upper_entry(int e, int c, int& i, int& j) {
    i = 0;
    while (e >= c - i) e -= c - i++;
    j = i + e;
}
__global__ __launch_bounds__(BLOCK) void k_gram_finish(State* st, const double* __restrict__ gpart,
                                                       const double* __restrict__ gpart_y, const double* rpart, int gv, int nbv, int gy,
                                                       int nby, double* out) {
    __shared__ double shm[3][BLOCK / 64];
    __shared__ int s_last;
    if (st->status != 0) return;
    const int c = min(st->j, st->m), K = st->K;
    const int ev = c * (c + 1) / 2, ey = gy > 0 ? K * (K + 1) / 2 : 0, er = gy > 0 ? K : 0;
    const int lane = threadIdx.x & 63;
    for (int e = blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6); e < ev + ey + er; e += gridDim.x * (BLOCK / 64)) {
        const double* src;
        int64_t stride = GRAM_SLOT;
        int parts = gv, i, j;
        if (e < ev) {
            upper_entry(e, c, i, j);
            src = gpart + gram_place(i, j, nbv);
        } else if (e < ev + ey) {
            upper_entry(e - ev, K, i, j);
            src = gpart_y + gram_place(i, j, nby);
            parts = gy;
        } else {
            src = rpart + (e - ev - ey);
            stride = 64;
            parts = gy;
        }
        double s = 0.0;
#pragma unroll 4
        for (int b = lane; b < parts; b += 64) s += src[b * stride];
        s = wave_sum(s);
        if (lane == 0) st_dev(&out[e], s);
    }
    if (!last_block(&st->ticket[TK_GRAM], gridDim.x, &s_last)) return;
    double wv = 0.0, wy = 0.0, ang = 0.0;
    for (int e = threadIdx.x; e < ev + ey; e += BLOCK) {
        int i, j;
        upper_entry(e < ev ? e : e - ev, e < ev ? c : K, i, j);
        const double g = ld_dev(&out[e]), off = fabs(g - (i == j ? 1.0 : 0.0));
        // fmax drops a NaN, as the per-thread maxima always did.
        if (e < ev) {
            wv = fmax(wv, off);
        } else {
            wy = fmax(wy, off);
            if (i < j) ang += acos(fmin(1.0, fabs(g))) * (180.0 / 3.14159265358979323846);
        }
    }
    wv = wave_max(wv);
    wy = wave_max(wy);
    ang = wave_sum(ang);
    if (lane == 0) {
        shm[0][threadIdx.x >> 6] = wv;
        shm[1][threadIdx.x >> 6] = wy;
        shm[2][threadIdx.x >> 6] = ang;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < BLOCK / 64; ++w) {
            wv = fmax(wv, shm[0][w]);
            wy = fmax(wy, shm[1][w]);
            ang += shm[2][w];
        }
        st->ortho_loss = wv;
        if (gy > 0) {
            st->ritz_ortho_loss = wy;
            st->mean_angle_deg = K > 1 ? ang / (0.5 * K * (K - 1)) : 90.0;
        }
    }
    if ((int)threadIdx.x < er) {
        const double a2 = sqrt(ld_dev(&out[ev + ey + threadIdx.x]));
        const double tl = st->theta[st->sel[threadIdx.x]];
        st->abs_resid[threadIdx.x] = a2;
        st->resid[threadIdx.x] = tl != 0.0 ? a2 / fabs(tl) : a2;
    }
}

// ---------------------------------------------------------------- launchers
static int pow2_at_least(int k) {
    int v = 1;
    while (v < k) v <<= 1;
    return v;
}

// Workgroups of a Gram pass whose wavefronts take `rows` rows at a time.
static int gram_grid(int64_t n, int rows) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(GRAM_GRID, (n + rows * WAVES - 1) / (rows * WAVES)));
}

// Basis of at most cmax columns; returns its grid.
template <class T>
static int launch_gram(const State* st, const T* X, int64_t ldx, int64_t n, int cmax, double* gpart, hipStream_t s) {
    const int g = gram_grid(n, 32);
    switch ((cmax + 15) / 16) {
        case 1: hipLaunchKernelGGL((k_gram<T, 1>), dim3(g), dim3(BLOCK), 0, s, st, X, ldx, n, gpart); break;
        case 2: hipLaunchKernelGGL((k_gram<T, 2>), dim3(g), dim3(BLOCK), 0, s, st, X, ldx, n, gpart); break;
        case 3: hipLaunchKernelGGL((k_gram<T, 3>), dim3(g), dim3(BLOCK), 0, s, st, X, ldx, n, gpart); break;
        default: hipLaunchKernelGGL((k_gram<T, 4>), dim3(g), dim3(BLOCK), 0, s, st, X, ldx, n, gpart); break;
    }
    return g;
}

// Returns its grid; a wavefront takes 32 rows, past 32 columns 16.
template <bool REPORT>
static int launch_out(const State* st, const double* Y, const double* Z, int64_t n, int K, double* out, double* gpart,
                      double* rpart, hipStream_t s) {
    const int nb = (K + 15) / 16, g = gram_grid(n, nb <= 2 ? 32 : 16);
    switch (nb) {
        case 1: hipLaunchKernelGGL((k_out<1, REPORT>), dim3(g), dim3(BLOCK), 0, s, st, Y, Z, n, out, gpart, rpart); break;
        case 2: hipLaunchKernelGGL((k_out<2, REPORT>), dim3(g), dim3(BLOCK), 0, s, st, Y, Z, n, out, gpart, rpart); break;
        case 3: hipLaunchKernelGGL((k_out<3, REPORT>), dim3(g), dim3(BLOCK), 0, s, st, Y, Z, n, out, gpart, rpart); break;
        default: hipLaunchKernelGGL((k_out<4, REPORT>), dim3(g), dim3(BLOCK), 0, s, st, Y, Z, n, out, gpart, rpart); break;
    }
    return g;
}

template <int P>
static hipError_t finish_p(const Plan& p, const Bufs& b, const Csr& a, double* out_vals, double* out_vecs,
                           int report, hipStream_t s) {
    using VT = typename Tr<P>::V;
    const VT* V = (const VT*)b.V;
    hipLaunchKernelGGL(k_jacobi_select, dim3(1), dim3(JBLOCK), 0, s, b.st, out_vals, p.strict_m);
    // A wavefront takes 64 rows at a time.
    const int gr = (int)std::max<int64_t>(1, std::min<int64_t>(1024, (p.n + 64 * WAVES - 1) / (64 * WAVES)));
    switch ((p.K + 15) / 16) {
        case 1: hipLaunchKernelGGL((k_ritz<P, 1>), dim3(gr), dim3(BLOCK), 0, s, b.st, V, p.n, p.ld, b.Y, b.part); break;
        case 2: hipLaunchKernelGGL((k_ritz<P, 2>), dim3(gr), dim3(BLOCK), 0, s, b.st, V, p.n, p.ld, b.Y, b.part); break;
        case 3: hipLaunchKernelGGL((k_ritz<P, 3>), dim3(gr), dim3(BLOCK), 0, s, b.st, V, p.n, p.ld, b.Y, b.part); break;
        default: hipLaunchKernelGGL((k_ritz<P, 4>), dim3(gr), dim3(BLOCK), 0, s, b.st, V, p.n, p.ld, b.Y, b.part); break;
    }
    const int kb2 = pow2_at_least(p.K);
    if (report && p.ooc) {
        // Host-resident matrix: the residual product streams the slabs too.
        const hipError_t e = ooc_pass(*p.ooc, b.st, s,
                                      [&](const int32_t* col, const void* val, int64_t tb, int64_t te, int, int) {
                                          hipLaunchKernelGGL((k_spmm<P>), dim3(p.g_slab), dim3(BLOCK), 0, s, b.st,
                                                             b.Y, b.Z, p.n, p.nnz, p.n_tiles, b.ob, b.tk, b.head,
                                                             b.tail, kb2, a.rowptr, col, val, nullptr, nullptr,
                                                             nullptr, tb, te);
                                      });
        if (e != hipSuccess) return e;
    } else if (report) {
        // Up to 8192 workgroups: 2048 took 0.5 ms more at R-MAT 23 and 25.
        const unsigned gt = (unsigned)(std::min<int64_t>(1024, (p.n_tiles + 8 * WAVES - 1) / (8 * WAVES)) * 8);
        hipLaunchKernelGGL((k_spmm<P>), dim3(gt), dim3(BLOCK), 0, s, b.st, b.Y, b.Z, p.n, p.nnz, p.n_tiles,
                           b.ob, b.tk, b.head, b.tail, kb2, a.rowptr, a.col, a.val, b.rp2, b.col2, b.val2,
                           (int64_t)0, p.n_tiles);
    }
    if (!report) {
        launch_out<false>(b.st, b.Y, nullptr, p.n, p.K, out_vecs, nullptr, nullptr, s);
        return hipGetLastError();
    }
    double* gpart_y = b.gram + (int64_t)GRAM_GRID * GRAM_SLOT;
    const int gy = launch_out<true>(b.st, b.Y, b.Z, p.n, p.K, out_vecs, gpart_y, b.part2, s);
    const int gv = launch_gram<VT>(b.st, V, p.ld, p.n, p.m, b.gram, s);
    const int values = p.m * (p.m + 1) / 2 + p.K * (p.K + 1) / 2 + p.K;
    hipLaunchKernelGGL(k_gram_finish, dim3((values + BLOCK / 64 - 1) / (BLOCK / 64)), dim3(BLOCK), 0, s, b.st, b.gram,
                       gpart_y, b.part2, gv, (p.m + 15) / 16, gy, (p.K + 15) / 16, b.gram + GRAM_OUT);
    return hipGetLastError();
}

hipError_t launch_finish(const Plan& p, const Bufs& b, const Csr& a, double* out_vals, double* out_vecs, int report,
                         hipStream_t s) {
    switch (p.prec) {
        case 0: return finish_p<0>(p, b, a, out_vals, out_vecs, report, s);
        case 1: return finish_p<1>(p, b, a, out_vals, out_vecs, report, s);
        case 2: return finish_p<2>(p, b, a, out_vals, out_vecs, report, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gram_only(int prec, const void* X, int64_t ldx, int64_t n, int c, State* st, double* gram,
                            hipStream_t s) {
    int g = 0;
    switch (prec) {
        case 0: g = launch_gram<double>(st, (const double*)X, ldx, n, c, gram, s); break;
        case 1: g = launch_gram<float>(st, (const float*)X, ldx, n, c, gram, s); break;
        case 2: g = launch_gram<uint16_t>(st, (const uint16_t*)X, ldx, n, c, gram, s); break;
        default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_gram_finish, dim3((c * (c + 1) / 2 + BLOCK / 64 - 1) / (BLOCK / 64)), dim3(BLOCK), 0, s, st,
                       gram, nullptr, nullptr, g, (c + 15) / 16, 0, 0, gram + GRAM_OUT);
    return hipGetLastError();
}

hipError_t launch_jacobi_only(const double* alpha, const double* offdiag, int m, State* st, hipStream_t s) {
    hipLaunchKernelGGL(k_jacobi_only, dim3(1), dim3(JBLOCK), 0, s, alpha, offdiag, m, st);
    return hipGetLastError();
}

}  // namespace lz
