// stencil_pipe64.hpp -- FP64 stencils of many targets as a pipeline of kernels
// (scalar bases of at most 20 monomials, staggered and Neumann-constrained
// stencils among them, and divergence-free bases whose scalar basis has at
// most 10), all of it in FP64.
//
// The stencil of a functional lambda is alpha = W P c with M c = lambda' on
// the plain monomials s^a (M_ab = mu_(a+b), the moments of Section 2.1's
// normal equations; lambda' the functional of Section 2.5 on them).  Solving
// with the Cholesky factor of the formed moment matrix loses cond(M) 2^-53;
// one corrected step with the residual taken over the rows,
//     c += M^-1 (lambda' - P^T (W P c)),
// removes that (corrected seminormal equations, Bjorck 1987): the residual's
// rounding enters as A^T d with A = W^1/2 P, which the weights W P M^-1 A^T d
// see through a projection, so what is left is the cond(A) 2^-53 of the
// Householder QR path.  Kernels:
//   records, A moments   those of the mixed pipeline (stencil_pipe.hpp)
//   B k_pipe_chol<0>     M = L L^T and c, four lanes per target
//   R k_pipe_sums        P^T (W P c) over the rows
//   B k_pipe_chol<1>     the correction (and the constraint's elimination)
//     k_pipe_solve_div   the two B steps of the divergence-free basis
//   C weights            that of the mixed pipeline
// A target whose factor meets a pivot at or below kCholTol of its diagonal
// entry (rank deficiency among it), or whose correction is larger than kCorrTol
// of its solution (cond(M) above about 2e8), goes to the QR kernel, which also
// applies the rank test.
//
// Why not QR for every target: a wavefront per target spends its time in the
// round trips of Q dependent column sums (2M targets of about 110 neighbours,
// order 3: 23.6 ms); here the row work is row-parallel and the Q x Q work four
// lanes per target (moments 2.4, factors 0.33 + 0.33, sums 1.7, weights 1.95
// ms; the step 26.6 -> 10.6 ms), and the weights' error against 64 bits is
// smaller (100k 2-D order-4 targets 1.2e-14 -> 8.5e-15, 60k one-sided order-3
// targets 2.2e-14 -> 1.2e-14).
#pragma once

#include <type_traits>

#include "stencil_pipe.hpp"

namespace gmls {

// a functional of Section 2.5 on the plain monomial s^a (index a, compile
// time), times nothing but powers of 1/eps
template <int DIM, int ORDER>
__device__ __forceinline__ double plain_lambda(int kind, int a, double ie) {
  constexpr Mono<DIM, ORDER> M{};
  const int deg = M.e[a][0] + M.e[a][1] + M.e[a][2];
  if (deg == 0) return kind == FK_VALUE ? 1.0 : 0.0;
  if (deg == 1) {
    const int d = M.e[a][0] ? 0 : M.e[a][1] ? 1 : 2;
    return kind == FK_GRAD0 + d ? ie : 0.0;
  }
  if (deg == 2 && (M.e[a][0] == 2 || M.e[a][1] == 2 || M.e[a][2] == 2)) return kind == FK_LAP ? 2.0 * ie * ie : 0.0;
  return 0.0;
}

// v of lane L of this lane's quad (L a constant after unrolling)
__device__ __forceinline__ double quad_bcast(double v, int L) {
  switch (L) {
    case 0: return dpp_d<0x00>(v);
    case 1: return dpp_d<0x55>(v);
    case 2: return dpp_d<0xAA>(v);
    default: return dpp_d<0xFF>(v);
  }
}

// sum over the quad, the same bits in its four lanes
__device__ __forceinline__ double quad_sum(double v) {
#pragma clang fp contract(off)
  v += dpp_d<0xB1>(v);
  return v + dpp_d<0x4E>(v);
}

// The lower triangle of a Q x Q matrix over a quad: row i = 4 q + l on lane
// l, columns 0 .. 4 q + 3 of slot q (above the diagonal, and in the padding
// rows i >= Q, finite values that no result depends on).
template <int Q>
struct QuadTri {
  static constexpr int QB = (Q + 3) / 4;
  static constexpr int N = 2 * QB * (QB + 1);
  static constexpr int at(int q, int k) { return 2 * q * (q + 1) + k; }
};

// Column J of the right-looking Cholesky factorisation, then the rest: L
// below the diagonal, 1/L_jj on it.  ok: false where a pivot is not above
// kCholTol times its diagonal entry diag.  All lanes of the quad take part.
template <int Q, int J>
__device__ __forceinline__ void quad_cholesky(double (&M)[QuadTri<Q>::N], const double (&diag)[QuadTri<Q>::QB], int l,
                                              bool &ok) {
  using T = QuadTri<Q>;
  constexpr int qj = J / 4, lj = J % 4;
  const double piv = M[T::at(qj, J)];
  ok = ok && (l != lj || piv > kCholTol * diag[qj]);
  const double d = quad_bcast(piv, lj);
  // 1/sqrt(d): the hardware estimate and two Newton steps
  double y = __builtin_amdgcn_rsq(d);
  y = fma(y, fma(-(0.5 * d) * y, y, 0.5), y);
  y = fma(y, fma(-(0.5 * d) * y, y, 0.5), y);
#pragma unroll
  for (int q = qj; q < T::QB; ++q) M[T::at(q, J)] *= y;
  M[T::at(qj, J)] = l == lj ? y : M[T::at(qj, J)];
#pragma unroll
  for (int k = J + 1; k < Q; ++k) {
    const double lk = quad_bcast(M[T::at(k / 4, J)], k % 4);
#pragma unroll
    for (int q = k / 4; q < T::QB; ++q) M[T::at(q, k)] = fma(-M[T::at(q, J)], lk, M[T::at(q, k)]);
  }
  // finish the column's updates here (left to itself the compiler defers
  // each to the step that reads it and keeps every earlier column live)
#pragma unroll
  for (int k = J; k < Q; ++k)
#pragma unroll
    for (int q = k / 4; q < T::QB; ++q) asm volatile("" : "+v"(M[T::at(q, k)]));
  if constexpr (J + 1 < Q) quad_cholesky<Q, J + 1>(M, diag, l, ok);
}

// b <- (L L^T)^-1 b for NR right-hand sides (b[r][q]: entry 4 q + l on lane
// l).  Every fused multiply-add is written out, so that a right-hand side's
// solution is the same bits whichever others it is solved with: a functional
// along the constraint's row has to equal the constraint's solution.
template <int Q, int NR>
__device__ __forceinline__ void quad_solve(const double (&M)[QuadTri<Q>::N], double (&b)[NR][QuadTri<Q>::QB], int l) {
#pragma clang fp contract(off)
  using T = QuadTri<Q>;
  double z[NR][T::QB];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int q = 0; q < T::QB; ++q) z[r][q] = 0.0;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int qj = j / 4, lj = j % 4;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double t = b[r][qj] * M[T::at(qj, j)];  // lane lj: 1/L_jj
      z[r][qj] = l == lj ? t : z[r][qj];
      const double zj = quad_bcast(t, lj);
#pragma unroll
      for (int q = qj; q < T::QB; ++q) b[r][q] = fma(-M[T::at(q, j)], zj, b[r][q]);
#pragma unroll
      for (int q = qj; q < T::QB; ++q) asm volatile("" : "+v"(b[r][q]));
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int q = 0; q < T::QB; ++q) b[r][q] = 0.0;
#pragma unroll
  for (int j = Q - 1; j >= 0; --j) {
    const int qj = j / 4, lj = j % 4;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      // entries below j are still 0 in b; the diagonal's is too, so the
      // sum over the column is that over the rows after j
      double s = 0.0;
#pragma unroll
      for (int q = qj; q < T::QB; ++q) s = fma(M[T::at(q, j)], b[r][q], s);
      s = quad_sum(s);
      const double t = (z[r][qj] - s) * M[T::at(qj, j)];
      b[r][qj] = l == lj ? t : b[r][qj];
    }
  }
}

// B. Four lanes per target: the factor of 20 monomials is 60 doubles a lane,
// which two wavefronts per SIMD hold but for 4 and 12 spilled registers of the
// two passes (constrained: 11 and 32; one thread per target needs 210 doubles;
// a wavefront per target idles 44 lanes), and
// pivots and columns pass between the lanes by DPP.  Bound by instruction
// issue: a third are those moves (2 per double).  0.33 ms per million targets
// and pass at order 3 and one right-hand side, 0.12 ms for each more; compiled
// for three wavefronts per SIMD it spills and takes 2.6 times as long.
//
// PASS 0: the factor and c = M^-1 lambda' of every functional into coef
// [slot][F][Q] (CON: [F + 1], the constraint's solution last).  PASS 1: the
// same factor again (taking it once more costs less than 1.7 KB per target
// through memory) and c += M^-1 (lambda' - sums).  The
// constraint f . c = 0 of the Neumann stencils is eliminated in both: with
// z = M^-1 f, g = f.c / f.z is the boundary weight and c -= g z (Section 2.3);
// PASS 1 corrects c and g together, from the residual lambda' - sums - g f, and
// eliminates what the correction brings back.  Corrected apart from each other
// c and z bring their own errors to the difference: root mean square errors of
// one-sided 3-D order-3 targets, 24 neighbours 9.5e-14 (QR 9.0e-14), 80
// neighbours 3.9e-15 (5.8e-15); corrected together 5.7e-15 and 8.1e-16.
template <int DIM, int ORDER, int SKIP, int PASS, bool CON>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_pipe_chol(
    StencilArgs a, PipeRec *rec, int win_lo, int win_hi, const double *mom, double *coef, const double *sums,
    int *left_list, int *left, BinMeta *meta) {
#pragma clang fp contract(off)
  constexpr int Q = num_mono(DIM, ORDER) - SKIP;
  constexpr int NM = num_mono(DIM, 2 * ORDER);
  static_assert(NM <= 256, "moment indices fit a byte");
  using T = QuadTri<Q>;
  constexpr SumIndex<DIM, ORDER> SI{};
  __shared__ double mls[16 * NM];
  const int lane = lane_id(), l = lane & 3, tq = lane >> 2;
  const int F = a.F;
  const RowKinds rk = row_kinds(DIM, 0, a.mask);
  const SlotRange R = slot_range(meta, 0, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  for (int s0 = first + xcd_block() * 16; s0 < last; s0 += gridDim.x * 16) {
    const int cnt = last - s0 < 16 ? last - s0 : 16;
    const double *mp = mom + (int64_t)(s0 - c0) * NM;
    const int elast = cnt * NM - 1;  // groups past the last target take that target's moments
    double mv[NM / 4];
#pragma unroll
    for (int u = 0; u < NM / 4; ++u) {
      const int e = 64 * u + lane;
      mv[u] = mp[e < elast ? e : elast];
    }
#pragma unroll
    for (int u = 0; u < NM / 4; ++u) mls[64 * u + lane] = mv[u];
    if constexpr (NM % 4 != 0) {
      const int e = 64 * (NM / 4) + lane;
      if (e < 16 * NM) mls[e] = mp[e < elast ? e : elast];
    }
    wave_lds_sync();
    const bool valid = tq < cnt;
    const int64_t loc = (valid ? s0 + tq : s0) - c0;
    const int t = rec[loc].t;
    const double ie = rec[loc].ie;
    const bool use = valid && (PASS == 0 || rec[loc].ok);
    if constexpr (PASS == 1) {
      if (__ballot(use) == 0) continue;  // left to the QR kernel, all of them
    }
    // row i = 4 q + l: its moments' indices, a byte per lane of the quad
    const double *mt = mls + tq * NM;
    double M[T::N], diag[T::QB];
#pragma unroll
    for (int q = 0; q < T::QB; ++q) {
      diag[q] = 1.0;
#pragma unroll
      for (int k = 0; k < 4 * q + 4; ++k) {
        if (k >= Q) {
          M[T::at(q, k)] = 0.0;
          continue;
        }
        unsigned idx = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (4 * q + u < Q) idx |= (unsigned)SI.idx[4 * q + u + SKIP][k + SKIP] << (8 * u);
        const double v = mt[(idx >> (8 * l)) & 255u];
        M[T::at(q, k)] = 4 * q + 3 < Q || 4 * q + l < Q ? v : 0.0;
        if (k >= 4 * q) diag[q] = l == k - 4 * q ? v : diag[q];
      }
    }
#pragma unroll
    for (int e = 0; e < T::N; ++e) asm volatile("" : "+v"(M[e]));
    bool ok = true;
    quad_cholesky<Q, 0>(M, diag, l, ok);
    if constexpr (PASS == 0) {
      // the quad's verdict in its four lanes
      const uint64_t bad = __ballot(!ok);
      ok = ((bad >> (lane & ~3)) & 15u) == 0;
    }
    // M_ii of entry 4 q + l (0 in the padding)
    auto mii = [&](int q) {
      unsigned idx = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (4 * q + u < Q) idx |= (unsigned)SI.idx[4 * q + u + SKIP][4 * q + u + SKIP] << (8 * u);
      const double v = mt[(idx >> (8 * l)) & 255u];
      return 4 * q + 3 < Q || 4 * q + l < Q ? v : 0.0;
    };
    bool good = true;  // PASS 1: every correction is small (kCorrTol)
    // entry of the constraint's row on this lane, among the linear monomials
    auto row = [&](int d) { return l == (1 + d) % 4 ? a.normals[(int64_t)t * DIM + d] * ie : 0.0; };
    // right-hand side f (PASS 1: its residual over the rows; the multiplier's
    // part is taken off on constrained stencils)
    auto rhs = [&](int f, double(&b)[T::QB]) {
#pragma unroll
      for (int q = 0; q < T::QB; ++q) {
        b[q] = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = 4 * q + u;
          if (i >= Q || i + SKIP > num_mono(DIM, ORDER < 2 ? ORDER : 2) - 1) continue;
          const double v = plain_lambda<DIM, ORDER>(rk.kind[f], i + SKIP, ie);
          b[q] = l == u ? v : b[q];
        }
        if constexpr (PASS == 1) {
          const int i = 4 * q + l;
          if (i < Q) b[q] -= sums[(loc * F + f) * Q + i];
        }
      }
      if constexpr (CON && PASS == 1) {
        const double g = a.hweights[(int64_t)t * F + f];
#pragma unroll
        for (int d = 0; d < DIM; ++d)
          b[(1 + d) / 4] -= g * row(d);
      }
    };
    // entry i of the solution of right-hand side f
    auto at = [&](int f, int q) { return (loc * (CON ? F + 1 : F) + f) * Q + 4 * q + l; };
    // CON: z = M^-1 row (kept behind the functionals' coefficients, the registers
    // being full) and row . z
    double fz = 0.0;
    bool con = false;
    if constexpr (CON) {
      if constexpr (PASS == 0) {
        double b[1][T::QB];
#pragma unroll
        for (int q = 0; q < T::QB; ++q) b[0][q] = 0.0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) b[0][(1 + d) / 4] += row(d);
        quad_solve<Q, 1>(M, b, l);
#pragma unroll
        for (int q = 0; q < T::QB; ++q)
          if (use && 4 * q + l < Q) coef[at(F, q)] = b[0][q];
      }
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        con = con || a.normals[(int64_t)t * DIM + d] != 0.0;
        fz += l == (1 + d) % 4 ? row(d) * coef[at(F, (1 + d) / 4)] : 0.0;
      }
      fz = quad_sum(fz);
    }
    auto finish = [&](int f, const double(&b)[T::QB]) {
#pragma clang fp contract(off)
      double c[T::QB], excess = 0.0;  // the squared sizes of correction - bound, summed over the quad below
#pragma unroll
      for (int q = 0; q < T::QB; ++q) {
        c[q] = b[q];
        if constexpr (PASS == 1) {
          c[q] += 4 * q + l < Q ? coef[at(f, q)] : 0.0;
          excess = fma(fma(-kCorrTol * kCorrTol * c[q], c[q], b[q] * b[q]), mii(q), excess);
        }
      }
      if constexpr (CON) {
        double fc = 0.0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) fc += l == (1 + d) % 4 ? row(d) * c[(1 + d) / 4] : 0.0;
        fc = quad_sum(fc);
        double g = con ? fc / fz : 0.0;
        const double g0 = PASS == 1 ? a.hweights[(int64_t)t * F + f] : 0.0;
        if (con) {
#pragma unroll
          for (int q = 0; q < T::QB; ++q) {
            const double z = 4 * q + l < Q ? coef[at(F, q)] : 0.0;
            c[q] = fma(-g, z, c[q]);
            // (the eliminated part is of the solution's size too)
            if constexpr (PASS == 1) excess = fma(-kCorrTol * kCorrTol * g0 * g0 * z * z, mii(q), excess);
          }
        }
        g += g0;
        if (use && l == 0) a.hweights[(int64_t)t * F + f] = g;
      }
      if constexpr (PASS == 1) good = good && quad_sum(excess) <= 0.0;
      if (use) {
#pragma unroll
        for (int q = 0; q < T::QB; ++q)
          if (4 * q + l < Q) coef[at(f, q)] = c[q];
      }
    };
    int f = 0;
    for (; f + 1 < F; f += 2) {
      double b[2][T::QB];
      rhs(f, b[0]);
      rhs(f + 1, b[1]);
      quad_solve<Q, 2>(M, b, l);
      finish(f, b[0]);
      finish(f + 1, b[1]);
    }
    if (f < F) {
      double b[1][T::QB];
      rhs(f, b[0]);
      quad_solve<Q, 1>(M, b, l);
      finish(f, b[0]);
    }
    if constexpr (PASS == 0) {
      if (valid && l == 0) {
        rec[loc].ok = ok ? 1 : 0;
        if (ok) a.status[t] = GMLS_TARGET_OK;
      }
      leave_targets(valid && l == 0 && !ok, s0 + tq, t, meta, left_list, left);
    } else {
      const bool leave = use && l == 0 && !good;
      if (leave) rec[loc].ok = 0;
      leave_targets(leave, s0 + tq, t, meta, left_list, left);
    }
    wave_lds_sync();  // the moments' buffer is rewritten
  }
}

// R. sums [slot][F][Q]: P^T (W P c) of every right-hand side's coefficients,
// a group of G lanes per target (rows as in the moment kernel: the same
// scaled offsets and weights), the group's partial sums added through LDS in
// lane order.  The rows are gathered once for all right-hand sides (LOOP, the
// long bin: once per chunk and right-hand side).  Bound as the moment kernel,
// by FP64 arithmetic and the reduction: about 110 FP64 operations a row for
// one right-hand side at order 3 (1.7 ms at 220M rows, the moments 2.4).
template <int DIM, int ORDER, int G, int RPL, int SKIP = 0, bool LOOP = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_pipe_sums(
    StencilArgs a, const PipeRec *rec, const BinMeta *meta, int bin, int win_lo, int win_hi, const double *coef,
    double *sums) {
  constexpr int QF = num_mono(DIM, ORDER);
  constexpr int Q = QF - SKIP;
  constexpr int TPW = 64 / G;
  constexpr int RW = 66;
  constexpr MonoIndex<DIM, ORDER> H{};
  __shared__ __align__(16) double red[Q * RW];
  const SlotRange R = slot_range(meta, bin, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  const int lane = lane_id();
  const int grp = lane / G, lg = lane % G, grp0 = lane - lg;
  const int F = a.F, cs = (F + (a.normals ? 1 : 0)) * Q;  // coefficients of a target
  for (int i0 = first + xcd_block() * TPW; i0 < last; i0 += gridDim.x * TPW) {
    const int i = i0 + grp;
    const bool valid = i < last;
    const int64_t loc = (valid ? i : first) - c0;
    const PipeRec rc = rec[loc];
    if (__ballot(valid && rc.ok) == 0) continue;  // left to the QR kernel, all of them
    const int64_t base = rc.base;
    const int N = rc.n;
    double xt[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) xt[d] = rc.x[d];
    const int cend = chunk_end<LOOP, G * RPL>(N);
    double s[RPL][DIM], w[RPL];
    auto load = [&](int q0) {
      const int nrem = N - q0;
      double xs[RPL][DIM];
      gather_rows<DIM, RPL, G, true>(a, base + (nrem > 0 ? q0 : 0), nrem > 0 ? nrem : N, lg, xs);
      rows_sw<DIM>(xs, xt, rc.ie, a.p, [&](int r) { return lg + G * r < nrem; }, s, w);
    };
    if constexpr (!LOOP) load(0);
    for (int f = 0; f < F; ++f) {
      double cf[QF], acc[QF];
      if constexpr (SKIP != 0) cf[0] = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) cf[q + SKIP] = coef[loc * cs + f * Q + q];
#pragma unroll
      for (int q = 0; q < QF; ++q) acc[q] = 0.0;
      for (int q0 = 0; q0 < cend; q0 += G * RPL) {
        if constexpr (LOOP) load(q0);
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
          const double u = w[r] * horner<DIM, ORDER>(cf, s[r]);
          // u s^a, the last coordinate's powers innermost
          double pl[ORDER + 1];
          pl[0] = 1.0;
#pragma unroll
          for (int c = 1; c <= ORDER; ++c) pl[c] = c == 1 ? s[r][DIM - 1] : pl[c - 1] * s[r][DIM - 1];
          double ua = u;
#pragma unroll
          for (int ex = 0; ex <= ORDER; ++ex) {
            if (ex > 0) ua *= s[r][0];
            double ub = ua;
            if constexpr (DIM == 3) {
#pragma unroll
              for (int ey = 0; ey <= ORDER - ex; ++ey) {
                if (ey > 0) ub *= s[r][1];
#pragma unroll
                for (int ez = 0; ez <= ORDER - ex - ey; ++ez)
                  acc[H.idx[ex][ey][ez]] = ez == 0 ? acc[H.idx[ex][ey][ez]] + ub : fma(ub, pl[ez], acc[H.idx[ex][ey][ez]]);
              }
            } else {
#pragma unroll
              for (int ey = 0; ey <= ORDER - ex; ++ey)
                acc[H.idx[ex][ey][0]] = ey == 0 ? acc[H.idx[ex][ey][0]] + ub : fma(ub, pl[ey], acc[H.idx[ex][ey][0]]);
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < QF; ++q) asm volatile("" : "+v"(acc[q]));  // as in the moment kernel
#pragma unroll
      for (int q = 0; q < Q; ++q) red[q * RW + lane] = acc[q + SKIP];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < (Q + G - 1) / G; ++k) {
        const int q = lg + G * k;
        if (q < Q) {
          const double2 *row = reinterpret_cast<const double2 *>(red + q * RW + grp0);
          double v = 0.0;
#pragma unroll
          for (int e = 0; e < G / 2; ++e) {
            const double2 p = row[e];
            v += p.x;
            v += p.y;
          }
          if (valid) sums[(loc * F + f) * Q + q] = v;
        }
      }
      __syncthreads();
    }
  }
}

template <int DIM, int ORDER, int SKIP, int BIN>
static void pipe_sums_bin(const StencilArgs &a, const PipeRec *rec, const BinMeta *meta, int win_lo, int win_hi,
                          int n_max, const double *coef, double *sums, int cus, hipStream_t s) {
  constexpr PipeShape S = kPipeShapes[BIN][pipe_default_shape(DIM, ORDER, false, false, false, BIN)];
  constexpr int TPW = 64 / S.g;
  int nb = (n_max + TPW - 1) / TPW;
  if (nb > cus * 32) nb = cus * 32;
  k_pipe_sums<DIM, ORDER, S.g, S.rpl, SKIP, BIN == kLongBin>
      <<<xcd_grid(nb), 64, 0, s>>>(a, rec, meta, BIN, win_lo, win_hi, coef, sums);
}

// kernel `what` (0 moments, 1 sums, 2 weights) of every bin of a window
template <int DIM, int ORDER, int SKIP, int BASIS>
static void pipe64_bins(int what, const StencilArgs &a, const PipeRec *rec, const BinMeta *hm, const BinMeta *meta,
                        int win_lo, int win_hi, double *mom, double *coef, double *sums, int cus, hipStream_t s) {
  for (int b = 1; b < kNumBins; ++b) {
    int n = win_hi - win_lo;
    if (hm) {
      const int lo = hm->offset[b] > win_lo ? hm->offset[b] : win_lo;
      const int hi = hm->offset[b] + hm->count[b] < win_hi ? hm->offset[b] + hm->count[b] : win_hi;
      if (lo >= hi) continue;
      n = hi - lo;
    }
    switch (b) {
#define GMLS_PIPE64_BIN(B_)                                                                                       \
  case B_:                                                                                                        \
    if (what == 1)                                                                                                \
      pipe_sums_bin<DIM, ORDER, SKIP, B_>(a, rec, meta, win_lo, win_hi, n, coef, sums, cus, s);                   \
    else                                                                                                          \
      pipe_bin_shape<DIM, ORDER, SKIP, BASIS, B_>(-1, what == 2, a, rec, meta, win_lo, win_hi, n,                  \
                                                  what == 2 ? coef : mom, cus, s);                                \
    break;
      GMLS_PIPE64_BIN(1) GMLS_PIPE64_BIN(2) GMLS_PIPE64_BIN(3) GMLS_PIPE64_BIN(4) GMLS_PIPE64_BIN(5)
#undef GMLS_PIPE64_BIN
      default: break;
    }
  }
}

// The FP64 pipeline over the list slots of bins 1 and up, in windows of
// `chunk` slots from slot 0 (their bounds do not depend on the bin table, so
// that a captured call needs no host copy of it; hm, where there is one, skips
// empty windows and bins and sizes the grids).  ss, sv: a scalar and a
// divergence-free set (either may be null), the records and moments of a
// window serving both.  mom, coef, sums, rec: buffers of one window.
template <int DIM, int ORDER, int SKIP>
hipError_t launch_pipe64(const Pipe64Set *ss, const Pipe64Set *sv, const int *list, const BinMeta *hm, BinMeta *meta,
                         double *mom, double *coef, double *sums, PipeRec *rec, int64_t chunk, int n_max, int cus,
                         hipStream_t s) {
  if (sv && !(SKIP == 0 && has_pipe_div<DIM, ORDER>())) return hipErrorInvalidValue;
  const StencilArgs &a = ss ? ss->a : sv->a;
  for (int64_t w0 = 0; w0 < n_max; w0 += chunk) {
    const int win_lo = (int)w0;
    const int win_hi = (int)(w0 + chunk < n_max ? w0 + chunk : n_max);
    if (hm && win_hi <= hm->offset[1]) continue;
    const int n_win = win_hi - win_lo;
    int nbp = (n_win + 255) / 256;
    if (nbp > cus * 8) nbp = cus * 8;
    k_pipe_prep<DIM><<<nbp, 256, 0, s>>>(a, list, meta, win_lo, win_hi, rec);
    pipe64_bins<DIM, ORDER, SKIP, 0>(0, a, rec, hm, meta, win_lo, win_hi, mom, coef, sums, cus, s);
    if (ss) {
      int nbc = (n_win + 15) / 16;
      if (nbc > cus * 64) nbc = cus * 64;
      nbc = xcd_grid(nbc);
      auto chol = [&](auto pass) {
        constexpr int P = decltype(pass)::value;
        if constexpr (SKIP == 0) {
          if (ss->a.normals) {
            k_pipe_chol<DIM, ORDER, 0, P, true>
                <<<nbc, 64, 0, s>>>(ss->a, rec, win_lo, win_hi, mom, coef, sums, ss->left_list, ss->left, meta);
            return;
          }
        }
        k_pipe_chol<DIM, ORDER, SKIP, P, false>
            <<<nbc, 64, 0, s>>>(ss->a, rec, win_lo, win_hi, mom, coef, sums, ss->left_list, ss->left, meta);
      };
      chol(std::integral_constant<int, 0>{});
      pipe64_bins<DIM, ORDER, SKIP, 0>(1, ss->a, rec, hm, meta, win_lo, win_hi, mom, coef, sums, cus, s);
      chol(std::integral_constant<int, 1>{});
      pipe64_bins<DIM, ORDER, SKIP, 0>(2, ss->a, rec, hm, meta, win_lo, win_hi, mom, coef, sums, cus, s);
    }
    if constexpr (SKIP == 0 && has_pipe_div<DIM, ORDER>()) {
      if (sv) {
        int nbs = (n_win + 63) / 64;
        if (nbs > cus * 16) nbs = cus * 16;
        nbs = xcd_grid(nbs);
        StencilArgs each = sv->a;  // every component of every row as a right-hand side of its own
        each.F = sv->a.F * DIM;
        k_pipe_solve_div<DIM, ORDER, 0><<<nbs, 64, 0, s>>>(sv->a, rec, win_lo, win_hi, mom, coef, sums, sv->left_list,
                                                           sv->left, meta, nullptr, Options());
        pipe64_bins<DIM, ORDER, 0, 0>(1, each, rec, hm, meta, win_lo, win_hi, mom, coef, sums, cus, s);
        k_pipe_solve_div<DIM, ORDER, 1><<<nbs, 64, 0, s>>>(sv->a, rec, win_lo, win_hi, mom, coef, sums, sv->left_list,
                                                           sv->left, meta, nullptr, Options());
        pipe64_bins<DIM, ORDER, 0, 1>(2, sv->a, rec, hm, meta, win_lo, win_hi, mom, coef, sums, cus, s);
      }
    }
  }
  return hipGetLastError();
}

}  // namespace gmls
