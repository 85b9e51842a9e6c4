// stencil_wave.hpp -- mixed-path stencils with one wavefront per target, for
// bases too large for the one-thread solve of the pipeline (scalar bases of
// up to 35 monomials, divergence-free bases whose scalar part has up to 35).
//
// The stencil of a functional lambda is alpha = W P y with (P^T W P) y =
// lambda (Section 2.1, normal equations; Section 2.5, functionals).  For one
// target the wavefront
//  1. gathers its rows j = lane + 64 r once (eps-scaled offsets s_j, kernel
//     weights w_j, kept in registers);
//  2. forms the FP64 moments mu_g = sum_j w_j s_j^g, |g| <= 2m: per-lane
//     partial sums in lexicographic order of g, summed over the wavefront
//     through LDS in rounds of 16 moments (fixed order: reproducible);
//  3. builds the Jacobi-equilibrated moment Gram E_ik = mu_(i+k) / sqrt(
//     mu_2i mu_2k) (the factorials of the scaled basis cancel), lane i
//     holding row i, and inverts it in FP64 by symmetric sweeps (Gauss-Jordan
//     on a symmetric positive definite matrix, no pivoting: every pivot is a
//     Schur-complement diagonal in (0, 1]); the 1-norm condition number is
//     exact here, ||E||_1 ||E^-1||_1, and is held against the threshold;
//  4. scalar basis: y = G^-1 lambda with G^-1 = Dg E^-1 Dg (Dg_i = i! /
//     sqrt(mu_2i)); divergence-free basis (Section 2.2): the fit over the
//     kernel of the divergence map, as in the pipeline (g = G^-1 (l - D^T t),
//     S t = D G^-1 l, S = D G^-1 D^T), with S equilibrated and swept too;
//  5. alpha_j = w_j p(s_j) . y by Horner steps, the coefficients broadcast
//     through LDS, stores coalesced over the rows.
// Targets whose sweep meets a non-positive pivot or whose condition number
// exceeds the threshold are queued for the FP64 QR fallback.
#pragma once

#include <float.h>
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "basis.hpp"
#include "gmls_internal.hpp"
#include "stencil_mixed64.hpp"
#include "stencil_pipe.hpp"

namespace gmls {

// index of the moment s^(x,y,z), |g| <= D2, in lexicographic order (x
// slowest): the order in which the wavefront accumulates them
template <int DIM, int D2>
struct LexMoments {
  static constexpr int N = num_mono(DIM, D2);
  int id[D2 + 1][D2 + 1][D2 + 1];
  int e[N][3];
  constexpr LexMoments() : id{}, e{} {
    int n = 0;
    for (int x = 0; x <= D2; ++x)
      for (int y = 0; y <= (DIM >= 2 ? D2 - x : 0); ++y)
        for (int z = 0; z <= (DIM == 3 ? D2 - x - y : 0); ++z) {
          id[x][y][z] = n;
          e[n][0] = x;
          e[n][1] = y;
          e[n][2] = z;
          ++n;
        }
  }
};

// lexicographic moment index of basis monomials i + k (row-major Q x Q)
template <int DIM, int ORDER>
struct WavePairs {
  static constexpr int Q = num_mono(DIM, ORDER);
  unsigned char p[Q * Q];
  constexpr WavePairs() : p{} {
    Mono<DIM, ORDER> M{};
    LexMoments<DIM, 2 * ORDER> L{};
    for (int i = 0; i < Q; ++i)
      for (int k = 0; k < Q; ++k)
        p[i * Q + k] =
            (unsigned char)L.id[M.e[i][0] + M.e[k][0]][M.e[i][1] + M.e[k][1]][M.e[i][2] + M.e[k][2]];
  }
};
static_assert(num_mono(3, 8) < 256, "moment indices fit a byte");

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}

// f(integral_constant<int, I>) for I = B .. E - 1
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Broadcast factors.  The sweeps and the coefficient steps multiply every
// lane's entries by a vector that all lanes need whole.  Read from LDS entry by
// entry that is 8 cycles of the compute unit's LDS for 16 bytes in every lane,
// shared by four SIMDs whose two multiply-adds take 8 cycles each.  Here a lane
// holds entries 16 m + lane % 16, so that each row of 16 lanes holds the whole
// vector, and the multiply-add takes its factor from lane L of its own row (500k
// targets of order 4, both sets: 11.95 -> 10.2 ms; 100k scalar targets, whole
// call, 1720 -> 1430 us).
template <int N>
struct RowVec {
  static constexpr int NB = (N + 15) / 16;
  double x[NB];
  // v: 16 NB doubles of LDS that may be read (those past N are not used)
  __device__ __forceinline__ void load(const double *v) {
#pragma unroll
    for (int m = 0; m < NB; ++m) x[m] = v[16 * m + (lane_id() & 15)];
  }
};

// a += x0[lane L of the row] * e0, then a += x1[..] * e1 (and b, of lane
// L + 1).  Every lane must be active.  The wait states are for a factor written
// by the vector instruction before, which the compiler does not see to inside
// asm; one wait per multiply-add cost as much as the multiply-adds saved, so
// several share it.
#define GMLS_FMAC_ROW(A, X, E, L) "v_fmac_f64_dpp " A ", " X ", " E " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
template <int L>
__device__ __forceinline__ void fmac_row2(double &a, double x0, double e0, double x1, double e1) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%1", "%2", "%c5") GMLS_FMAC_ROW("%0", "%3", "%4", "%c5")
      : "+&v"(a)
      : "v"(x0), "v"(e0), "v"(x1), "v"(e1), "n"(L));
}
template <int L>
__device__ __forceinline__ void fmac_row2(double &a, double &b, double x0, double e0, double x1, double e1) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%2", "%3", "%c6") GMLS_FMAC_ROW("%1", "%2", "%3", "%c7")
          GMLS_FMAC_ROW("%0", "%4", "%5", "%c6") GMLS_FMAC_ROW("%1", "%4", "%5", "%c7")
      : "+&v"(a), "+&v"(b)
      : "v"(x0), "v"(e0), "v"(x1), "v"(e1), "n"(L), "n"(L + 1));
}

// a[d] += x[d][lane L of the row] * e[d]
template <int L>
__device__ __forceinline__ void fmac_rows(double (&a)[1], const double (&x)[1], const double (&e)[1]) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%1", "%2", "%c3") : "+&v"(a[0]) : "v"(x[0]), "v"(e[0]), "n"(L));
}
template <int L>
__device__ __forceinline__ void fmac_rows(double (&a)[2], const double (&x)[2], const double (&e)[2]) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%2", "%4", "%c6") GMLS_FMAC_ROW("%1", "%3", "%5", "%c6")
      : "+&v"(a[0]), "+&v"(a[1])
      : "v"(x[0]), "v"(x[1]), "v"(e[0]), "v"(e[1]), "n"(L));
}
template <int L>
__device__ __forceinline__ void fmac_rows(double (&a)[3], const double (&x)[3], const double (&e)[3]) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%3", "%6", "%c9") GMLS_FMAC_ROW("%1", "%4", "%7", "%c9")
          GMLS_FMAC_ROW("%2", "%5", "%8", "%c9")
      : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2])
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(e[0]), "v"(e[1]), "v"(e[2]), "n"(L));
}
// a[d] += x[lane L + d of the row] * e
template <int L>
__device__ __forceinline__ void fmac_rows1(double (&a)[2], double x, double e) {
  asm("s_nop 1\n\t" GMLS_FMAC_ROW("%0", "%2", "%3", "%c4") GMLS_FMAC_ROW("%1", "%2", "%3", "%c5")
      : "+&v"(a[0]), "+&v"(a[1])
      : "v"(x), "v"(e), "n"(L), "n"(L + 1));
}
#undef GMLS_FMAC_ROW

// sum_i e[i] v[i], in order of i (e: this lane's, v: every lane's)
template <int N>
__device__ __forceinline__ double row_vec_dot(const double (&e)[N], const RowVec<N> &v) {
  double d[1] = {0.0};
  static_for<0, N>([&](auto I) { fmac_rows<I % 16>(d, {v.x[I / 16]}, {e[I]}); });
  return d[0];
}

// Symmetric sweep of every pivot of the Q x Q symmetric matrix whose row
// `lane` is a[] (lanes >= Q hold zeros): on return a[] is row `lane` of
// -A^-1.  Sweeping the pivot set P: A_PP <- -A_PP^-1, A_iP <- A_iP A_PP^-1,
// A_Pj <- A_PP^-1 A_Pj, A_ij <- A_ij - A_iP A_PP^-1 A_Pj (i, j not in P);
// sweeps of disjoint sets commute, so the pivots are taken two at a time
// (2 x 2 blocks, one reciprocal of the determinant each) and a trailing
// single pivot for odd Q.  The matrix stays symmetric, so columns k, k+1
// (one LDS store per lane) are also rows k, k+1; the column buffers
// alternate between steps (col: 4 x 64 doubles, 16-byte aligned), one
// barrier per step.
// Each step updates the next step's pivot columns first, stores them, and
// takes the next pivot block (from the registers of its lanes) and its
// reciprocal before the rest of its update, so that this chain overlaps
// the step's bulk of independent multiply-adds.
// Returns false when a leading pivot of a block is not above tol
// (wave-uniform).
template <int Q>
__device__ __forceinline__ bool sweep_inverse(double (&a)[Q], double *col, double tol) {
  const int lane = lane_id();
  bool ok = true;
  // a step's two pivot columns, interleaved: cc[j] = (A_jk, A_j,k+1), so
  // that one 16-byte LDS read brings both operands of the update of a[j]
  double2 *cb[2] = {(double2 *)col, (double2 *)(col + 128)};
  // pivot block of the current step: p00, p01, p11 and 1/det (2 x 2), or
  // p00 and 1/p00 (the trailing single pivot)
  double p00 = 0.0, p01 = 0.0, p11 = 0.0, det = 1.0, id = 1.0;
  if constexpr (Q >= 2) {
    if (lane < Q) cb[0][lane] = make_double2(a[0], a[1]);
    p00 = readlane_d(a[0], 0);
    p01 = readlane_d(a[0], 1);
    p11 = readlane_d(a[1], 1);
    det = p00 * p11 - p01 * p01;
    id = 1.0 / det;
  } else {
    if (lane < Q) cb[0][lane].x = a[0];
    p00 = readlane_d(a[0], 0);
    id = 1.0 / p00;
  }
#pragma unroll
  for (int k = 0; k + 1 < Q; k += 2) {
    const double2 *cc = cb[(k >> 1) & 1];
    double2 *nc = cb[((k >> 1) + 1) & 1];  // the next step's columns
    __syncthreads();
    ok = ok && p00 > tol && det > tol * p00;
    const double i00 = p11 * id, i01 = -p01 * id, i11 = p00 * id;
    const double ak = a[k], ak1 = a[k + 1];
    const double f0 = ak * i00 + ak1 * i01, f1 = ak * i01 + ak1 * i11;
    RowVec<Q> c0, c1;  // columns k, k + 1
#pragma unroll
    for (int m = 0; m < RowVec<Q>::NB; ++m) {
      const double2 c = cc[16 * m + (lane & 15)];
      c0.x[m] = c.x;
      c1.x[m] = c.y;
    }
    // rows k, k+1 themselves become A_PP^-1 A_Pj: their f is the unit
    // vector up to rounding, so the same update with e = A_PP^-1 applies
    const bool l0 = lane == k, l1 = lane == k + 1;
    const double e0 = (l0 ? i00 : l1 ? i01 : 0.0) - f0;
    const double e1 = (l0 ? i01 : l1 ? i11 : 0.0) - f1;
    // pivots of the next step: 2, 1 (the trailing single pivot) or none
    // (the loop is unrolled, so NX and the indices below are constants)
    const int NX = (k + 3 < Q) ? 2 : (k + 2 < Q ? 1 : 0);
    const int q0 = k + 2 < Q ? k + 2 : Q - 1, q1 = k + 3 < Q ? k + 3 : Q - 1;
    if (NX >= 1) {
      const double2 c = cc[q0];
      a[q0] = fma(e0, c.x, fma(e1, c.y, a[q0]));
    }
    if (NX == 2) {
      const double2 c = cc[q1];
      a[q1] = fma(e0, c.x, fma(e1, c.y, a[q1]));
    }
    if (NX == 2) {
      if (lane < Q) nc[lane] = make_double2(a[q0], a[q1]);
      p00 = readlane_d(a[q0], q0);
      p01 = readlane_d(a[q0], q1);
      p11 = readlane_d(a[q1], q1);
      det = p00 * p11 - p01 * p01;
      id = 1.0 / det;
    } else if (NX == 1) {
      if (lane < Q) nc[lane].x = a[q0];
      p00 = readlane_d(a[q0], q0);
      id = 1.0 / p00;
    }
    static_for<0, (Q + 1) / 2>([&](auto J) {
      constexpr int j = 2 * J, m = j / 16;
      if (j == k || (NX > 0 && j == k + 2)) return;
      if constexpr (j + 1 < Q)
        fmac_row2<j % 16>(a[j], a[j + 1], c1.x[m], e1, c0.x[m], e0);
      else
        fmac_row2<j % 16>(a[j], c1.x[m], e1, c0.x[m], e0);
    });
    a[k] = l0 ? -i00 : l1 ? -i01 : f0;
    a[k + 1] = l0 ? -i01 : l1 ? -i11 : f1;
    // finish this step's updates here: left alone, the compiler defers each
    // a[j] update to the step that first reads it, which keeps every
    // earlier pivot column live (quadratic register use)
#pragma unroll
    for (int j = 0; j < Q; ++j) asm volatile("" : "+v"(a[j]));
  }
  if constexpr (Q % 2 == 1) {
    constexpr int k = Q - 1;
    const double2 *cc = cb[(Q / 2) & 1];
    __syncthreads();
    ok = ok && p00 > tol;
    const double d = id;
    const double f = a[k] * d;
    const double ef = (lane == k ? d : 0.0) - f;
    RowVec<Q> c0;
#pragma unroll
    for (int m = 0; m < RowVec<Q>::NB; ++m) c0.x[m] = cc[16 * m + (lane & 15)].x;
    static_for<0, Q / 2>([&](auto J) {
      constexpr int j = 2 * J;
      double p[2] = {a[j], a[j + 1]};
      // lanes j and j + 1 of the row
      fmac_rows1<j % 16>(p, c0.x[j / 16], ef);
      a[j] = p[0];
      a[j + 1] = p[1];
    });
    a[k] = lane == k ? -d : f;
  }
  __syncthreads();  // the buffers may be rewritten after this
  return ok;
}

// Moments mu_g (lexicographic order) of the rows held by the wavefront into
// mu[]; red is the LDS reduction buffer (64 x (RS + 1) doubles, 16-byte aligned).  One step per
// moment, unrolled by template recursion so that every exponent, register
// index and round boundary is a compile-time constant.  RS moments go
// through LDS per round (8, 16 or 32: the autotuner's choice, a trade of
// registers and LDS for barriers).

// sum one round over the wavefront: every lane stores its partials
// (moment q of lane L at q * 66 + L: a moment's partials are contiguous),
// then lanes q + RS p add lanes RS p .. RS p + RS - 1 of moment q, read 16
// bytes at a time, and butterfly steps combine the 64 / RS parts (fixed
// order).  red: 16-byte aligned, RS * 66 <= 64 * (RS + 1) doubles.
template <int NM, int RS>
__device__ __forceinline__ void wave_round(const double (&acc)[RS], int g0, double *red, double *mu) {
  static_assert(RS == 8 || RS == 16 || RS == 32, "round size");
  constexpr int W = 66;
  static_assert(RS * W <= 64 * (RS + 1), "the tile fits the reduction buffer");
  const int lane = lane_id();
#pragma unroll
  for (int q = 0; q < RS; ++q) red[q * W + lane] = acc[q];
  __syncthreads();
  const int q = lane & (RS - 1), part = lane / RS;
  // pairwise sum of the RS lanes' values (fixed order; a chain of log2 RS
  // dependent adds instead of RS)
  double v[RS];
  const double2 *row = reinterpret_cast<const double2 *>(red + q * W + part * RS);
#pragma unroll
  for (int l = 0; l < RS / 2; ++l) {
    const double2 t = row[l];
    v[2 * l] = t.x;
    v[2 * l + 1] = t.y;
  }
#pragma unroll
  for (int h = RS / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int l = 0; l < h; ++l) v[l] = v[l] + v[l + h];
  double t = v[0];
#pragma unroll
  for (int o = RS; o < 64; o <<= 1) t += __shfl_xor(t, o);
  if (lane < RS && g0 + lane < NM) mu[g0 + lane] = t;
  __syncthreads();
}

template <int DIM, int D2, int RPL, int RS, int G>
struct WaveMoment {
  static constexpr int NM = num_mono(DIM, D2);
  // wab = w s_x^a [s_y^b] of the current prefix, pl = powers of the last coordinate
  static __device__ __forceinline__ void run(const double (&s)[RPL][DIM], const double (&pl)[RPL][D2 + 1],
                                             double (&wa)[RPL], double (&wab)[RPL], double (&acc)[RS],
                                             double *red, double *mu) {
    constexpr LexMoments<DIM, D2> LM{};
    constexpr int ey = LM.e[G][1];
    constexpr int el = DIM == 3 ? LM.e[G][2] : LM.e[G][1];
    // a new (x[, y]) prefix starts where the last exponent is 0
    if constexpr (G > 0 && el == 0) {
      if constexpr (DIM == 3 && ey == 0) {
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
          wa[r] *= s[r][0];
          wab[r] = wa[r];
        }
      } else if constexpr (DIM == 3) {
#pragma unroll
        for (int r = 0; r < RPL; ++r) wab[r] *= s[r][1];
      } else {
#pragma unroll
        for (int r = 0; r < RPL; ++r) wab[r] *= s[r][0];
      }
    }
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < RPL; ++r) v = fma(wab[r], pl[r][el], v);
    acc[G % RS] = v;
    if constexpr (G % RS == RS - 1 || G == NM - 1) wave_round<NM, RS>(acc, G - G % RS, red, mu);
    if constexpr (G + 1 < NM) WaveMoment<DIM, D2, RPL, RS, G + 1>::run(s, pl, wa, wab, acc, red, mu);
  }
};

// (of degree <= D2: 2m for the Gram, m for the residual of the FP64 path)
template <int DIM, int D2, int RPL, int RS>
__device__ __forceinline__ void wave_moments(const double (&s)[RPL][DIM], const double (&w)[RPL], double *red,
                                             double *mu) {
  double pl[RPL][D2 + 1], wa[RPL], wab[RPL];
#pragma unroll
  for (int r = 0; r < RPL; ++r) {
    pl[r][0] = 1.0;
#pragma unroll
    for (int c = 1; c <= D2; ++c) pl[r][c] = pl[r][c - 1] * s[r][DIM - 1];
    wa[r] = w[r];
    wab[r] = w[r];
  }
  double acc[RS];
  WaveMoment<DIM, D2, RPL, RS, 0>::run(s, pl, wa, wab, acc, red, mu);
}

// sum_q e[q] Dg_q lambda_q over the nonzero entries lambda_q of a functional
// on the scaled basis (Section 2.5), Dg_q = q! dsc_q: the value reads monomial
// 0; a gradient component the linear monomial s_d (1/eps); the Laplacian the
// three pure squares s_d^2 (1/eps^2 each, their 1/2! cancelled by q!).  The
// monomial indices are compile-time, so e[] stays in registers.
template <int DIM, int ORDER, int QS, int I>
__device__ __forceinline__ double lam_term(const double (&e)[QS], const double *dsc) {
  constexpr InvFact64<DIM, ORDER> IF{};
  return e[I] * (dsc[I] * (1.0 / IF.v[I]));
}

template <int DIM, int ORDER, int QS>
__device__ __forceinline__ double lambda_dot(int kind, const double (&e)[QS], const double *dsc, double ie) {
  constexpr MonoIndex<DIM, ORDER> MI{};
  if (kind == FK_VALUE) return lam_term<DIM, ORDER, QS, 0>(e, dsc);
  if constexpr (ORDER >= 1) {
    if (kind == FK_GRAD0) return ie * lam_term<DIM, ORDER, QS, MI.idx[1][0][0]>(e, dsc);
    if (kind == FK_GRAD1) return ie * lam_term<DIM, ORDER, QS, MI.idx[0][1][0]>(e, dsc);
    if constexpr (DIM == 3)
      if (kind == FK_GRAD2) return ie * lam_term<DIM, ORDER, QS, MI.idx[0][0][1]>(e, dsc);
  }
  if constexpr (ORDER >= 2) {
    if (kind == FK_LAP) {
      double t = lam_term<DIM, ORDER, QS, MI.idx[2][0][0]>(e, dsc) + lam_term<DIM, ORDER, QS, MI.idx[0][2][0]>(e, dsc);
      if constexpr (DIM == 3) t += lam_term<DIM, ORDER, QS, MI.idx[0][0][2]>(e, dsc);
      return ie * ie * t;
    }
  }
  return 0.0;
}

// Per-block counters, added to the call's statistics once per block.
struct WaveCounts {
  unsigned long long good = 0, fell = 0;
  double cond = 0.0;
};

// Queue of one stencil set: its arguments, fallback list and counter (FP64
// path: the list in parts by bin, a counter per bin).
struct WaveSet {
  StencilArgs a;
  int *fb_list;
  int *fb_count;
};

// The rows are written in two steps: first the polynomial coefficients of
// every functional of every set, into LDS, while the rows of E^-1 (and of
// S^-1) are in registers; then the weights of every row from those
// coefficients, with the inverses dead (their registers free for the
// coefficients of the Horner steps).

// Scalar basis, coefficients: y_i / i! = dsc_i (E^-1 Dg lambda)_i of
// functional f into cf[f * 64 + i], from e = row `lane` of -E^-1.
template <int DIM, int ORDER>
__device__ __forceinline__ void wave_scalar_coefs(const StencilArgs &as, const RowKinds &rk,
                                                  const double (&e)[num_mono(DIM, ORDER)], double dsc,
                                                  const double *dscv, double ie, double *cf) {
  constexpr int QS = num_mono(DIM, ORDER);
  const int lane = lane_id();
  for (int f = 0; f < as.F; ++f) cf[f * 64 + lane] = -dsc * lambda_dot<DIM, ORDER, QS>(rk.kind[f], e, dscv, ie);
}

// Scalar basis, weights of every row of `as` (cfb: the coefficients above,
// visible to the whole wavefront).
template <int DIM, int ORDER, int RPL>
__device__ __forceinline__ void wave_scalar_weights(const StencilArgs &as, int64_t base, int N,
                                                    const double (&s)[RPL][DIM], const double (&w)[RPL],
                                                    const double *cfb) {
  constexpr int QS = num_mono(DIM, ORDER);
  const int lane = lane_id();
  const int F = as.F;
  double *wout = as.weights + (int64_t)F * base;
  for (int f = 0; f < F; ++f) {
    double cf[QS];
#pragma unroll
    for (int k = 0; k < QS; ++k) cf[k] = cfb[f * 64 + k];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = lane + 64 * r;
      const double val = w[r] * horner<DIM, ORDER>(cf, s[r]);
      if (j < N) wout[(int64_t)f * N + j] = val;
    }
  }
}

// Divergence-free basis, offsets in `big` of the coefficient step's buffers:
// [c][QM] ds_b r_b, [c][k][QM] t_b Dg_(b+e_k), then per row group g (at most
// two groups precede the divergence row) [g][c][k][QS] g / q!.
template <int DIM, int ORDER>
struct DivBuf {
  static constexpr int QS = num_mono(DIM, ORDER);
  static constexpr int QM = ORDER >= 1 ? num_mono(DIM, ORDER - 1) : 1;
  static constexpr int RB = 0, TDG = DIM * QM;
  static constexpr int CF = TDG + (DIM * QM > QS ? DIM * DIM * QM : DIM * QS);
  static constexpr int GROUP = DIM * DIM * QS;
  static constexpr int SIZE = CF + 2 * GROUP;
  // the corrected step's buffers: one group, then a reduction tile of 8
  static constexpr int RED = (CF + GROUP + 1) & ~1;
  static constexpr int REF_SIZE = RED + 8 * 66;
};

// Divergence-free basis: S = D G^-1 D^T from E^-1, equilibrated (ds_b =
// 1/sqrt(S_bb)) and swept: sr = row `lane` of -(ds S ds)^-1.  Returns false
// when S breaks down, and, where cond_max > 0, when its 1-norm condition
// number exceeds that.  `big`, vb and colb are free on entry; vb[2] holds Dg
// afterwards.
template <int DIM, int ORDER>
__device__ __forceinline__ bool wave_schur(const double (&e)[num_mono(DIM, ORDER)], double dg, const int (&ubl)[3],
                                           double *big, double (*vb)[64], double *colb, double cond_max,
                                           double (&sr)[num_mono(DIM, ORDER - 1)], double &ds) {
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int QM = num_mono(DIM, ORDER - 1);
  constexpr DivUp<DIM, ORDER> DU{};
  const int lane = lane_id();
  // S = D G^-1 D^T: S_(b,b2) = sum_k G^-1_(up[b][k], up[b2][k]); lane b holds row b
  if (lane < QS)
#pragma unroll
    for (int k = 0; k < QS; ++k) big[lane * QS + k] = e[k];
  vb[2][lane] = dg;
  __syncthreads();
  double sdiag = 1.0;
#pragma unroll
  for (int b2 = 0; b2 < QM; ++b2) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) v -= vb[2][ubl[k]] * big[ubl[k] * QS + DU.up[b2][k]] * vb[2][DU.up[b2][k]];
    sr[b2] = lane < QM ? v : 0.0;
    if (lane == b2) sdiag = v;
  }
  ds = lane < QM ? 1.0 / sqrt(sdiag) : 0.0;
  vb[3][lane] = ds;
  __syncthreads();
#pragma unroll
  for (int b2 = 0; b2 < QM; ++b2) sr[b2] *= ds * vb[3][b2];
  double rs = 0.0, anorm = 0.0;
  if (cond_max > 0.0) {
#pragma unroll
    for (int b2 = 0; b2 < QM; ++b2) rs += fabs(sr[b2]);
    anorm = wave_max(rs);
  }
  if (!sweep_inverse<QM>(sr, colb, 1e-14)) return false;  // ends with a barrier: big is free
  if (cond_max > 0.0) {
    rs = 0.0;
#pragma unroll
    for (int b2 = 0; b2 < QM; ++b2) rs += fabs(sr[b2]);
    if (!(anorm * wave_max(rs) <= cond_max)) return false;
  }
  return true;
}

// u_k = sum_b e[up[b][k]] tdg[k * QM + b], tdg in LDS
template <int DIM, int ORDER>
__device__ __forceinline__ void wave_grad_terms(const double (&e)[num_mono(DIM, ORDER)], const double *tdg,
                                                double (&u)[DIM]) {
  constexpr int QM = num_mono(DIM, ORDER - 1);
  RowVec<QM> td[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    td[k].load(tdg + k * QM);
    u[k] = 0.0;
  }
  static_for<0, QM>([&](auto B) {
    constexpr DivUp<DIM, ORDER> DU{};
    constexpr int u0 = DU.up[B][0], u1 = DU.up[B][1], u2 = DU.up[B][DIM - 1];
    if constexpr (DIM == 2)
      fmac_rows<B % 16>(u, {td[0].x[B / 16], td[1].x[B / 16]}, {e[u0], e[u1]});
    else
      fmac_rows<B % 16>(u, {td[0].x[B / 16], td[1].x[B / 16], td[2].x[B / 16]}, {e[u0], e[u1], e[u2]});
  });
}

// Coefficients of one row group (functional `kind`, components c = 0 ..
// DIM - 1) into cfb: v = G^-1 l (the same for every c), r_b = v_(b + e_c),
//   t = S^-1 r = ds (ds S ds)^-1 ds r,
//   g_(c,k) = delta_(k,c) v - G^-1 D_k^T t, D_k^T t = sum_b t_b e_(b+e_k),
// whose columns of E^-1 are this lane's registers.  KEEP_T: rb holds t [c][QM]
// afterwards.
template <int DIM, int ORDER, bool KEEP_T = false>
__device__ __forceinline__ void wave_divfree_group(int kind, const double (&e)[num_mono(DIM, ORDER)],
                                                   const double (&sr)[num_mono(DIM, ORDER - 1)], double ds, double dg,
                                                   double ifac, const int (&ubl)[3], const double *dscv, double ie,
                                                   double *rb, double *tdg, double *cfb, double (*vb)[64]) {
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int QM = num_mono(DIM, ORDER - 1);
  constexpr DivUp<DIM, ORDER> DU{};
  const int lane = lane_id();
  const double v = -dg * lambda_dot<DIM, ORDER, QS>(kind, e, dscv, ie);
  vb[1][lane] = v;
  __syncthreads();
  if (lane < QM)
#pragma unroll
    for (int c = 0; c < DIM; ++c) rb[c * QM + lane] = vb[1][ubl[c]] * ds;
  __syncthreads();
  double tk[DIM];
  {
    RowVec<QM> r[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
      r[c].load(rb + c * QM);
      tk[c] = 0.0;
    }
    static_for<0, QM>([&](auto B) {
      double x[DIM], f[DIM];
#pragma unroll
      for (int c = 0; c < DIM; ++c) {
        x[c] = r[c].x[B / 16];
        f[c] = sr[B];
      }
      fmac_rows<B % 16>(tk, x, f);
    });
  }
#pragma unroll
  for (int c = 0; c < DIM; ++c) {
    tk[c] *= -ds;
    if (lane < QM)
#pragma unroll
      for (int k = 0; k < DIM; ++k) tdg[(c * DIM + k) * QM + lane] = tk[c] * vb[2][ubl[k]];
  }
  __syncthreads();
  if constexpr (KEEP_T) {
    if (lane < QM)
#pragma unroll
      for (int c = 0; c < DIM; ++c) rb[c * QM + lane] = tk[c];
  }
#pragma unroll
  for (int c = 0; c < DIM; ++c) {
    double u[DIM];
    wave_grad_terms<DIM, ORDER>(e, tdg + c * DIM * QM, u);
    if (lane < QS)
#pragma unroll
      for (int k = 0; k < DIM; ++k) cfb[(c * DIM + k) * QS + lane] = ((k == c ? v : 0.0) + dg * u[k]) * ifac;
  }
}

// Divergence-free basis, coefficients of every row group of `av` into big
// (DivBuf).  Rows come in groups of DIM (one kind, components 0..DIM-1), then
// the divergence row.  Returns false when S breaks down (the target then goes
// to the FP64 kernel); `big`, vb and colb are free on entry.
template <int DIM, int ORDER>
__device__ __forceinline__ bool wave_divfree_coefs(const StencilArgs &av, const RowKinds &rk,
                                                   const double (&e)[num_mono(DIM, ORDER)], double dg, double ifac,
                                                   const int (&ubl)[3], const double *dscv, double ie, double *big,
                                                   double (*vb)[64], double *colb) {
  constexpr int QM = ORDER >= 1 ? num_mono(DIM, ORDER - 1) : 1;
  using DB = DivBuf<DIM, ORDER>;
  double sr[QM], ds;
  if (!wave_schur<DIM, ORDER>(e, dg, ubl, big, vb, colb, 0.0, sr, ds)) return false;
  for (int f0 = 0, g = 0; f0 < av.F; f0 += DIM, ++g) {
    const int kind = rk.kind[f0];
    if (kind == FK_DIV) break;  // identically zero on a divergence-free fit: the last row
    wave_divfree_group<DIM, ORDER>(kind, e, sr, ds, dg, ifac, ubl, dscv, ie, big + DB::RB, big + DB::TDG,
                                   big + DB::CF + g * DB::GROUP, vb);
  }
  return true;
}

// Divergence-free basis, weights of every row in the DIM functional rows from
// f0 on, from their group's coefficients (visible to the whole wavefront).
template <int DIM, int ORDER, int RPL>
__device__ __forceinline__ void wave_divfree_group_weights(double *wout, int f0, int N, const double (&s)[RPL][DIM],
                                                           const double (&w)[RPL], const double *cfb) {
  constexpr int QS = num_mono(DIM, ORDER);
  const int lane = lane_id();
#pragma unroll
  for (int c = 0; c < DIM; ++c)
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      double cf[QS];
#pragma unroll
      for (int q = 0; q < QS; ++q) cf[q] = cfb[(c * DIM + k) * QS + q];
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const int j = lane + 64 * r;
        const double val = w[r] * horner<DIM, ORDER>(cf, s[r]);
        if (j < N) wout[((int64_t)(f0 + c) * N + j) * DIM + k] = val;
      }
    }
}

// the divergence row f0: zeros
template <int DIM, int RPL>
__device__ __forceinline__ void wave_divergence_row(double *wout, int f0, int N) {
  const int lane = lane_id();
#pragma unroll
  for (int r = 0; r < RPL; ++r) {
    const int j = lane + 64 * r;
#pragma unroll
    for (int k = 0; k < DIM; ++k)
      if (j < N) wout[((int64_t)f0 * N + j) * DIM + k] = 0.0;
  }
}

// Divergence-free basis, weights of every row of `av` from the coefficients
// in big (visible to the whole wavefront).
template <int DIM, int ORDER, int RPL>
__device__ __forceinline__ void wave_divfree_weights(const StencilArgs &av, const RowKinds &rk, int64_t base,
                                                     int N, const double (&s)[RPL][DIM], const double (&w)[RPL],
                                                     const double *big) {
  using DB = DivBuf<DIM, ORDER>;
  double *wout = av.weights + (int64_t)av.F * DIM * base;
  for (int f0 = 0, g = 0; f0 < av.F; f0 += DIM, ++g) {
    if (rk.kind[f0] == FK_DIV) {
      wave_divergence_row<DIM, RPL>(wout, f0, N);
      break;  // the last row
    }
    wave_divfree_group_weights<DIM, ORDER, RPL>(wout, f0, N, s, w, big + DB::CF + g * DB::GROUP);
  }
}

// ---------------------------------------------------------------------------
// The FP64 path (REF): the coefficients above, from the moment Gram, carry
// cond(G) 2^-53; one corrected step with the residual taken over the rows
// leaves the cond(G)^1/2 2^-53 of a Householder QR (stencil_pipe64.hpp has
// the argument).  60k targets of 170 neighbours, order 4, scalar and
// divergence-free set: 7.3 ms by the shared QR kernel, 3.2 ms here.
// ---------------------------------------------------------------------------
// condition numbers (exact, 1-norm, of the equilibrated Gram and Schur
// complement) up to which the corrected step is taken; the rest go to the QR
// kernel
constexpr double kWave64Cond = 1e7;

// lexicographic index (degree <= ORDER) of basis monomial i, and the index of
// i - e_k among the monomials of degree < ORDER (-1: none)
template <int DIM, int ORDER>
struct WaveLex {
  static constexpr int Q = num_mono(DIM, ORDER);
  signed char lex[Q], down[3][Q];
  constexpr WaveLex() : lex{}, down{} {
    Mono<DIM, ORDER> M{};
    LexMoments<DIM, ORDER> L{};
    for (int i = 0; i < Q; ++i) {
      lex[i] = (signed char)L.id[M.e[i][0]][M.e[i][1]][M.e[i][2]];
      for (int k = 0; k < 3; ++k) {
        down[k][i] = -1;
        if (M.e[i][k] == 0) continue;
        int x[3] = {M.e[i][0], M.e[i][1], M.e[i][2]};
        x[k] -= 1;
        down[k][i] = (signed char)M.index(x[0], x[1], x[2]);
      }
    }
  }
};

// the functional `kind` on plain monomial `lane`
template <int DIM, int ORDER>
__device__ __forceinline__ double lane_lambda(int kind, double ie) {
  constexpr MonoIndex<DIM, ORDER> MI{};
  const int lane = lane_id();
  if (kind == FK_VALUE) return lane == 0 ? 1.0 : 0.0;
  bool hit = false;
  if constexpr (ORDER >= 1) {
    if (kind == FK_GRAD0) hit = lane == MI.idx[1][0][0];
    if (kind == FK_GRAD1) hit = lane == MI.idx[0][1][0];
    if constexpr (DIM == 3)
      if (kind == FK_GRAD2) hit = lane == MI.idx[0][0][1];
    if (kind != FK_LAP) return hit ? ie : 0.0;
  }
  if constexpr (ORDER >= 2) {
    hit = lane == MI.idx[2][0][0] || lane == MI.idx[0][2][0];
    if constexpr (DIM == 3) hit = hit || lane == MI.idx[0][0][2];
  }
  return hit ? 2.0 * ie * ie : 0.0;
}

// P^T (W P c) over the wavefront's rows, entry `lane`, c = cf[0 .. QS)
// (visible to the whole wavefront); sums: num_mono(DIM, ORDER) doubles of LDS
template <int DIM, int ORDER, int RPL, int RS>
__device__ __forceinline__ double wave_row_sums(const double (&s)[RPL][DIM], const double (&w)[RPL], const double *cf,
                                                double *red, double *sums, int lexl) {
  constexpr int QS = num_mono(DIM, ORDER);
  double c[QS], u[RPL];
#pragma unroll
  for (int q = 0; q < QS; ++q) c[q] = cf[q];
#pragma unroll
  for (int r = 0; r < RPL; ++r) u[r] = w[r] * horner<DIM, ORDER>(c, s[r]);
  wave_moments<DIM, ORDER, RPL, RS>(s, u, red, sums);
  return sums[lexl];
}

// -(E^-1 v)_lane for v in LDS
template <int QS>
__device__ __forceinline__ double row_dot(const double (&e)[QS], const double *v) {
  RowVec<QS> x;
  x.load(v);
  return row_vec_dot<QS>(e, x);
}

// Scalar basis: the corrected step on the coefficients cf[f * 64 + i].
template <int DIM, int ORDER, int RPL, int RS>
__device__ __forceinline__ void wave_scalar_refine(const StencilArgs &as, const RowKinds &rk,
                                                   const double (&e)[num_mono(DIM, ORDER)], double dsc, double ie,
                                                   const double (&s)[RPL][DIM], const double (&w)[RPL], int lexl,
                                                   double *red, double *sums, double *vec, double *cf) {
  constexpr int QS = num_mono(DIM, ORDER);
  const int lane = lane_id();
  for (int f = 0; f < as.F; ++f) {
    __syncthreads();
    const double t = wave_row_sums<DIM, ORDER, RPL, RS>(s, w, cf + f * 64, red, sums, lexl);
    vec[lane] = dsc * (lane_lambda<DIM, ORDER>(rk.kind[f], ie) - t);  // dsc is 0 from lane QS on
    __syncthreads();
    const double d = row_dot<QS>(e, vec);
    if (lane < QS) cf[f * 64 + lane] -= dsc * d;
  }
}

// Divergence-free basis: S, then per row group the coefficients, the
// corrected step and the weights.  The step's residual, per component c and
// k: rho_k = delta_(k,c) lambda - G g_k - D_k^T t (G g_k over the rows), and
// D g; then dv_k = G^-1 rho_k, S dt = D (dv + g), g_k += dv_k - G^-1 D_k^T dt.
// Returns false where S breaks down or its condition number is too large.
template <int DIM, int ORDER, int RPL>
__device__ __forceinline__ bool wave_divfree_refined(const StencilArgs &av, const RowKinds &rk,
                                                     const double (&e)[num_mono(DIM, ORDER)], double dsc, double ifac,
                                                     const int (&ubl)[3], const int (&dnl)[3], int lexl,
                                                     const double *dscv, double ie, int64_t base, int N,
                                                     const double (&s)[RPL][DIM], const double (&w)[RPL], double *big,
                                                     double *sums, double (*vb)[64], double *colb) {
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int QM = num_mono(DIM, ORDER - 1);
  constexpr DivUp<DIM, ORDER> DU{};
  using DB = DivBuf<DIM, ORDER>;
  const int lane = lane_id();
  const double dg = dsc / ifac;
  double sr[QM], ds;
  if (!wave_schur<DIM, ORDER>(e, dg, ubl, big, vb, colb, kWave64Cond, sr, ds)) return false;
  double *rb = big + DB::RB, *tdg = big + DB::TDG, *cfb = big + DB::CF, *red = big + DB::RED;
  double *wout = av.weights + (int64_t)av.F * DIM * base;
  for (int f0 = 0; f0 < av.F; f0 += DIM) {
    const int kind = rk.kind[f0];
    if (kind == FK_DIV) {
      wave_divergence_row<DIM, RPL>(wout, f0, N);
      break;
    }
    wave_divfree_group<DIM, ORDER, true>(kind, e, sr, ds, dg, ifac, ubl, dscv, ie, rb, tdg, cfb, vb);
    const double lam = lane_lambda<DIM, ORDER>(kind, ie);
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
      double dv[DIM];
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        __syncthreads();
        double *cf = cfb + (c * DIM + k) * QS;
        const double t = wave_row_sums<DIM, ORDER, RPL, 8>(s, w, cf, red, sums, lexl);
        // plain monomials: the scaled basis' entries times i!
        double rho = (k == c ? lam : 0.0) - t;
        if (dnl[k] >= 0) rho -= rb[c * QM + dnl[k]] / ifac;
        vb[1][lane] = dsc * rho;
        __syncthreads();
        dv[k] = -dsc * row_dot<QS>(e, vb[1]);
        // (dv_k + g_k) of the scaled basis, for the constraint
        if (lane < QS) tdg[k * QS + lane] = (dv[k] + cf[lane]) / ifac;
      }
      __syncthreads();
      double sg = 0.0;
      if (lane < QM) {
#pragma unroll
        for (int k = 0; k < DIM; ++k) sg += tdg[k * QS + ubl[k]];
      }
      vb[1][lane] = ds * sg;
      __syncthreads();
      const double dt = -ds * row_dot<QM>(sr, vb[1]);
      if (lane < QM) {
#pragma unroll
        for (int k = 0; k < DIM; ++k) tdg[k * QM + lane] = dt * vb[2][ubl[k]];
      }
      __syncthreads();
      double u[DIM];
      wave_grad_terms<DIM, ORDER>(e, tdg, u);
      if (lane < QS)
#pragma unroll
        for (int k = 0; k < DIM; ++k) cfb[(c * DIM + k) * QS + lane] += dv[k] + dsc * u[k];
    }
    __syncthreads();
    wave_divfree_group_weights<DIM, ORDER, RPL>(wout, f0, N, s, w, cfb);
    __syncthreads();
  }
  return true;
}

// BASIS 0 scalar set (ss), 1 divergence-free set (sv), 3 both on the same
// neighbour lists: the moments and the swept Gram are formed once per target
// for both sets (Section 2.2: the divergence-free fit is the scalar fit under
// D c = 0, so both take the same G).
// CAND: the compiled variant (kWaveCand).  REF: the FP64 path (the corrected
// step; targets it does not take go to the QR kernel, and neither the mixed
// path's options nor its statistics apply).
template <int DIM, int ORDER, int BASIS, int RPL, int CAND, bool REF = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaveCand[CAND].wpe))) void k_wave(
    WaveSet ss, WaveSet sv, const int *list, BinMeta *meta, int bin, Stats *stats, Options opt) {
  constexpr bool SCAL = BASIS == 0 || BASIS == 3, DIVF = BASIS == 1 || BASIS == 3;
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int NM = num_mono(DIM, 2 * ORDER);
  constexpr int QM = ORDER >= 1 ? num_mono(DIM, ORDER - 1) : 1;
  constexpr int RS = kWaveCand[CAND].rs;
  constexpr int RED = 64 * (RS + 1);
  constexpr int BIG = (DIVF && QS * QS > RED) ? QS * QS : RED;
  static_assert(QS <= 64, "one basis function per lane");
  static_assert(!DIVF || DivBuf<DIM, ORDER>::SIZE <= BIG, "divergence-free buffers fit");
  static_assert(5 * 64 <= BIG, "scalar coefficients fit");
  static_assert(!REF || !DIVF || DivBuf<DIM, ORDER>::REF_SIZE <= BIG, "the corrected step's buffers fit");
  __shared__ __align__(16) double big[BIG];  // moment reduction, then (divergence-free) -E^-1
  __shared__ double mu[NM];        // moments, lexicographic order
  __shared__ double vb[4][64];     // broadcast vectors
  __shared__ __align__(16) double colb[4 * 64];  // pivot columns of the sweeps
  __shared__ unsigned char pidx[QS * QS];
  // the scalar set's coefficients [f][64]: their own buffer when the
  // divergence-free set's coefficients take `big` (shared calls), or the
  // residual's reductions do
  constexpr bool OWN = BASIS == 3 || (REF && SCAL);
  __shared__ double cfs_own[OWN ? 5 * 64 : 1];
  double *cfs = OWN ? cfs_own : big;
  constexpr WavePairs<DIM, ORDER> WP{};
  constexpr InvFact64<DIM, ORDER> IF{};
  const StencilArgs &a = SCAL ? ss.a : sv.a;  // the common inputs
  const int lane = lane_id();
  for (int q = lane; q < QS * QS; q += 64) pidx[q] = WP.p[q];
  const double ifac = IF.v[lane < QS ? lane : 0];  // 1 / i!
  int ubl[3] = {0, 0, 0};                             // divergence-free: index of b + e_k, b = lane
  if constexpr (DIVF) {
    constexpr DivUp<DIM, ORDER> DU{};
    if (lane < QM)
#pragma unroll
      for (int k = 0; k < DIM; ++k) ubl[k] = DU.up[lane][k];
  }
  int lexl = 0, dnl[3] = {-1, -1, -1};  // corrected step: lexicographic index of monomial `lane`, that of lane - e_k
  if constexpr (REF) {
    constexpr WaveLex<DIM, ORDER> WL{};
    if (lane < QS) {
      lexl = WL.lex[lane];
#pragma unroll
      for (int k = 0; k < DIM; ++k) dnl[k] = WL.down[k][lane];
    }
  }
  __syncthreads();
  const RowKinds rks = row_kinds(DIM, 0, ss.a.mask), rkv = row_kinds(DIM, 1, sv.a.mask);
  WaveCounts cnt, cntv;
  const SlotRange R = slot_range(meta, bin, -1, INT_MAX);
  const int left0 = R.first;  // the bin's part of the FP64 path's queues
  for (int i = R.first + xcd_block(); i < R.last; i += gridDim.x) {
    const int t = list[i];
    const int64_t base = a.row_ptr[t];
    const int N = (int)(a.row_ptr[t + 1] - base);
    const double ie = 1.0 / a.eps[t];
    double xt[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) xt[d] = a.targets[(int64_t)t * DIM + d];
    double s[RPL][DIM], w[RPL];
    {
      double xs[RPL][DIM];
      gather_rows<DIM, RPL, 64>(a, base, N, lane, xs);
#pragma unroll
      for (int r = 0; r < RPL; ++r) w[r] = row_sw<DIM, REF>(xs[r], xt, ie, a.p, lane + 64 * r < N, s[r]);
    }
    wave_moments<DIM, 2 * ORDER, RPL, RS>(s, w, big, mu);

    // equilibrated Gram, row `lane` (lanes >= QS hold zeros; li keeps their
    // table reads in bounds)
    const int li = lane < QS ? lane : 0;
    const double dsc = lane < QS ? 1.0 / sqrt(mu[pidx[li * QS + li]]) : 0.0;
    vb[0][lane] = dsc;
    __syncthreads();
    double e[QS];
#pragma unroll
    for (int k = 0; k < QS; ++k) {
      // every lane loads (li is in range), so the QS reads go out together
      const double v = mu[pidx[li * QS + k]] * dsc * vb[0][k];
      e[k] = lane < QS ? v : 0.0;
    }
    double rs = 0.0;
#pragma unroll
    for (int k = 0; k < QS; ++k) rs += fabs(e[k]);
    const double anorm = wave_max(rs);
    bool ok = sweep_inverse<QS>(e, colb, 1e-14);  // e = row `lane` of -E^-1
    rs = 0.0;
#pragma unroll
    for (int k = 0; k < QS; ++k) rs += fabs(e[k]);
    const double cond = anorm * wave_max(rs);
    if constexpr (REF) {
      if (!(cond <= kWave64Cond)) ok = false;
    } else {
      if (lane == 0 && a.cond_out) a.cond_out[t] = (float)cond;
      if (!(cond <= opt.cond_threshold)) ok = false;
      if (opt.force_fallback) ok = false;
    }
    const double dg = dsc / ifac;  // Dg_lane: G^-1 = Dg E^-1 Dg

    // the coefficients of both sets while the inverse rows are in
    // registers, then the weights of every row with those registers free
    if constexpr (SCAL)
      if (ok) wave_scalar_coefs<DIM, ORDER>(ss.a, rks, e, dsc, vb[0], ie, cfs);
    if constexpr (REF && SCAL)
      if (ok) wave_scalar_refine<DIM, ORDER, RPL, RS>(ss.a, rks, e, dsc, ie, s, w, lexl, big, mu, vb[1], cfs);
    bool okv = ok;
    if constexpr (REF && DIVF) {
      __syncthreads();
      if (ok)
        okv = wave_divfree_refined<DIM, ORDER, RPL>(sv.a, rkv, e, dsc, ifac, ubl, dnl, lexl, vb[0], ie, base, N, s, w,
                                                    big, mu, vb, colb);
    }
    if constexpr (!REF && DIVF)
      if (ok) okv = wave_divfree_coefs<DIM, ORDER>(sv.a, rkv, e, dg, ifac, ubl, vb[0], ie, big, vb, colb);
    __syncthreads();
    if constexpr (SCAL) {
      if (ok) wave_scalar_weights<DIM, ORDER, RPL>(ss.a, base, N, s, w, cfs);
      if (lane == 0) {
        ss.a.status[t] = ok ? GMLS_TARGET_OK : GMLS_TARGET_FALLBACK;
        if (!ok) ss.fb_list[REF ? left0 + atomicAdd(ss.fb_count + bin, 1) : atomicAdd(ss.fb_count, 1)] = t;
      }
    }
    if constexpr (DIVF) {
      if constexpr (!REF)
        if (okv) wave_divfree_weights<DIM, ORDER, RPL>(sv.a, rkv, base, N, s, w, big);
      if (lane == 0) {
        sv.a.status[t] = okv ? GMLS_TARGET_OK : GMLS_TARGET_FALLBACK;
        if (!okv) sv.fb_list[REF ? left0 + atomicAdd(sv.fb_count + bin, 1) : atomicAdd(sv.fb_count, 1)] = t;
      }
    }
    __syncthreads();
    const bool good = SCAL ? ok : okv;  // statistics of the first set
    cnt.good += good ? 1 : 0;
    cnt.fell += good ? 0 : 1;
    if (cond >= 0.0) cnt.cond = fmax(cnt.cond, cond);  // NaN estimates are skipped
    if constexpr (BASIS == 3) {  // the divergence-free set of a shared call: its own counters
      cntv.good += okv ? 1 : 0;
      cntv.fell += okv ? 0 : 1;
    }
  }
  if (!REF && lane == 0) {
    if (cnt.good) atomicAdd(&stats->sweep_hist[0], cnt.good);
    if (cnt.fell) atomicAdd(&stats->n_fallback, cnt.fell);
    if (cnt.cond > 0.0) atomicMax(&stats->cond_max_bits, (unsigned long long)__double_as_longlong(cnt.cond));
    if constexpr (BASIS == 3) {  // stats[1]: the second set (shared calls pass two records)
      if (cntv.good) atomicAdd(&stats[1].sweep_hist[0], cntv.good);
      if (cntv.fell) atomicAdd(&stats[1].n_fallback, cntv.fell);
      if (cnt.cond > 0.0)
        atomicMax(&stats[1].cond_max_bits, (unsigned long long)__double_as_longlong(cnt.cond));
    }
  }
}

// One launch per non-empty row-count bin (bin b: rows <= 64 b, b rows per
// lane).  With a host copy of the bin table (hm) empty bins are skipped and
// grids sized to the bin; without one every bin is launched, sized for n_max
// targets, its bounds read on the device.
template <int DIM, int ORDER, int BASIS>
hipError_t launch_wave(const WaveSet &ss, const WaveSet &sv, const int *list, const BinMeta *hm, BinMeta *meta,
                       Stats *stats, const Options &opt, int n_max, int cus, PipeTimer *timer, hipStream_t s) {
  for (int b = 1; b < kNumBins; ++b) {
    int cnt = n_max;
    if (hm) {
      cnt = hm->count[b];
      if (cnt == 0) continue;
    }
    if (b == kLongBin) {  // rows over 256: the FP64 QR kernels take them in chunks
      hipError_t e = hipSuccess;
      if constexpr (BASIS == 0 || BASIS == 3)
        e = launch_defer_bin(ss.a.status, list, meta, b, ss.fb_list, ss.fb_count, stats, s);
      if constexpr (BASIS == 1 || BASIS == 3)
        if (e == hipSuccess)
          e = launch_defer_bin(sv.a.status, list, meta, b, sv.fb_list, sv.fb_count, BASIS == 3 ? stats + 1 : stats,
                               s);
      if (e != hipSuccess) return e;
      continue;
    }
    int nb = cnt < cus * 16 ? cnt : cus * 16;
    nb = xcd_grid(nb);
    const int c = opt.wave_shape[b] >= 0 && opt.wave_shape[b] < kWaveCands ? opt.wave_shape[b] : 0;
    if (timer) {
      const hipError_t e = hipEventRecord(timer->ev[2][b][0], s);
      if (e != hipSuccess) return e;
    }
    switch (b * 4 + c) {
#define GMLS_WAVE_CASE(B_, C_)                                                                                  \
  case B_ * 4 + C_:                                                                                             \
    k_wave<DIM, ORDER, BASIS, B_, C_><<<nb, 64, 0, s>>>(ss, sv, list, meta, b, stats, opt);                     \
    break;
      GMLS_WAVE_CASE(1, 0) GMLS_WAVE_CASE(1, 1) GMLS_WAVE_CASE(1, 2)
      GMLS_WAVE_CASE(2, 0) GMLS_WAVE_CASE(2, 1) GMLS_WAVE_CASE(2, 2)
      GMLS_WAVE_CASE(3, 0) GMLS_WAVE_CASE(3, 1) GMLS_WAVE_CASE(3, 2)
      GMLS_WAVE_CASE(4, 0) GMLS_WAVE_CASE(4, 1) GMLS_WAVE_CASE(4, 2)
#undef GMLS_WAVE_CASE
      default: return hipErrorInvalidValue;
    }
    if (timer) {
      const hipError_t e = hipEventRecord(timer->ev[2][b][1], s);
      if (e != hipSuccess) return e;
      timer->used[2][b] = 1;
    }
  }
  return hipGetLastError();
}

// The FP64 path: as launch_wave, in the default variant, without the long bin.
template <int DIM, int ORDER, int BASIS>
hipError_t launch_wave64(const WaveSet &ss, const WaveSet &sv, const int *list, const BinMeta *hm, BinMeta *meta,
                         int n_max, int cus, hipStream_t s) {
  const Options opt;
  for (int b = 1; b < kLongBin; ++b) {
    int cnt = n_max;
    if (hm) {
      cnt = hm->count[b];
      if (cnt == 0) continue;
    }
    const int nb = xcd_grid(cnt < cus * 16 ? cnt : cus * 16);
    switch (b) {
      case 1: k_wave<DIM, ORDER, BASIS, 1, 0, true><<<nb, 64, 0, s>>>(ss, sv, list, meta, b, nullptr, opt); break;
      case 2: k_wave<DIM, ORDER, BASIS, 2, 0, true><<<nb, 64, 0, s>>>(ss, sv, list, meta, b, nullptr, opt); break;
      case 3: k_wave<DIM, ORDER, BASIS, 3, 0, true><<<nb, 64, 0, s>>>(ss, sv, list, meta, b, nullptr, opt); break;
      case 4: k_wave<DIM, ORDER, BASIS, 4, 0, true><<<nb, 64, 0, s>>>(ss, sv, list, meta, b, nullptr, opt); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace gmls
