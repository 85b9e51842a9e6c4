// stencil_pipe.hpp -- mixed-precision stencils as a three-kernel pipeline for
// small scalar bases (Q <= 20: 3D order <= 3, 2D order <= 4).
//
// The stencil of a functional lambda is alpha = W P y with (P^T W P) y = lambda
// (Section 2.1, normal equations; Section 2.5, functionals on the basis).
//
//  A. moments (a group of G lanes per target, rows spread over the group):
//     mu_g = sum_j w_j s_j^g for |g| <= 2m in FP64, reduce-scattered over the
//     group and stored to HBM, moment-major [g][slot];
//  B. solve (one thread per target, the whole system in registers):
//     A64_ab = mu_(a+b)/(a! b!) is the Gram; its Jacobi-equilibrated FP32
//     copy is factored by a fully unrolled packed Cholesky, its 1-norm
//     condition number is estimated (Hager's estimator, three solves), then
//     y = D A~^-1 D lambda is refined with FP64 residuals r = lambda - A64 y
//     (FP32 correction, FP64 accumulation) until the predicted error
//     rho*|dy| <= tol*|y|; y_a / a!, the coefficients of the plain monomials,
//     are stored to HBM, [slot][f][a];
//  C. weights (a group of G lanes per target): alpha_j = w_j p(s_j) . y in
//     FP64, the rows gathered again.
// Targets that break down, exceed the condition threshold or do not converge
// are queued for the FP64 QR fallback.  Every lane of kernel B runs the same
// instruction stream (no row-count divergence), and no lane is idle.
#pragma once

#include <float.h>
#include <limits.h>
#include <math.h>

#include "basis.hpp"
#include "gmls_internal.hpp"
#include "stencil_mixed64.hpp"

namespace gmls {

// Per-target record of one pipeline chunk, in list-slot order, so that the
// three kernels read what they need about a target with one coalesced load
// instead of a chain of scattered ones (list -> row_ptr, eps, coordinates).
struct PipeRec {
  int64_t base;  // row_ptr[t]
  int n;         // row count
  int t;         // target index
  double ie;     // 1 / eps_t
  double x[3];   // target coordinates
  int ok;        // written by the solve: 1 = weights to be formed here
  int pad;
  double pad2;
};
static_assert(sizeof(PipeRec) == kPipeRecBytes, "record size");

// List slots a launch covers: bin `bin` (0: bins 1..4 together) clipped to
// the window [win_lo, win_hi); win_lo < 0 opens the window at the first slot
// of bin 1.  c0 is the window's first slot (records and buffers are indexed
// from it).  The bounds come from the device bin table, so a launch needs no
// host copy of it.
struct SlotRange {
  int first, last, c0;
};

__device__ __forceinline__ SlotRange slot_range(const BinMeta *meta, int bin, int win_lo, int win_hi) {
  const int c0 = win_lo >= 0 ? win_lo : meta->offset[1];
  int lo, hi;
  if (bin > 0) {
    lo = meta->offset[bin];
    hi = lo + meta->count[bin];
  } else {
    lo = meta->offset[1];
    hi = meta->offset[kNumBins - 1] + meta->count[kNumBins - 1];
  }
  lo = lo > c0 ? lo : c0;
  hi = hi < win_hi ? hi : win_hi;
  return {readfirstlane_i(lo), readfirstlane_i(hi), readfirstlane_i(c0)};
}

// The FP64 path's queues: the targets t of list slots `slot` that a lane leaves
// to the QR kernel, in their bin's part of left_list (in any order), one atomic
// per wavefront and bin.  All lanes take part.
__device__ __forceinline__ void leave_targets(bool leave, int slot, int t, const BinMeta *meta, int *left_list,
                                              int *left) {
  if (__ballot(leave) == 0) return;
  for (int b = 1; b < kNumBins; ++b) {
    const int lo = meta->offset[b];
    uint64_t m;
    const bool mine = leave && slot >= lo && slot < lo + meta->count[b];
    const int k = ballot_prefix(mine, &m);
    if (m == 0) continue;
    int base = 0;
    if (lane_id() == 0) base = atomicAdd(left + b, __popcll(m));
    base = lo + __builtin_amdgcn_readfirstlane(base);
    if (mine) left_list[base + k] = t;
  }
}

template <int DIM>
__global__ __launch_bounds__(256) void k_pipe_prep(StencilArgs a, const int *list, const BinMeta *meta, int win_lo,
                                                   int win_hi, PipeRec *rec) {
  const SlotRange R = slot_range(meta, 0, win_lo, win_hi);
  const int first = R.first, last = R.last;
  for (int i = first + blockIdx.x * blockDim.x + threadIdx.x; i < last; i += gridDim.x * blockDim.x) {
    const int t = list[i];
    PipeRec r;
    r.base = a.row_ptr[t];
    r.n = (int)(a.row_ptr[t + 1] - r.base);
    r.t = t;
    r.ie = 1.0 / a.eps[t];
    for (int d = 0; d < 3; ++d) r.x[d] = d < DIM ? a.targets[(int64_t)t * DIM + d] : 0.0;
    r.ok = 0;
    r.pad = 0;
    rec[i - R.c0] = r;
  }
}

// ---------------------------------------------------------------------------
// A. moments
// ---------------------------------------------------------------------------
// v of the other lane of the pair (2i, 2i + 1)
__device__ __forceinline__ int64_t swap_lanes(int64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0xB1, 0xF, 0xF, true);
  return ((int64_t)hi << 32) | (uint32_t)lo;
}

// Rows j = lg + G*r (r < RPL) of a target, gathered without branches: rows
// past N re-read row N-1 and get weight 0, so all column indices, then all
// coordinates, are requested together (two memory round trips per target
// instead of two per row).
template <int DIM, int RPL, int G, bool PAIR = false>
__device__ __forceinline__ void gather_rows(const StencilArgs &a, int64_t base, int N, int lg,
                                            double (&xs)[RPL][DIM]) {
  int c[RPL];
#pragma unroll
  for (int r = 0; r < RPL; ++r) {
    const int j = lg + G * r;
    c[r] = a.col[base + (j < N ? j : N - 1)];
  }
  if constexpr (DIM == 2 || !PAIR) {
#pragma unroll
    for (int r = 0; r < RPL; ++r)
#pragma unroll
      for (int d = 0; d < DIM; ++d) xs[r][d] = a.coords[(int64_t)c[r] * a.cstride + d];
  } else {
    // Lanes 2i and 2i + 1 fetch their two rows' records together, first the
    // even lane's, then the odd lane's: one of them (x, y), the other (y, z).
    // An instruction then touches 32 cache lines, not 64 (weights 710 -> 622 us
    // for 1M targets of 60 rows, 855 -> 786 for 1M of 95 random rows; not the
    // moment kernel, 1110 -> 1240, whose registers are full).
    typedef double Two __attribute__((ext_vector_type(2), aligned(8)));
    const bool odd = lg & 1;
    Two u[RPL], v[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int64_t p = (int64_t)(a.coords + (int64_t)c[r] * a.cstride), q = swap_lanes(p) + 8;
      u[r] = *(const Two *)(odd ? q : p);
      v[r] = *(const Two *)(odd ? p : q);
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      xs[r][0] = odd ? v[r].x : u[r].x;
      xs[r][1] = odd ? v[r].y : u[r].y;
      xs[r][2] = __builtin_bit_cast(double, swap_lanes(__builtin_bit_cast(int64_t, odd ? u[r].y : v[r].y)));
    }
  }
}

// scaled offset s = (x_j - x_T)/eps and kernel weight (1 - |s|)^p (0 outside
// the support, and 0 when `live` is false); base: 1 - |s| in its place
// EXACT: good to an ulp, what the FP64 path takes its weights from
template <int DIM, bool EXACT = true, bool BASE = false>
__device__ __forceinline__ double row_sw(const double *xj, const double *xt, double ie, int p, bool live,
                                         double *s) {
  double rr = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    s[d] = (xj[d] - xt[d]) * ie;
    rr += s[d] * s[d];
  }
  // |s| from the hardware reciprocal square root and one Newton step for the
  // square root (relative error about the square of the estimate's, far
  // below the mixed path's tolerance), EXACT after one for the estimate
  // itself, in place of the correctly rounded sqrt sequence; the support test
  // uses |s|^2 itself
  double y = __builtin_amdgcn_rsq(rr);
  if constexpr (EXACT) y = fma(y, fma(-(0.5 * rr) * y, y, 0.5), y);
  const double r0 = rr * y;
  const double rad = rr > 0.0 ? fma(fma(-r0, r0, rr), 0.5 * y, r0) : 0.0;
  if constexpr (BASE) return live && rr < 1.0 ? 1.0 - rad : 0.0;
  return (live && rr < 1.0) ? int_pow(1.0 - rad, p) : 0.0;
}

// The same of all of a lane's rows, the powers multiplied up together in one
// uniform loop over p: with a loop per row behind the support test's branch
// the rows' arithmetic stays apart.  Faster where the rows' offsets are kept
// anyway (weights and sums, 3 to 5 %); the moment kernel, whose sums fill the
// registers, forms one row at a time (1110 against 1250 us at 16 x 8, order 3).
template <int DIM, int RPL, class Live>
__device__ __forceinline__ void rows_sw(const double (&xs)[RPL][DIM], const double *xt, double ie, int p, Live live,
                                        double (&s)[RPL][DIM], double (&w)[RPL]) {
  double b[RPL];
#pragma unroll
  for (int r = 0; r < RPL; ++r) w[r] = b[r] = row_sw<DIM, true, true>(xs[r], xt, ie, p, live(r), s[r]);
  for (int q = 1; q < p; ++q)  // 1 <= p <= 12
#pragma unroll
    for (int r = 0; r < RPL; ++r) w[r] *= b[r];
}

// Trip count of the chunk loop over a row: one pass of G * RPL rows, or for
// the long bin (LOOP) enough passes for the longest row of the wavefront's
// targets (the same for every lane: the loop holds no divergent barrier).
template <bool LOOP, int CH>
__device__ __forceinline__ int chunk_end(int N) {
  if constexpr (!LOOP) {
    return 1;
  } else {
    int m = N;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = max(m, __shfl_xor(m, o));
    return readfirstlane_i(m);
  }
}

// `t` is a target of the bin even for an invalid group (whose sums are not
// stored), so that every gathered row exists.  LOOP: rows in chunks of
// G * RPL (the long bin), the partial sums carried over the chunks.
template <int DIM, int ORDER, int G, int RPL, bool LOOP = false>
__device__ void pipe_moments_target(const StencilArgs &a, const PipeRec &rc, bool valid, int slot, int lg,
                                    double *mom) {
  constexpr int NM = num_mono(DIM, 2 * ORDER);
  constexpr int RS = 32;  // moments per LDS reduction round
  constexpr int RW = 66;  // row of the reduction tile: one moment, 64 lanes (+2: rows start in other banks)
  __shared__ __align__(16) double red[RS * RW];
  const int64_t base = rc.base;
  const int N = rc.n;
  const double ie = rc.ie;
  double xt[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) xt[d] = rc.x[d];
  double mu[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) mu[m] = 0.0;
  constexpr MomentSplit<DIM, ORDER> MS{};
  const int cend = chunk_end<LOOP, G * RPL>(N);
  for (int c0 = 0; c0 < cend; c0 += G * RPL) {
    const int nrem = N - c0;  // rows of this chunk and after (may be <= 0 in a long loop)
    double xs[RPL][DIM];
    gather_rows<DIM, RPL, G>(a, base + (nrem > 0 ? c0 : 0), nrem > 0 ? nrem : N, lg, xs);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      double s[DIM];
      const double w = row_sw<DIM>(xs[r], xt, ie, a.p, lg + G * r < nrem, s);
      double lastp[2 * ORDER + 1];
      lastp[0] = 1.0;
#pragma unroll
      for (int c = 1; c <= 2 * ORDER; ++c) lastp[c] = lastp[c - 1] * s[DIM - 1];
      double wp[MS.NP];
      wp[0] = w;
#pragma unroll
      for (int pi = 1; pi < MS.NP; ++pi) wp[pi] = wp[MS.parent[pi]] * s[MS.pdim[pi]];
#pragma unroll
      for (int pi = 0; pi < MS.NP; ++pi)
#pragma unroll
        for (int c = 0; c <= 2 * ORDER - MS.deg[pi]; ++c) mu[MS.midx[pi][c]] += wp[pi] * lastp[c];
    }
  }
  // the sums are complete here: without this the compiler sinks each
  // moment's FMA chain into the reduction round that stores it and keeps
  // every row's products live until then
#pragma unroll
  for (int m = 0; m < NM; ++m) asm volatile("" : "+v"(mu[m]));
  // sum the G lanes' partial moments through LDS, RS moments per round:
  // every lane writes its partials (moment q of lane L at q * RW + L), then
  // lane lg of the group adds moment lg + G*k (< RS) over the group's lanes,
  // in lane order, reading them two at a time (the group's lanes are
  // contiguous in a moment's row), and stores it
  const int lane = lane_id(), grp0 = lane - lg;
#pragma unroll
  for (int r0 = 0; r0 < NM; r0 += RS) {
#pragma unroll
    for (int q = 0; q < RS; ++q) red[q * RW + lane] = r0 + q < NM ? mu[r0 + q] : 0.0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < (RS + G - 1) / G; ++k) {
      const int q = lg + G * k;
      if (q < RS) {
        const double2 *row = reinterpret_cast<const double2 *>(red + q * RW + grp0);
        double acc = 0.0;
#pragma unroll
        for (int l = 0; l < G / 2; ++l) {
          const double2 t = row[l];
          acc += t.x;
          acc += t.y;
        }
        if (valid && r0 + q < NM) mom[(int64_t)slot * NM + r0 + q] = acc;
      }
    }
    __syncthreads();
  }
}

// Targets list[first .. last) of one row-count bin; moment g of the target
// in list slot i goes to mom[(i - c0) * NM + g] (target-major, so that a
// group writes its target's moments contiguously).
template <int DIM, int ORDER, int G, int RPL, bool LOOP = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_pipe_moments(
    StencilArgs a, const PipeRec *rec, const BinMeta *meta, int bin, int win_lo, int win_hi, double *mom) {
  const SlotRange R = slot_range(meta, bin, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  constexpr int TPW = 64 / G;
  const int lane = lane_id();
  const int grp = lane / G, lg = lane % G;
  for (int i0 = first + xcd_block() * TPW; i0 < last; i0 += gridDim.x * TPW) {
    const int i = i0 + grp;
    const bool valid = i < last;
    const PipeRec rc = rec[(valid ? i : first) - c0];
    pipe_moments_target<DIM, ORDER, G, RPL, LOOP>(a, rc, valid, i - c0, lg, mom);
  }
}

// ---------------------------------------------------------------------------
// B. solve, one thread per target
// ---------------------------------------------------------------------------
template <int Q>
struct Packed {
  static constexpr int n = Q * (Q + 1) / 2;
  static constexpr int at(int i, int k) { return i * (i + 1) / 2 + k; }  // k <= i
};

// x <- (L L^T)^-1 x for a packed lower-triangular L whose diagonal slots hold
// 1/L_jj (registers, fully unrolled)
template <int Q>
__device__ __forceinline__ void packed_solve(const float (&L)[Q * (Q + 1) / 2], float (&x)[Q]) {
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    float v = x[i];
#pragma unroll
    for (int k = 0; k < i; ++k) v -= L[Packed<Q>::at(i, k)] * x[k];
    x[i] = v * L[Packed<Q>::at(i, i)];
  }
#pragma unroll
  for (int i = Q - 1; i >= 0; --i) {
    float v = x[i];
#pragma unroll
    for (int k = i + 1; k < Q; ++k) v -= L[Packed<Q>::at(k, i)] * x[k];
    x[i] = v * L[Packed<Q>::at(i, i)];
  }
}

// All (a, b) pairs of the Q x Q moment Gram ordered by the moment index of
// a + b, so that the residual streams each moment once.
template <int DIM, int ORDER>
struct MomentPairs {
  static constexpr int Q = num_mono(DIM, ORDER);
  static constexpr int NM = num_mono(DIM, 2 * ORDER);
  static constexpr int P = Q * Q;
  int m[P], a[P], b[P];
  constexpr MomentPairs() : m{}, a{}, b{} {
    SumIndex<DIM, ORDER> S{};
    int p = 0;
    for (int g = 0; g < NM; ++g)
      for (int i = 0; i < Q; ++i)
        for (int k = 0; k < Q; ++k)
          if (S.idx[i][k] == g) {
            m[p] = g;
            a[p] = i;
            b[p] = k;
            ++p;
          }
  }
};

// SKIP = 1 (staggered stencils): the constant monomial is not a column, so
// the Gram is the trailing (Q-1) x (Q-1) block of the moment Gram and the
// functionals act on monomials 1..Q-1.
template <int DIM, int ORDER, int SKIP = 0>
__global__ __launch_bounds__(64) void k_pipe_solve(StencilArgs a, PipeRec *rec, int win_lo, int win_hi,
                                                   const double *mom, double *yout, int *fb_list, BinMeta *meta,
                                                   Stats *stats, Options opt) {
  constexpr int Q = num_mono(DIM, ORDER) - SKIP;
  constexpr int NP = Q * (Q + 1) / 2;
  constexpr InvFact64<DIM, ORDER> IF{};
  constexpr SumIndex<DIM, ORDER> SI{};
  constexpr MomentPairs<DIM, ORDER> MP{};
  constexpr int NM = MomentPairs<DIM, ORDER>::NM;
  // thread-private LDS columns (lane l uses [.][l] only)
  __shared__ double mls[NM][64];  // FP64 moments of this thread's target
  __shared__ double ybuf[Q][64];  // this thread's solution
  const int lane = lane_id();
  const RowKinds rk = row_kinds(DIM, 0, a.mask);
  const int F = a.F;
  const SlotRange R = slot_range(meta, 0, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  for (int slot = first + xcd_block() * 64 + lane; slot - lane < last; slot += gridDim.x * 64) {
    const bool valid = slot < last;
    const int sl = valid ? slot : first;
    const int t = rec[sl - c0].t;
    const double ie = rec[sl - c0].ie;
    const int64_t loc = sl - c0;
    // stage this thread's moments into its LDS column; the wave's 84 loads
    // walk one contiguous block of 64*NM doubles, so lines are reused from L1
    if (valid) {
#pragma unroll
      for (int m = 0; m < NM; ++m) mls[m][lane] = mom[loc * NM + m];
    }
#define GMLS_MU(g, off) mls[(g)][lane + (off)]
    // equilibration D_a = 1/sqrt(A64_aa) = a!/sqrt(mu_2a); equilibrated FP32
    // Gram D A64 D, packed lower
    float dsc[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i)
      dsc[i] = (float)(1.0 / IF.v[i + SKIP]) * rsqrtf((float)GMLS_MU(SI.idx[i + SKIP][i + SKIP], 0));
    float L[NP];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const double di = (double)dsc[i] * IF.v[i + SKIP];
#pragma unroll
      for (int k = 0; k <= i; ++k)
        L[Packed<Q>::at(i, k)] =
            (float)(GMLS_MU(SI.idx[i + SKIP][k + SKIP], 0) * di * ((double)dsc[k] * IF.v[k + SKIP]));
    }
    float anorm = 0.f;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < Q; ++i) sum += fabsf(i >= k ? L[Packed<Q>::at(i, k)] : L[Packed<Q>::at(k, i)]);
      anorm = fmaxf(anorm, sum);
    }
    // Cholesky in place; the diagonal keeps 1/L_jj
    bool ok = valid;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      float dj = L[Packed<Q>::at(j, j)];
#pragma unroll
      for (int k = 0; k < j; ++k) dj -= L[Packed<Q>::at(j, k)] * L[Packed<Q>::at(j, k)];
      const bool pos = dj > 1e-12f;
      ok = ok && pos;
      const float inv = pos ? rsqrtf(dj) : 1.0f;
      L[Packed<Q>::at(j, j)] = inv;
#pragma unroll
      for (int i = j + 1; i < Q; ++i) {
        float v = L[Packed<Q>::at(i, j)];
#pragma unroll
        for (int k = 0; k < j; ++k) v -= L[Packed<Q>::at(i, k)] * L[Packed<Q>::at(j, k)];
        L[Packed<Q>::at(i, j)] = v * inv;
      }
    }
    // Hager's 1-norm estimate of A~^-1 (A~ symmetric)
    float x[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) x[i] = 1.0f / Q;
    packed_solve<Q>(L, x);
    float est = 0.f;
#pragma unroll
    for (int i = 0; i < Q; ++i) est += fabsf(x[i]);
#pragma unroll
    for (int i = 0; i < Q; ++i) x[i] = x[i] >= 0.f ? 1.f : -1.f;
    packed_solve<Q>(L, x);
    int jmax = 0;
    float zmax = -1.f;
#pragma unroll
    for (int i = 0; i < Q; ++i)
      if (fabsf(x[i]) > zmax) {
        zmax = fabsf(x[i]);
        jmax = i;
      }
#pragma unroll
    for (int i = 0; i < Q; ++i) x[i] = i == jmax ? 1.f : 0.f;
    packed_solve<Q>(L, x);
    float est2 = 0.f;
#pragma unroll
    for (int i = 0; i < Q; ++i) est2 += fabsf(x[i]);
    const float cond = anorm * fmaxf(est, est2);
    if (valid && a.cond_out) a.cond_out[t] = cond;
    if (!(cond <= opt.cond_threshold)) ok = false;
    if (opt.force_fallback) ok = false;
    const double rho = fmin(0.5, 2.0 * Q * (double)cond * 5.960464477539063e-08);

    int sweeps_max = 0;
    bool conv_all = true;
    for (int f = 0; f < F; ++f) {
      const int kind = rk.kind[f];
      // y0 = D A~^-1 D lambda
#pragma unroll
      for (int i = 0; i < Q; ++i) x[i] = (float)scalar_lambda<DIM, ORDER>(kind, i + SKIP, ie) * dsc[i];
      packed_solve<Q>(L, x);
#pragma unroll
      for (int i = 0; i < Q; ++i) ybuf[i][lane] = (double)(x[i] * dsc[i]);
      bool conv = false;
      int sweeps = 0;
      for (int it = 0; it < opt.max_sweeps && ok && !conv; ++it) {
        // r_a = lambda_a - (1/a!) sum_b mu_(a+b) y_b / b!  (FP64), moment-major;
        // the empty asm keeps the moment loads inside the sweep (hoisting
        // all of them would hold NM doubles live across the loop)
        int zoff = 0;
        asm volatile("" : "+v"(zoff));
        double yf[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) yf[k] = ybuf[k][lane] * IF.v[k + SKIP];
        double acc[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) acc[i] = 0.0;
#pragma unroll
        for (int pp = 0; pp < MP.P; ++pp) {
          if (MP.a[pp] < SKIP || MP.b[pp] < SKIP) continue;
          const double mv = GMLS_MU(MP.m[pp], zoff);
          acc[MP.a[pp] - SKIP] += mv * yf[MP.b[pp] - SKIP];
        }
#pragma unroll
        for (int i = 0; i < Q; ++i)
          x[i] = (float)((scalar_lambda<DIM, ORDER>(kind, i + SKIP, ie) - IF.v[i + SKIP] * acc[i]) * (double)dsc[i]);
        packed_solve<Q>(L, x);
        double dmax = 0.0, ymax = 0.0;
        bool finite = true;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const double dy = (double)x[i] * (double)dsc[i];
          const double yn = ybuf[i][lane] + dy;
          ybuf[i][lane] = yn;
          finite = finite && isfinite(dy);
          dmax = fmax(dmax, fabs(dy));
          ymax = fmax(ymax, fabs(yn));
        }
        sweeps = it + 1;
        if (!finite) break;
        if (rho * dmax <= opt.refine_tol * ymax) conv = true;
      }
      conv_all = conv_all && conv;
      sweeps_max = sweeps > sweeps_max ? sweeps : sweeps_max;
      if (valid) {
#pragma unroll
        for (int i = 0; i < Q; ++i) yout[(loc * F + f) * Q + i] = ybuf[i][lane] * IF.v[i + SKIP];
      }
    }
    const bool good = valid && ok && conv_all;
    const bool not_conv = valid && ok && !conv_all;
    const bool fell = valid && !ok;
    if (valid) {
      a.status[t] = good ? GMLS_TARGET_OK : not_conv ? GMLS_TARGET_NOT_CONVERGED : GMLS_TARGET_FALLBACK;
      rec[sl - c0].ok = good ? 1 : 0;
    }
    if (not_conv || fell) fb_list[atomicAdd(&meta->fb_count, 1)] = t;
    // statistics, aggregated over the wavefront (one atomic per counter)
    const int sw = sweeps_max < 15 ? sweeps_max : 15;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const unsigned long long m = __ballot(good && sw == k);
      if (lane == 0 && m) atomicAdd(&stats->sweep_hist[k], (unsigned long long)__popcll(m));
    }
    const unsigned long long mnc = __ballot(not_conv), mfb = __ballot(fell);
    if (lane == 0 && mnc) atomicAdd(&stats->n_not_converged, (unsigned long long)__popcll(mnc));
    if (lane == 0 && mfb) atomicAdd(&stats->n_fallback, (unsigned long long)__popcll(mfb));
    double cd = valid && (double)cond >= 0.0 ? (double)cond : 0.0;  // NaN estimates are skipped
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cd = fmax(cd, __shfl_xor(cd, o));
    if (lane == 0 && cd > 0.0) atomicMax(&stats->cond_max_bits, (unsigned long long)__double_as_longlong(cd));
  }
#undef GMLS_MU
}

// ---------------------------------------------------------------------------
// C. weights
// ---------------------------------------------------------------------------
// The weights w_j p(s_j) . c_f of the group's rows, one functional row f after
// the other: the rows' scaled offsets and kernel weights stay in registers, the
// coefficients come one row ahead, and each functional row's weights are
// collected in LDS and leave as whole runs.  Without the stores the kernel ran
// 1M targets of 60 rows and three functional rows in 266 of 785 us: stores of
// 8-lane segments at unaligned row starts, not arithmetic, bounded it.  As runs
// of 64 consecutive doubles, not kept in the caches: 611 us; staggered, 500k
// targets, four rows 1140 -> 870; 2M targets on random rows, one row, 1730 ->
// 1620, there bound by the gathers (gather_rows).
//
// The coefficients of one functional row of the wavefront's TPW targets,
// fetched by all lanes together (CW per target, targets `stride` apart) and
// passed on through LDS.
template <int TPW, int CW>
struct CoefFetch {
  static constexpr int NL = (TPW * CW + 63) / 64;
  double pre[NL];
  __device__ __forceinline__ void fetch(const double *c, int64_t stride, int n_targets) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = lane_id() + 64 * u, tt = e / CW;
      pre[u] = e < TPW * CW && tt < n_targets ? c[tt * stride + (e - tt * CW)] : 0.0;
    }
  }
  __device__ __forceinline__ void put(double *lds) const {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = lane_id() + 64 * u;
      if (e < TPW * CW) lds[e] = pre[u];
    }
  }
};

// Runs of W doubles a row, the wavefront's targets' `live` rows, from LDS
// (target tt's at stage[tt * STR]) to out: one target after the other, 64
// consecutive doubles an instruction, past the caches (the weights do not fit
// them: 1 to 5 % of a call).
template <int G, int RPL, int W, int STR>
__device__ __forceinline__ void store_runs(const double *stage, double *out, int live, int lane) {
  constexpr int TPW = 64 / G;
#pragma unroll
  for (int tt = 0; tt < TPW; ++tt) {
    const int n = __builtin_amdgcn_readlane(live, tt * G) * W;
    const uint64_t o = (uint64_t)out;
    double *run = (double *)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(o >> 32), tt * G) << 32) |
                             (uint32_t)__builtin_amdgcn_readlane((int)o, tt * G));
#pragma unroll
    for (int m = 0; m < G * RPL * W; m += 64)
      if (m + lane < n) __builtin_nontemporal_store(stage[tt * STR + m + lane], run + m + lane);
  }
}

// SKIP = 1 (staggered): columns are monomials 1..Q-1, and the group also
// writes each row's target weight -sum_j alpha_j.
// Targets of at most DIRECT rows write from registers: their runs are no longer
// than the segments (300k 2-D targets of 12 rows, four functional rows: 60 us
// so, 91 through LDS; of 25 and 30 rows the same within 5 %).
template <int DIM, int ORDER, int G, int RPL, int SKIP = 0, bool LOOP = false>
__global__ __launch_bounds__(64) void k_pipe_weights(StencilArgs a, const PipeRec *rec, const BinMeta *meta, int bin,
                                                     int win_lo, int win_hi, const double *yin) {
  const SlotRange R = slot_range(meta, bin, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  constexpr int QF = num_mono(DIM, ORDER);
  constexpr int Q = QF - SKIP;
  constexpr int TPW = 64 / G;
  constexpr int STR = G * RPL + G;
  constexpr int DIRECT = 32;
  __shared__ __align__(16) double stage[TPW * STR];
  __shared__ __align__(16) double cfs[TPW * Q];
  __shared__ double rs[SKIP != 0 && LOOP ? 5 * 64 : 1];
  const int lane = lane_id();
  const int grp = lane / G, lg = lane % G;
  const int F = a.F;
  // the coefficients of the plain monomials (constrained stencils keep one more
  // solution per target)
  const int ys = (F + (a.normals ? 1 : 0)) * Q;
  for (int i0 = first + xcd_block() * TPW; i0 < last; i0 += gridDim.x * TPW) {
    const int i = i0 + grp;
    const bool valid = i < last;
    const int64_t loc = (valid ? i : first) - c0;
    const PipeRec rc = rec[loc];
    const bool good = valid && rc.ok;
    if (__ballot(good) == 0) continue;  // no target to form weights of
    const double *y0 = yin + (int64_t)(i0 - c0) * ys;
    CoefFetch<TPW, Q> cq;
    cq.fetch(y0, ys, last - i0);
    const int64_t base = rc.base;
    const int N = rc.n;
    const double ie = rc.ie;
    double xt[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) xt[d] = rc.x[d];
    double *wout = a.weights + (int64_t)F * base;
    const int cend = chunk_end<LOOP, G * RPL>(N);
    const int nmax = chunk_end<true, 1>(N);
    for (int q0 = 0; q0 < cend; q0 += G * RPL) {  // one pass unless LOOP (the long bin)
      const int nrem = N - q0;
      double s[RPL][DIM], w[RPL];
      {
        double xs[RPL][DIM];
        gather_rows<DIM, RPL, G, true>(a, base + (nrem > 0 ? q0 : 0), nrem > 0 ? nrem : N, lg, xs);
        rows_sw<DIM>(xs, xt, ie, a.p, [](int) { return true; }, s, w);
      }
      for (int f = 0; f < F; ++f) {
        cq.put(cfs);
        wave_lds_sync();
        double cf[QF];
        if constexpr (SKIP != 0) cf[0] = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) cf[q + SKIP] = cfs[grp * Q + q];
        if (f + 1 < F || (LOOP && q0 + G * RPL < cend)) cq.fetch(y0 + (f + 1 < F ? f + 1 : 0) * Q, ys, last - i0);
        double rsum = SKIP != 0 && LOOP && q0 > 0 ? rs[f * 64 + lane] : 0.0;
        double *run = wout + (int64_t)f * N + q0;
        if (!LOOP && G * RPL == 64 && nmax <= DIRECT) {
#pragma unroll
          for (int r = 0; r < (DIRECT + G - 1) / G; ++r) {
            const double v = w[r] * horner<DIM, ORDER>(cf, s[r]);
            if (good && lg + G * r < nrem) run[lg + G * r] = v;
            if constexpr (SKIP != 0) rsum += lg + G * r < nrem ? v : 0.0;
          }
          wave_lds_sync();  // cfs is rewritten for the next row
        } else {
#pragma unroll
          for (int r = 0; r < RPL; ++r) {
            const double v = w[r] * horner<DIM, ORDER>(cf, s[r]);
            stage[grp * STR + lg + G * r] = v;
            if constexpr (SKIP != 0) rsum += lg + G * r < nrem ? v : 0.0;
          }
          wave_lds_sync();
          store_runs<G, RPL, 1, STR>(stage, run, good ? nrem : 0, lane);
          wave_lds_sync();
        }
        if constexpr (SKIP != 0) {
          if (LOOP && q0 + G * RPL < cend) {
            rs[f * 64 + lane] = rsum;
            continue;
          }
          // the group's row sums, its G lanes in a fixed butterfly order
#pragma unroll
          for (int off = 1; off < G; off <<= 1) rsum += __shfl_xor(rsum, off, 64);
          if (good && lg == 0) a.hweights[(int64_t)rc.t * F + f] = -rsum;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Divergence-free basis (Section 2.2) on the pipeline, for scalar bases of
// at most 10 monomials.  The divergence-free span is the kernel of the
// divergence map D on the full vector polynomial space (coefficients c_(a,k)
// of p_a e_k): with the eps-scaled Taylor monomials, d/ds_k p_a = p_(a-e_k),
// so (D c)_b = sum_k c_(b+e_k, k) for every monomial b of degree < m.  The
// weighted least squares over that span is the vector fit with Gram
// I (x) G_s (G_s the scalar moment Gram, Section 2.1) under D c = 0; for a
// functional l its value is g^T (P^T W u) with
//     g = G^-1 (l - D^T t),   S t = D G^-1 l,   S = D G^-1 D^T
// (G = I (x) G_s), which takes only solves with the scalar Gram and a small
// Schur complement.  Solve kernel: one thread per target, G_s equilibrated
// and factored by Cholesky in FP64 (the moment Gram has at most 10 columns
// here), Hager's estimate of its condition number against the threshold;
// g for every (functional, component) goes to HBM, and the weights kernel
// forms alpha_(j,c) = w_j p(s_j) . g_c.  The divergence functional of a
// divergence-free fit is identically zero: its g is 0.
//
// The FP64 path runs the solve kernel twice (stencil_pipe64.hpp): PASS 0 as
// above, a pivot at or below kCholTol of its diagonal entry leaving the
// target to the QR kernel (fb_list, fb_count: its queues by bin); PASS 1 corrects g with the residual taken over the
// rows, sums [slot][F][DIM][QS] = P^T (W P g_k) on the plain monomials: per
// component c, rho_k = delta_(k,c) l - G_s g_k - D_k^T t, dv_k = G_s^-1 rho_k,
// S dt = D (dv + g), g_k += dv_k - G_s^-1 D_k^T dt.
// ---------------------------------------------------------------------------
constexpr double kCholTol = 1e-6;
// A small pivot shows a large condition number, a large condition number need
// not show in any pivot: what bounds it is the correction itself, whose size
// relative to the solution (both in the norm of the equilibrated system) is the
// first solve's error, some cond(M) 2^-54.  Above this bound (cond(M) of some
// 2e8, 1.5e4 for the weighted sample matrix) the target is left to QR.  By the
// pivots alone 1200 one-sided 2-D order-4 targets of 15 neighbours had errors
// up to 7.5e-7, QR's at most 1e-9.
constexpr double kCorrTol = 0x1p-27;

template <int DIM, int ORDER>
struct DivUp {
  static constexpr int QS = num_mono(DIM, ORDER);
  static constexpr int QM = ORDER >= 1 ? num_mono(DIM, ORDER - 1) : 1;
  int up[QM][3];  // index of the monomial b + e_k
  constexpr DivUp() : up{} {
    Mono<DIM, ORDER> M{};
    for (int b = 0; b < QM; ++b)
      for (int k = 0; k < 3; ++k) {
        up[b][k] = -1;
        if (k >= DIM) continue;
        int e[3] = {M.e[b][0], M.e[b][1], M.e[b][2]};
        e[k] += 1;
        for (int a = 0; a < QS; ++a)
          if (M.e[a][0] == e[0] && M.e[a][1] == e[1] && M.e[a][2] == e[2]) up[b][k] = a;
      }
  }
};

// x <- (L L^T)^-1 x for a packed lower-triangular FP64 L with 1/L_jj on the
// diagonal
template <int Q>
__device__ __forceinline__ void packed_solve64(const double *L, double *x) {
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    double v = x[i];
#pragma unroll
    for (int k = 0; k < i; ++k) v -= L[Packed<Q>::at(i, k)] * x[k];
    x[i] = v * L[Packed<Q>::at(i, i)];
  }
#pragma unroll
  for (int i = Q - 1; i >= 0; --i) {
    double v = x[i];
#pragma unroll
    for (int k = i + 1; k < Q; ++k) v -= L[Packed<Q>::at(k, i)] * x[k];
    x[i] = v * L[Packed<Q>::at(i, i)];
  }
}

// in-place packed Cholesky (diagonal keeps 1/L_jj); false on a pivot <= tol
// (REL: times its diagonal entry)
template <int Q, bool REL = false>
__device__ __forceinline__ bool packed_cholesky64(double *L, double tol) {
  bool ok = true;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    double dj = L[Packed<Q>::at(j, j)];
    const double lim = REL ? tol * dj : tol;
#pragma unroll
    for (int k = 0; k < j; ++k) dj -= L[Packed<Q>::at(j, k)] * L[Packed<Q>::at(j, k)];
    const bool pos = dj > lim;
    ok = ok && pos;
    const double inv = pos ? 1.0 / sqrt(dj) : 1.0;
    L[Packed<Q>::at(j, j)] = inv;
#pragma unroll
    for (int i = j + 1; i < Q; ++i) {
      double v = L[Packed<Q>::at(i, j)];
#pragma unroll
      for (int k = 0; k < j; ++k) v -= L[Packed<Q>::at(i, k)] * L[Packed<Q>::at(j, k)];
      L[Packed<Q>::at(i, j)] = v * inv;
    }
  }
  return ok;
}

// gout: g_i / i!, the coefficients of the plain monomials
template <int DIM, int ORDER, int PASS = -1>
__global__ __launch_bounds__(64) void k_pipe_solve_div(StencilArgs a, PipeRec *rec, int win_lo, int win_hi,
                                                       const double *mom, double *gout, const double *sums,
                                                       int *fb_list, int *fb_count, BinMeta *meta, Stats *stats,
                                                       Options opt) {
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int QM = DivUp<DIM, ORDER>::QM;
  constexpr int NP = QS * (QS + 1) / 2;
  constexpr InvFact64<DIM, ORDER> IF{};
  constexpr SumIndex<DIM, ORDER> SI{};
  constexpr DivUp<DIM, ORDER> DU{};
  constexpr int NM = num_mono(DIM, 2 * ORDER);
  __shared__ double mls[NM][64];  // thread-private columns: lane l uses [.][l]
  const int lane = lane_id();
  const RowKinds rk = row_kinds(DIM, 1, a.mask);
  const int F = a.F;
  const SlotRange R = slot_range(meta, 0, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  for (int slot = first + xcd_block() * 64 + lane; slot - lane < last; slot += gridDim.x * 64) {
    const bool valid = slot < last;
    const int sl = valid ? slot : first;
    const int t = rec[sl - c0].t;
    const double ie = rec[sl - c0].ie;
    const int64_t loc = sl - c0;
    if (valid) {
#pragma unroll
      for (int m = 0; m < NM; ++m) mls[m][lane] = mom[loc * NM + m];
    }
    // G_s_ab = mu_(a+b)/(a! b!); its equilibration sc G_s sc (sc_a =
    // 1/sqrt(G_s_aa)) is the moment matrix scaled by dsc_a = 1/sqrt(mu_2a)
    double dsc[QS], sc[QS];
#pragma unroll
    for (int i = 0; i < QS; ++i) {
      dsc[i] = 1.0 / sqrt(mls[SI.idx[i][i]][lane]);
      sc[i] = dsc[i] / IF.v[i];
    }
    double L[NP];
#pragma unroll
    for (int i = 0; i < QS; ++i)
#pragma unroll
      for (int k = 0; k <= i; ++k) L[Packed<QS>::at(i, k)] = mls[SI.idx[i][k]][lane] * dsc[i] * dsc[k];
    double anorm = 0.0;
#pragma unroll
    for (int k = 0; k < QS; ++k) {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < QS; ++i) sum += fabs(i >= k ? L[Packed<QS>::at(i, k)] : L[Packed<QS>::at(k, i)]);
      anorm = fmax(anorm, sum);
    }
    bool ok = valid && packed_cholesky64<QS>(L, PASS < 0 ? 1e-12 : kCholTol);
    if constexpr (PASS == 1) ok = valid && rec[sl - c0].ok;
    double x[QS], cond = 0.0;
    if constexpr (PASS < 0) {
    // Hager's 1-norm estimate of the inverse
#pragma unroll
    for (int i = 0; i < QS; ++i) x[i] = 1.0 / QS;
    packed_solve64<QS>(L, x);
    double est = 0.0;
#pragma unroll
    for (int i = 0; i < QS; ++i) est += fabs(x[i]);
#pragma unroll
    for (int i = 0; i < QS; ++i) x[i] = x[i] >= 0.0 ? 1.0 : -1.0;
    packed_solve64<QS>(L, x);
    int jmax = 0;
    double zmax = -1.0;
#pragma unroll
    for (int i = 0; i < QS; ++i)
      if (fabs(x[i]) > zmax) {
        zmax = fabs(x[i]);
        jmax = i;
      }
#pragma unroll
    for (int i = 0; i < QS; ++i) x[i] = i == jmax ? 1.0 : 0.0;
    packed_solve64<QS>(L, x);
    double est2 = 0.0;
#pragma unroll
    for (int i = 0; i < QS; ++i) est2 += fabs(x[i]);
    cond = anorm * fmax(est, est2);
    if (valid && a.cond_out) a.cond_out[t] = (float)cond;
    if (!(cond <= opt.cond_threshold)) ok = false;
    if (opt.force_fallback) ok = false;
    }
    // solves with the Gram: G_s^-1 v = sc . (L L^T)^-1 (sc . v)
    // S = D G^-1 D^T, column b2: component k contributes G_s^-1 e_(b2+e_k)
    // at rows b+e_k
    double S[QM * (QM + 1) / 2];
#pragma unroll
    for (int q = 0; q < QM * (QM + 1) / 2; ++q) S[q] = 0.0;
#pragma unroll
    for (int b2 = 0; b2 < QM; ++b2)
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
#pragma unroll
        for (int i = 0; i < QS; ++i) x[i] = i == DU.up[b2][k] ? sc[i] : 0.0;
        packed_solve64<QS>(L, x);
#pragma unroll
        for (int b = b2; b < QM; ++b) S[Packed<QM>::at(b, b2)] += x[DU.up[b][k]] * sc[DU.up[b][k]];
      }
    const bool s_ok = packed_cholesky64<QM, (PASS >= 0)>(S, PASS < 0 ? 1e-300 : kCholTol);
    if constexpr (PASS <= 0) ok = ok && s_ok;
    bool small = true;  // PASS 1: every correction is (kCorrTol)
    for (int f = 0; f < F; ++f) {
      const int kind = rk.kind[f], comp = rk.comp[f];
      double g[DIM][QS];
      if (kind == FK_DIV) {
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
          for (int i = 0; i < QS; ++i) g[k][i] = 0.0;
      } else {
        // v = G_s^-1 l (component comp), r_b = v_(b + e_comp), t = S^-1 r
        double lam[QS];
#pragma unroll
        for (int i = 0; i < QS; ++i) lam[i] = scalar_lambda<DIM, ORDER>(kind, i, ie);
#pragma unroll
        for (int i = 0; i < QS; ++i) x[i] = lam[i] * sc[i];
        packed_solve64<QS>(L, x);
        double ev = 0.0, ed = 0.0;  // PASS 1: sizes of v and of the correction, equilibrated
        if constexpr (PASS == 1) {
#pragma unroll
          for (int i = 0; i < QS; ++i) ev = fma(x[i], x[i], ev);
        }
        double tv[QM];
#pragma unroll
        for (int b = 0; b < QM; ++b) {
          tv[b] = 0.0;
#pragma unroll
          for (int k = 0; k < DIM; ++k)
            if (k == comp) tv[b] = x[DU.up[b][k]] * sc[DU.up[b][k]];
        }
        packed_solve64<QM>(S, tv);
        // g_k = G_s^-1 (delta_(k,comp) l - sum_b t_b e_(b+e_k)); PASS 1: dv_k
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
#pragma unroll
          for (int i = 0; i < QS; ++i) {
            double v = k == comp ? lam[i] : 0.0;
            if constexpr (PASS == 1) v -= sums[((loc * F + f) * DIM + k) * QS + i] * IF.v[i];
#pragma unroll
            for (int b = 0; b < QM; ++b)
              if (DU.up[b][k] == i) v -= tv[b];
            g[k][i] = v * sc[i];
          }
          packed_solve64<QS>(L, g[k]);
          if constexpr (PASS == 1) {
#pragma unroll
            for (int i = 0; i < QS; ++i) ed = fma(g[k][i], g[k][i], ed);
          }
#pragma unroll
          for (int i = 0; i < QS; ++i) g[k][i] *= sc[i];
        }
        if constexpr (PASS == 1) small = small && ed <= kCorrTol * kCorrTol * ev;
        if constexpr (PASS == 1) {
          // dv_k + g_k, then the constraint
#pragma unroll
          for (int k = 0; k < DIM; ++k)
#pragma unroll
            for (int i = 0; i < QS; ++i) g[k][i] += gout[((loc * F + f) * DIM + k) * QS + i] / IF.v[i];
#pragma unroll
          for (int b = 0; b < QM; ++b) {
            tv[b] = 0.0;
#pragma unroll
            for (int k = 0; k < DIM; ++k) tv[b] += g[k][DU.up[b][k]];
          }
          packed_solve64<QM>(S, tv);
#pragma unroll
          for (int k = 0; k < DIM; ++k) {
#pragma unroll
            for (int i = 0; i < QS; ++i) {
              double v = 0.0;
#pragma unroll
              for (int b = 0; b < QM; ++b)
                if (DU.up[b][k] == i) v = tv[b];
              x[i] = v * sc[i];
            }
            packed_solve64<QS>(L, x);
#pragma unroll
            for (int i = 0; i < QS; ++i) g[k][i] -= x[i] * sc[i];
          }
        }
      }
      if (PASS == 1 ? ok && kind != FK_DIV : valid) {
#pragma unroll
        for (int k = 0; k < DIM; ++k)
#pragma unroll
          for (int i = 0; i < QS; ++i) gout[((loc * F + f) * DIM + k) * QS + i] = g[k][i] * IF.v[i];
      }
    }
    if constexpr (PASS == 1) {
      const bool leave = ok && !small;
      if (leave) rec[sl - c0].ok = 0;
      leave_targets(leave, sl, t, meta, fb_list, fb_count);
      continue;
    }
    const bool good = valid && ok;
    const bool fell = valid && !ok;
    if (valid) {
      a.status[t] = good ? GMLS_TARGET_OK : GMLS_TARGET_FALLBACK;
      rec[sl - c0].ok = good ? 1 : 0;
    }
    if constexpr (PASS >= 0) {
      leave_targets(fell, sl, t, meta, fb_list, fb_count);
      continue;  // the mixed path's statistics follow
    }
    if (fell) fb_list[atomicAdd(fb_count, 1)] = t;
    const unsigned long long mg = __ballot(good), mfb = __ballot(fell);
    if (lane == 0 && mg) atomicAdd(&stats->sweep_hist[0], (unsigned long long)__popcll(mg));
    if (lane == 0 && mfb) atomicAdd(&stats->n_fallback, (unsigned long long)__popcll(mfb));
    double cd = valid && cond >= 0.0 ? cond : 0.0;  // NaN estimates are skipped
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cd = fmax(cd, __shfl_xor(cd, o));
    if (lane == 0 && cd > 0.0) atomicMax(&stats->cond_max_bits, (unsigned long long)__double_as_longlong(cd));
  }
}

// alpha_(j, f, c) = w_j p(s_j) . g_(f,c), one functional row f (its DIM
// components' coefficients in registers, Horner evaluation) per pass over
// the rows.  Bound by its stores: the weights of one functional row of a
// target are one run of N*DIM doubles, collected in LDS and stored 64
// consecutive doubles an instruction (1M targets of 60 rows, three functional
// rows, 4.3 GB: 1740 us with the runs cut at every G rows, 1390 whole).
template <int DIM, int ORDER, int G, int RPL, bool LOOP = false>
__global__ __launch_bounds__(64) void k_pipe_weights_div(StencilArgs a, const PipeRec *rec, const BinMeta *meta,
                                                         int bin, int win_lo, int win_hi, const double *gin) {
  const SlotRange R = slot_range(meta, bin, win_lo, win_hi);
  const int first = R.first, last = R.last, c0 = R.c0;
  constexpr int QS = num_mono(DIM, ORDER);
  constexpr int TPW = 64 / G;
  constexpr int CW = DIM * QS;  // coefficients of one target and row
  constexpr int STR = G * (RPL + 1) * DIM;
  __shared__ __align__(16) double stage[TPW * STR];
  __shared__ __align__(16) double cfs[TPW * CW];
  const int lane = lane_id();
  const int grp = lane / G, lg = lane % G;
  const int F = a.F, FC = F * DIM;
  for (int i0 = first + xcd_block() * TPW; i0 < last; i0 += gridDim.x * TPW) {
    // row 0's coefficients with the neighbour gathers, the others' one row ahead
    const double *g0 = gin + (int64_t)(i0 - c0) * FC * QS;
    CoefFetch<TPW, CW> cq;
    cq.fetch(g0, FC * QS, last - i0);
    const int i = i0 + grp;
    const bool valid = i < last;
    const int64_t loc = (valid ? i : first) - c0;
    const PipeRec rc = rec[loc];
    const bool good = valid && rc.ok;
    if (__ballot(good) == 0) continue;  // no target to form weights of
    const int64_t base = rc.base;
    const int N = rc.n;
    double xt[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) xt[d] = rc.x[d];
    double *wout = a.weights + (int64_t)FC * base;
    // one pass unless LOOP (the long bin): then every chunk of G * RPL rows
    // is gathered again for each functional row
    const int cend = chunk_end<LOOP, G * RPL>(N);
    double xs[RPL][DIM];
    gather_rows<DIM, RPL, G, true>(a, base, N, lg, xs);
    double s[RPL][DIM], w[RPL];
    rows_sw<DIM>(xs, xt, rc.ie, a.p, [](int) { return true; }, s, w);
    for (int f = 0; f < F; ++f) {
      cq.put(cfs);
      wave_lds_sync();
      double cf[DIM][QS];
#pragma unroll
      for (int c = 0; c < DIM; ++c)
#pragma unroll
        for (int q = 0; q < QS; ++q) cf[c][q] = cfs[grp * CW + c * QS + q];
      if (f + 1 < F) cq.fetch(g0 + (f + 1) * CW, FC * QS, last - i0);
      for (int q0 = 0; q0 < cend; q0 += G * RPL) {
        const int nrem = N - q0;
        if (LOOP && (q0 > 0 || f > 0)) {  // the rows of this chunk (chunk 0 of row 0 is loaded above)
          gather_rows<DIM, RPL, G, true>(a, base + (nrem > 0 ? q0 : 0), nrem > 0 ? nrem : N, lg, xs);
          rows_sw<DIM>(xs, xt, rc.ie, a.p, [](int) { return true; }, s, w);
        }
#pragma unroll
        for (int r = 0; r < RPL; ++r)
#pragma unroll
          for (int c = 0; c < DIM; ++c)
            stage[grp * STR + (lg + G * r) * DIM + c] = w[r] * horner<DIM, ORDER>(cf[c], s[r]);
        wave_lds_sync();
        store_runs<G, RPL, DIM, STR>(stage, wout + ((int64_t)f * N + q0) * DIM, good ? nrem : 0, lane);
        wave_lds_sync();
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host: the pipeline over the bins of one call, in chunks of list slots
// ---------------------------------------------------------------------------
template <int DIM, int ORDER>
constexpr bool has_pipe() {
  return num_mono(DIM, ORDER) <= 20;
}

// the divergence-free pipeline factors the scalar Gram in FP64 registers
template <int DIM, int ORDER>
constexpr bool has_pipe_div() {
  return ORDER >= 1 && num_mono(DIM, ORDER) <= 10;
}

template <int DIM, int ORDER, int G, int RPL, int SKIP, int BASIS = 0, bool LOOP = false>
static void pipe_bin_launch(bool weights, const StencilArgs &a, const PipeRec *rec, const BinMeta *meta, int bin,
                            int win_lo, int win_hi, int n_max, double *buf, int cus, hipStream_t s) {
  constexpr int TPW = 64 / G;
  int nb = (n_max + TPW - 1) / TPW;
  if (nb > cus * 32) nb = cus * 32;
  nb = xcd_grid(nb);
  if (!weights) {
    k_pipe_moments<DIM, ORDER, G, RPL, LOOP><<<nb, 64, 0, s>>>(a, rec, meta, bin, win_lo, win_hi, buf);
    return;
  }
  if constexpr (BASIS == 1) {
    k_pipe_weights_div<DIM, ORDER, G, RPL, LOOP><<<nb, 64, 0, s>>>(a, rec, meta, bin, win_lo, win_hi, buf);
    return;
  }
  k_pipe_weights<DIM, ORDER, G, RPL, SKIP, LOOP><<<nb, 64, 0, s>>>(a, rec, meta, bin, win_lo, win_hi, buf);
}

// the bin's launch in row shape `cand` (kPipeShapes; -1: the default)
template <int DIM, int ORDER, int SKIP, int BASIS, int BIN>
static void pipe_bin_shape(int cand, bool weights, const StencilArgs &a, const PipeRec *rec, const BinMeta *meta,
                           int win_lo, int win_hi, int n_max, double *buf, int cus, hipStream_t s) {
  constexpr PipeShape S0 = kPipeShapes[BIN][0], S1 = kPipeShapes[BIN][1], S2 = kPipeShapes[BIN][2];
  constexpr bool L = BIN == kLongBin;
  if (cand < 0) cand = pipe_default_shape(DIM, ORDER, BASIS == 1, SKIP != 0, weights, BIN);
  if (cand == 1)
    pipe_bin_launch<DIM, ORDER, S1.g, S1.rpl, SKIP, BASIS, L>(weights, a, rec, meta, BIN, win_lo, win_hi, n_max,
                                                              buf, cus, s);
  else if (cand == 2)
    pipe_bin_launch<DIM, ORDER, S2.g, S2.rpl, SKIP, BASIS, L>(weights, a, rec, meta, BIN, win_lo, win_hi, n_max,
                                                              buf, cus, s);
  else
    pipe_bin_launch<DIM, ORDER, S0.g, S0.rpl, SKIP, BASIS, L>(weights, a, rec, meta, BIN, win_lo, win_hi, n_max,
                                                              buf, cus, s);
}

// The pipeline over list slots [count[0], n) (bins 1..4, contiguous, in bin
// order).  With a host copy of the bin table (hm) it runs in chunks of
// `chunk` slots and skips empty bins; without one (hm == nullptr: nothing
// may wait for the device) it covers every slot in one window, all bounds
// read from the device table, grids sized for n_max slots.
// Lanes x rows per lane of the moment and weight kernels: the candidate
// opt.pipe_shape[kernel][bin] of kPipeShapes (-1: pipe_default_shape).  With a
// timer, events bracket every per-bin launch.
template <int DIM, int ORDER, int SKIP = 0, int BASIS = 0>
hipError_t launch_pipe(const StencilArgs &a, const int *list, const BinMeta *hm, BinMeta *meta, int *fb,
                       Stats *stats, const Options &opt, double *mom, double *y, PipeRec *rec, int64_t chunk,
                       int n_max, int cus, PipeTimer *timer, hipStream_t s) {
  int begin = 0, end = 1;
  if (hm) {
    begin = hm->offset[1];
    end = hm->offset[kNumBins - 1] + hm->count[kNumBins - 1];
  } else {
    chunk = 1;
  }
  for (int64_t c0 = begin; c0 < end; c0 += chunk) {
    const int win_lo = hm ? (int)c0 : -1;
    const int win_hi = hm ? (int)(c0 + chunk < end ? c0 + chunk : end) : INT_MAX;
    const int n_win = hm ? win_hi - win_lo : n_max;
    if (!opt.reuse_moments) {
      int nbp = (n_win + 255) / 256;
      if (nbp > cus * 8) nbp = cus * 8;
      if (nbp < 1) nbp = 1;
      k_pipe_prep<DIM><<<nbp, 256, 0, s>>>(a, list, meta, win_lo, win_hi, rec);
    }
    // a second stencil set on the same neighbour lists (one window) takes
    // the records and moments of the first
    for (int pass = opt.reuse_moments ? 1 : 0; pass < 2; ++pass) {
      if (pass == 1) {
        int nb = (n_win + 63) / 64;
        if (nb > cus * 16) nb = cus * 16;
        nb = xcd_grid(nb);
        if constexpr (BASIS == 1)
          k_pipe_solve_div<DIM, ORDER><<<nb, 64, 0, s>>>(a, rec, win_lo, win_hi, mom, y, nullptr, fb, &meta->fb_count, meta,
                                                         stats, opt);
        else
          k_pipe_solve<DIM, ORDER, SKIP><<<nb, 64, 0, s>>>(a, rec, win_lo, win_hi, mom, y, fb, meta, stats, opt);
      }
      const bool wts = pass == 1;
      for (int b = 1; b < kNumBins; ++b) {
        int nbin = n_max;
        if (hm) {
          const int lo = hm->offset[b] > win_lo ? hm->offset[b] : win_lo;
          const int hi = hm->offset[b] + hm->count[b] < win_hi ? hm->offset[b] + hm->count[b] : win_hi;
          if (lo >= hi) continue;
          nbin = hi - lo;
        }
        double *buf = wts ? y : mom;
        const int cand = opt.pipe_shape[pass][b];
        if (timer) {
          hipError_t e = hipEventRecord(timer->ev[pass][b][0], s);
          if (e != hipSuccess) return e;
        }
        if (b == 1)
          pipe_bin_shape<DIM, ORDER, SKIP, BASIS, 1>(cand, wts, a, rec, meta, win_lo, win_hi, nbin, buf, cus, s);
        else if (b == 2)
          pipe_bin_shape<DIM, ORDER, SKIP, BASIS, 2>(cand, wts, a, rec, meta, win_lo, win_hi, nbin, buf, cus, s);
        else if (b == 3)
          pipe_bin_shape<DIM, ORDER, SKIP, BASIS, 3>(cand, wts, a, rec, meta, win_lo, win_hi, nbin, buf, cus, s);
        else if (b == 4)
          pipe_bin_shape<DIM, ORDER, SKIP, BASIS, 4>(cand, wts, a, rec, meta, win_lo, win_hi, nbin, buf, cus, s);
        else
          pipe_bin_shape<DIM, ORDER, SKIP, BASIS, kLongBin>(cand, wts, a, rec, meta, win_lo, win_hi, nbin, buf, cus,
                                                            s);
        if (timer) {
          hipError_t e = hipEventRecord(timer->ev[pass][b][1], s);
          if (e != hipSuccess) return e;
          timer->used[pass][b] = 1;
        }
      }
    }
  }
  return hipGetLastError();
}

}  // namespace gmls
