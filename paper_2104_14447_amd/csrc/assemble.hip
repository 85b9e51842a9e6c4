// assemble.hip -- the global Stokes operator of Section 3.2 from stencils,
// and a CSR matrix-vector product.
//
// Unknowns and rows: velocity v_(J,c) at J*d + c, pressure phi_J at d*n + J,
// the zero-mean multiplier lambda at d*n + n.  Rows (nu the viscosity):
//   velocity, interior I, component c:
//       -nu sum_j sum_c' L^v_(I,c,j,c') v_(J,c') + sum_j G_(I,c,j) phi_J
//   velocity, boundary I:  v_(I,c)                         (Dirichlet)
//   pressure, interior I:  sum_j L^s_(I,j) phi_J + tau_I phi_I + lambda
//   pressure, boundary I:  nu beta_I sum_j sum_c' (n_I . L^v_(I,.,j,c')) v_(J,c')
//                          + sum_j L^n_(I,j) phi_J + lambda
//   multiplier:            sum_J phi_J
// with L^v the divergence-free vector Laplacian, G the scalar gradient, L^s
// the staggered Laplacian with target weight tau, L^n the Neumann-constrained
// Laplacian with h-weight beta (Section 2.3: Laplacian phi(x_I) =
// sum_j L^n phi_j + beta_I h_I, h_I = n.f + nu n.Laplacian v(x_I)).
// A velocity row holds the K block then the G block, a pressure row the N
// block (boundary), then the L block, then the multiplier; entries follow the
// neighbour order.  One wavefront writes all rows of a particle.
#include <atomic>
#include <mutex>

#include "common.hpp"
#include "gmls_internal.hpp"

namespace gmls {

// entries of the rows of particle I: d velocity rows then its pressure row
__device__ __forceinline__ void stokes_row_lengths(const StokesArgs &s, int64_t I, int N, bool self, int64_t *vlen,
                                                   int64_t *plen) {
  const int d = s.dim;
  if (s.boundary[I]) {
    *vlen = 1;
    *plen = (int64_t)d * N + N + 1;
  } else {
    *vlen = (int64_t)d * N + N;
    *plen = N + (self ? 0 : 1) + 1;
  }
}

// whether particle I is among its own neighbours (wave-uniform)
__device__ __forceinline__ bool self_listed(const StokesArgs &s, int64_t I, int64_t rb, int N) {
  bool hit = false;
  for (int q = lane_id(); q < N; q += 64) hit = hit || s.col[rb + q] == (int32_t)I;
  return __ballot(hit) != 0;
}

__global__ __launch_bounds__(256) void k_stokes_count(StokesArgs s, int64_t *rlen) {
  const int lane = lane_id();
  const int64_t wpb = blockDim.x >> 6;
  const int d = s.dim;
  for (int64_t I = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); I < s.n; I += (int64_t)gridDim.x * wpb) {
    const int64_t rb = s.row_ptr[I];
    const int N = (int)(s.row_ptr[I + 1] - rb);
    const bool self = self_listed(s, I, rb, N);
    int64_t vlen, plen;
    stokes_row_lengths(s, I, N, self, &vlen, &plen);
    if (lane < d) rlen[I * d + lane] = vlen;
    if (lane == 0) rlen[(int64_t)d * s.n + I] = plen;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) rlen[(int64_t)d * s.n + s.n] = s.n;
}

__global__ __launch_bounds__(256) void k_stokes_fill(StokesArgs s, const int64_t *arp, int32_t *acol, double *aval,
                                                     const int *flags) {
  if (*flags) return;  // over capacity: nothing is written
  const int lane = lane_id();
  const int64_t wpb = blockDim.x >> 6;
  const int d = s.dim;
  const int64_t n = s.n;
  const int32_t pcol0 = (int32_t)(d * n);  // column of phi_0
  for (int64_t I = (int64_t)blockIdx.x * wpb + (threadIdx.x >> 6); I < n; I += (int64_t)gridDim.x * wpb) {
    const int64_t rb = s.row_ptr[I];
    const int N = (int)(s.row_ptr[I + 1] - rb);
    const int32_t *nb = s.col + rb;
    const bool bnd = s.boundary[I] != 0;
    // velocity rows
    for (int c = 0; c < d; ++c) {
      const int64_t o = arp[I * d + c];
      if (bnd) {
        if (lane == 0) {
          acol[o] = (int32_t)(I * d + c);
          aval[o] = 1.0;
        }
        continue;
      }
      // K block: -nu L^v, weights (c*N + j)*d + c' of the particle's d*d*rb block
      const double *lv = s.vlap + (int64_t)d * d * rb + (int64_t)c * N * d;
      for (int q = lane; q < N * d; q += 64) {
        const int j = q / d, cp = q - j * d;
        acol[o + q] = nb[j] * d + cp;
        aval[o + q] = -s.nu * lv[q];
      }
      // G block
      const double *gr = s.grad + (int64_t)d * rb + (int64_t)c * N;
      for (int j = lane; j < N; j += 64) {
        acol[o + (int64_t)N * d + j] = pcol0 + nb[j];
        aval[o + (int64_t)N * d + j] = gr[j];
      }
    }
    // pressure row
    int64_t o = arp[d * n + I];
    if (bnd) {
      // N block: nu beta_I n_I . L^v
      const double beta = s.nlap_h[I];
      double nv[3] = {0.0, 0.0, 0.0};
      for (int c = 0; c < d; ++c) nv[c] = s.normals[I * d + c];
      const double *lv = s.vlap + (int64_t)d * d * rb;
      for (int q = lane; q < N * d; q += 64) {
        const int j = q / d, cp = q - j * d;
        double acc = 0.0;
        for (int c = 0; c < d; ++c) acc += nv[c] * lv[((int64_t)c * N + j) * d + cp];
        acol[o + q] = nb[j] * d + cp;
        aval[o + q] = s.nu * beta * acc;
      }
      o += (int64_t)N * d;
      for (int j = lane; j < N; j += 64) {
        acol[o + j] = pcol0 + nb[j];
        aval[o + j] = s.nlap[rb + j];
      }
      o += N;
    } else {
      const bool self = self_listed(s, I, rb, N);
      const double tau = s.plap_t[I];
      for (int j = lane; j < N; j += 64) {
        acol[o + j] = pcol0 + nb[j];
        aval[o + j] = s.plap[rb + j] + (nb[j] == (int32_t)I ? tau : 0.0);
      }
      o += N;
      if (!self) {
        if (lane == 0) {
          acol[o] = pcol0 + (int32_t)I;
          aval[o] = tau;
        }
        ++o;
      }
    }
    if (lane == 0) {
      acol[o] = (int32_t)(d * n + n);
      aval[o] = 1.0;
    }
  }
  // the multiplier row
  const int64_t o = arp[d * n + n];
  for (int64_t J = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; J < n; J += (int64_t)gridDim.x * blockDim.x) {
    acol[o + J] = pcol0 + (int32_t)J;
    aval[o + J] = 1.0;
  }
}

__global__ void k_stokes_check(const int64_t *arp, int64_t rows, int64_t capacity, int *flags) {
  if (threadIdx.x == 0) *flags = arp[rows] > capacity ? 1 : 0;
}

hipError_t launch_stokes_assembly(const StokesArgs &s, int64_t *rlen, int64_t *arp, int64_t *tmp, int32_t *acol,
                                  double *aval, int64_t capacity, int *flags, int cus, hipStream_t st) {
  const int64_t rows = (int64_t)s.dim * s.n + s.n + 1;
  const unsigned nb = (unsigned)xcd_grid(cus * 16);
  k_stokes_count<<<nb, 256, 0, st>>>(s, rlen);
  hipError_t e = scan_i64_exclusive(rlen, arp, rows, tmp, st);
  if (e != hipSuccess) return e;
  k_stokes_check<<<1, 64, 0, st>>>(arp, rows, capacity, flags);
  k_stokes_fill<<<nb, 256, 0, st>>>(s, arp, acol, aval, flags);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// y = A x for a CSR matrix: one wavefront per row (lane q takes entries q,
// q + 64, ... of four running sums, then a butterfly sum); rows longer than
// kLongRow are cut into segments, a block each, whose sums are added in
// segment order.  Every order depends on the matrix alone, so y is
// reproducible.
//
// Bound by the latency of a row's chain (row bounds, column indices, x
// gathers, sum) against the bandwidth of the 12 bytes per entry.  Four
// independent entries per lane are requested together (2 to 4 within 1 %, 5
// and 6 were 3 and 6 % slower, 8 14 %: fewer wavefronts' requests per CU);
// the last group takes no more than it needs, entries that are not there
// re-reading the row's last one.  A block per four rows, handed out by the
// dispatcher, where a grid of 64 blocks per CU walked the rows (996 -> 850
// us), in contiguous ranges per XCD (-> 826 us); loads that bypass the caches
// gain 2 % more there and lose a quarter on a matrix that the last-level
// cache holds (55 -> 72 us at 20M entries).  Long rows are cut over up
// to 64 blocks each (one block took 240 us for the multiplier row).  The 281M-entry Stokes
// operator of 287k particles: 1172 -> 826 us, 2.9 -> 4.1 TB/s.
// ---------------------------------------------------------------------------
constexpr int kLongRow = 8192;

// acc[u % 4] += val[q + S u] * x[col[q + S u]], u < K, for the entries below e
// (CLAMP: some may not be there; those re-read the row's last and are dropped)
template <int S, int K, bool CLAMP>
__device__ __forceinline__ void spmv_entries(const int32_t *col, const double *val, const double *x, int64_t q,
                                             int64_t e, double (&acc)[4]) {
  int c[K];
  double v[K], xv[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int64_t k = !CLAMP || q + S * u < e ? q + S * u : e - 1;
    c[u] = col[k];
    v[u] = val[k];
  }
#pragma unroll
  for (int u = 0; u < K; ++u) xv[u] = x[c[u]];
#pragma unroll
  for (int u = 0; u < K; ++u) acc[u % 4] = !CLAMP || q + S * u < e ? fma(v[u], xv[u], acc[u % 4]) : acc[u % 4];
}

// the last `left` entries (0 < left <= K S), as many per lane as that takes
template <int S, int K>
__device__ __forceinline__ void spmv_last(const int32_t *col, const double *val, const double *x, int64_t q, int64_t e,
                                          int64_t left, double (&acc)[4]) {
  if constexpr (K > 1) {
    if (left <= (K - 1) * S) return spmv_last<S, K - 1>(col, val, x, q, e, left, acc);
  }
  spmv_entries<S, K, true>(col, val, x, q, e, acc);
}

// entries b .. e of a row over S lanes (l: this one)
template <int S>
__device__ __forceinline__ double spmv_row(const int32_t *col, const double *val, const double *x, int64_t b,
                                           int64_t e, int l) {
  constexpr int K = 4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (; e - b > K * S; b += K * S) spmv_entries<S, K, false>(col, val, x, b + l, e, acc);
  if (e > b) spmv_last<S, K>(col, val, x, b + l, e, e - b, acc);
  return wave_sum_uniform((acc[0] + acc[1]) + (acc[2] + acc[3]));
}

__global__ __launch_bounds__(256) void k_spmv(int64_t rows, const int64_t *rp, const int32_t *col, const double *val,
                                              const double *x, double *y, int *long_rows, int *n_long) {
  const int lane = lane_id();
  const int64_t wpb = blockDim.x >> 6;
  for (int64_t r = (int64_t)xcd_block() * wpb + (threadIdx.x >> 6); r < rows; r += (int64_t)gridDim.x * wpb) {
    const int64_t b = uniform_i64(rp[r]), e = uniform_i64(rp[r + 1]);
    if (e - b > kLongRow) {
      if (lane == 0) long_rows[atomicAdd(n_long, 1)] = (int)r;
      continue;
    }
    const double sum = spmv_row<64>(col, val, x, b, e, lane);
    if (lane == 0) y[r] = sum;
  }
}

// Rows handed on by k_spmv: up to kSpmvSplit of them in segments, as many (a
// power of two, at most 64) as make no more than the grid's blocks, the block
// that finishes a row's last segment adding the sums in segment order; more
// rows than that, a block per row.  done: a finished-segment counter per cut
// row, cleared with n_long.  63 rows of 20000 entries beside 200k short ones:
// 193 us a product in 64 segments each (4032 of 312 entries, 16 to a block),
// 93 in 4; 64 of 400000 680 uncut, 262 in 4.
__global__ __launch_bounds__(256) void k_spmv_long(const int64_t *rp, const int32_t *col, const double *val,
                                                   const double *x, double *y, const int *long_rows,
                                                   const int *n_long, int *done, double *partial) {
  __shared__ double part[4];
  __shared__ int last;
  const int n = *n_long;
  int S = n <= kSpmvSplit ? 64 : 1;
  while (n * S > kSpmvSegments && S > 1) S >>= 1;
  for (int64_t w = blockIdx.x; w < (int64_t)n * S; w += gridDim.x) {
    const int k = (int)(w / S);
    const int64_t r = long_rows[k], g = w % S;
    const int64_t rb = rp[r], len = rp[r + 1] - rb;
    const int64_t b = rb + len * g / S, e = rb + len * (g + 1) / S;
    const double sum = spmv_row<256>(col, val, x, b, e, threadIdx.x);
    if (lane_id() == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
      const double t = (part[0] + part[1]) + (part[2] + part[3]);
      last = 0;
      if (S == 1) {
        y[r] = t;
      } else {
        __hip_atomic_store(partial + w, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = __hip_atomic_fetch_add(done + k, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == S - 1;
      }
    }
    __syncthreads();
    if (last && threadIdx.x < 64) {
      const double seg = (int)threadIdx.x < S ? __hip_atomic_load(partial + (int64_t)k * S + threadIdx.x, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT)
                                              : 0.0;
      const double t = wave_sum_uniform(seg);
      if (threadIdx.x == 0) y[r] = t;
    }
    __syncthreads();
  }
}

hipError_t launch_spmv(int64_t rows, const int64_t *rp, const int32_t *col, const double *val, const double *x,
                       double *y, int *long_rows, int *n_long, double *partial, int cus, hipStream_t s) {
  static_assert(1 + kSpmvSplit <= kSpmvListWord && 2 * kSpmvSplit <= kSpmvSegments, "scratch layout");
  hipError_t e = fill_zero(n_long, sizeof(int) * (1 + kSpmvSplit), s);
  if (e != hipSuccess) return e;
  int64_t g = (rows + 3) / 4;
  if (g > (1 << 22)) g = 1 << 22;
  g = xcd_grid((int)g);
  k_spmv<<<(unsigned)g, 256, 0, s>>>(rows, rp, col, val, x, y, long_rows, n_long);
  k_spmv_long<<<kSpmvSegments, 256, 0, s>>>(rp, col, val, x, y, long_rows, n_long, n_long + 1, partial);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of the allocation-free product (gmls_spmv_noalloc), for every row of
// a matrix of up to kNoAllocSpmvRows rows being long.  Each device holds its
// own copy until the process ends; host code reaches it only
// through the address hipGetSymbolAddress returns on that device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) int scratch[kSpmvScratchWords(kNoAllocSpmvRows)];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mutex;
static std::atomic<int *> g_scratch_ptr[kMaxScratchDevices];

hipError_t spmv_scratch_setup(int device) {
  if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
  if (g_scratch_ptr[device].load(std::memory_order_acquire)) return hipSuccess;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[device].load(std::memory_order_relaxed)) return hipSuccess;
  int *p = nullptr;  // the caller has made `device` current
  hipError_t e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  g_scratch_ptr[device].store(p, std::memory_order_release);
  return hipSuccess;
}

int *spmv_scratch(int device) {
  if (device < 0 || device >= kMaxScratchDevices) return nullptr;
  return g_scratch_ptr[device].load(std::memory_order_acquire);
}

}  // namespace gmls
