// CPR-AMG on the device (paper sec. 2.3.1: the two-stage constrained-
// pressure-residual preconditioner with an AMG for the pressure system).
//
// Setup, once per Jacobian: quasi-IMPES weights w_i with D_i^T w_i = e_p
// (D_i the diagonal block of row i), the pressure matrix (A_p)_ij =
// w_i^T A_ij e_p on the block pattern, the Galerkin coarse matrices of the
// aggregation hierarchy (each coarse entry the sum of its gather list of
// fine entries, in a fixed order) and the inverse of the coarsest matrix
// (in-place Gauss-Jordan with partial pivoting, at most 64 unknowns).
// Application, z = CPR(r): b_0 = w^T r; one V(1,1) cycle (damped Jacobi,
// omega = 2/3, before and after the coarse correction; the coarsest level
// by its inverse) gives x_p; x1 = e_p x_p; z = x1 + M_ILU^{-1} (r - A x1)
// with the (block-)ILU(0) factors of A.
//
// Down at level l one kernel forms the right-hand side b_l (w^T r, or the
// in-order sum of an unknown's children's residuals) and the pre-smoothed
// iterate x_l = omega D^{-1} b_l, and a second one the residual b_l - A_l x_l; up
// at level l one kernel writes the post-smoothed x + omega D^{-1} (b - A x) with
// x = x_l + P x_{l+1}.  The levels at the bottom, of at most 2048 unknowns, are
// one dense operator, formed at setup by running the cycle on each unit vector:
// their kernels are chains of dependent loads and the gaps between launches,
// the product is one pass over memory.
//
// Every kernel is a gather (no atomics), so results are the same on every
// run.  Contraction is off in this file: the 3x3 weight solves and the
// sparse products round like plain multiply-then-add code.
#include <algorithm>
#include <cstring>

#include "cpr_dev.h"

#pragma clang fp contract(off)

namespace opm {

int ilu_apply(const opm_problem* pb, void* ilu, int precision, const double* r, double* x,
              hipStream_t s, const int32_t* skip);

namespace {

constexpr double kOmega = 2.0 / 3.0;

inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }

// Gaussian elimination with partial pivoting on a 3x3 system (A row-major,
// b overwritten by the solution); false on a zero pivot.
__device__ bool solve3(double* A, double* b) {
  for (int col = 0; col < 3; ++col) {
    int piv = col;
    for (int r = col + 1; r < 3; ++r)
      if (fabs(A[r * 3 + col]) > fabs(A[piv * 3 + col])) piv = r;
    if (A[piv * 3 + col] == 0.0) return false;
    if (piv != col) {
      for (int c = 0; c < 3; ++c) {
        const double t = A[col * 3 + c];
        A[col * 3 + c] = A[piv * 3 + c];
        A[piv * 3 + c] = t;
      }
      const double t = b[col];
      b[col] = b[piv];
      b[piv] = t;
    }
    for (int r = col + 1; r < 3; ++r) {
      const double f = A[r * 3 + col] / A[col * 3 + col];
      if (f == 0.0) continue;
      for (int c = col; c < 3; ++c) A[r * 3 + c] -= f * A[col * 3 + c];
      b[r] -= f * b[col];
    }
  }
  for (int r = 2; r >= 0; --r) {
    double s = b[r];
    for (int c = r + 1; c < 3; ++c) s -= A[r * 3 + c] * b[c];
    b[r] = s / A[r * 3 + r];
  }
  return true;
}

// Rows of a level are spread over a wavefront seven lanes each (nine rows
// per wavefront, one entry per lane: the 7-point stencil and its Galerkin
// coarse stencils have at most seven entries per row; longer rows are
// strided over the same lanes).  Consecutive lanes read consecutive entries.
constexpr int kRowLanes = 7;
constexpr int kWaveRows = kWave / kRowLanes;   // 9

struct RowLane {
  int row, k;
  bool live;
};

__device__ __forceinline__ RowLane row_lane(int n) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  RowLane r;
  r.row = wave * kWaveRows + lane / kRowLanes;
  r.k = lane % kRowLanes;
  r.live = lane < kWaveRows * kRowLanes && r.row < n;
  return r;
}

inline int row_blocks(int n, int sets = 1) {
  const int waves = (n + kWaveRows * sets - 1) / (kWaveRows * sets);
  return std::max(1, (waves + kBlock / kWave - 1) / (kBlock / kWave));
}

// U sets of nine rows of a wavefront.  Each lane's entry of a row is found by
// two dependent loads (row bounds; column and value) and its vector values by
// up to three more; with every load of U sets issued together a wavefront waits
// once per step of that chain for U times the rows.  Lanes without an entry
// load the row's last one (no branch between the loads).
template <int U>
struct RowSets {
  int row[U], q[U], q1[U], col[U];
  double a[U];
  bool live[U], in[U];
  int k, base;
  __device__ __forceinline__ RowSets() {
    const int lane = threadIdx.x & (kWave - 1);
    k = lane % kRowLanes;
    base = lane - k;
  }
  // set u: rows from (first + u) * kWaveRows
  __device__ __forceinline__ void bounds(int n, const int32_t* row_ptr, int first) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = (first + u) * kWaveRows + lane / kRowLanes;
      live[u] = lane < kWaveRows * kRowLanes && r < n;
      row[u] = min(r, n - 1);
      q[u] = row_ptr[row[u]] + k;
      q1[u] = row_ptr[row[u] + 1];
    }
  }
  __device__ __forceinline__ int entry(int u) const { return min(q[u], max(q1[u] - 1, 0)); }
  __device__ __forceinline__ void columns(const int32_t* c) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      in[u] = live[u] && q[u] < q1[u];
      col[u] = c[entry(u)];
    }
  }
  __device__ __forceinline__ void values(const double* v) {
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = v[entry(u)];
  }
  // the lane of the row's diagonal entry (-1: not among its first seven)
  __device__ __forceinline__ int diag_lane(int u) const {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(in[u] && col[u] == row[u]);
    const unsigned own = (unsigned)(m >> base) & ((1u << kRowLanes) - 1u);
    return own != 0 ? base + __builtin_ctz(own) : -1;
  }
};

// first set of the wavefront
template <int U>
__device__ __forceinline__ int wave_sets() {
  return (int)(blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * U;
}

// Rows from which a wavefront takes four sets: with fewer rows the chip is
// not full (8192 resident wavefronts of 36 rows).
constexpr int kManyRows = 200000;

// Sum of p over the seven lanes of a row, in entry order (every lane of the
// wavefront takes part; the row's first lane holds the result).
__device__ __forceinline__ double row_sum(double p) {
  const int lane = threadIdx.x & (kWave - 1);
  const int base = lane - lane % kRowLanes;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kRowLanes; ++k) s += __shfl(p, base + k, kWave);
  return s;
}

// Weights and the level-0 diagonal (one lane per cell).
__global__ __launch_bounds__(kBlock) void k_cpr_weights(int n, const int32_t* diag_pos,
                                                         const double* J, double* w, double* d0,
                                                         int32_t* flags) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const double* D = J + 9 * (size_t)diag_pos[i];
  double T[9] = {D[0], D[3], D[6], D[1], D[4], D[7], D[2], D[5], D[8]};   // D^T
  double e[3] = {1.0, 0.0, 0.0};
  if (!solve3(T, e)) flags[0] = OPM_ESINGULAR;
  w[3 * i] = e[0];
  w[3 * i + 1] = e[1];
  w[3 * i + 2] = e[2];
  double v = 0.0;
  v += e[0] * D[0];
  v += e[1] * D[3];
  v += e[2] * D[6];
  d0[i] = v;
}

// The level-0 pressure matrix w_i^T A_ij e_p and the compact pressure
// column of J (one lane per block).
__global__ __launch_bounds__(kBlock) void k_cpr_pressure(int n, const int32_t* row_ptr,
                                                          const double* J, const double* w,
                                                          double* a0, double* jp) {
  const RowLane rl = row_lane(n);
  if (!rl.live) return;
  const int i = rl.row;
  const double w0 = w[3 * i], w1 = w[3 * i + 1], w2 = w[3 * i + 2];
  for (int q = row_ptr[i] + rl.k; q < row_ptr[i + 1]; q += kRowLanes) {
    const double* B = J + 9 * (size_t)q;
    const double c0 = B[0], c1 = B[3], c2 = B[6];
    double v = 0.0;
    v += w0 * c0;
    v += w1 * c1;
    v += w2 * c2;
    a0[q] = v;
    jp[3 * (size_t)q] = c0;
    jp[3 * (size_t)q + 1] = c1;
    jp[3 * (size_t)q + 2] = c2;
  }
}

// One coarse level's matrix by its gather lists (one lane per entry).
__global__ __launch_bounds__(kBlock) void k_cpr_galerkin(int nnz, const int32_t* gptr,
                                                          const int32_t* gmap, const double* fine,
                                                          double* coarse) {
  const int e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= nnz) return;
  double s = 0.0;
  for (int t = gptr[e]; t < gptr[e + 1]; ++t) s += fine[gmap[t]];
  coarse[e] = s;
}

__global__ __launch_bounds__(kBlock) void k_cpr_diag(int n, const int32_t* dpos, const double* a,
                                                      double* d) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) d[i] = a[dpos[i]];
}

// Inverse of the coarsest matrix (n <= 64) by in-place Gauss-Jordan
// elimination with partial pivoting in LDS (one workgroup): at step k the
// row with the largest |a_rk| (r >= k, lowest index on ties) is swapped
// into place, row k is divided by the pivot and eliminated from every other
// row, and column k becomes the corresponding column of the inverse; the
// row swaps are undone as column swaps at the end, last first.
constexpr int kGjThreads = 256;
__global__ __launch_bounds__(kGjThreads) void k_cpr_inverse(int n, const int32_t* row_ptr,
                                                             const int32_t* col, const double* a,
                                                             double* inv, int32_t* flags) {
  // rows padded to an odd stride: a column walk across lanes spreads over
  // the LDS banks
  __shared__ double A[OPM_AMG_COARSE * (OPM_AMG_COARSE + 1)];
  __shared__ int perm[OPM_AMG_COARSE];
  __shared__ int sel, bad;
  const int t = threadIdx.x, ld = n | 1;
  for (int k = t; k < n * ld; k += kGjThreads) A[k] = 0.0;
  if (t == 0) bad = 0;
  __syncthreads();
  for (int i = t; i < n; i += kGjThreads)
    for (int q = row_ptr[i]; q < row_ptr[i + 1]; ++q) A[i * ld + col[q]] = a[q];
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    if (t < kWave) {   // the first wave picks the pivot row
      double v = (t >= k && t < n) ? fabs(A[t * ld + k]) : -1.0;
      int idx = t;
      for (int off = kWave / 2; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(v, off, kWave);
        const int oi = __shfl_xor(idx, off, kWave);
        if (ov > v || (ov == v && oi < idx)) {
          v = ov;
          idx = oi;
        }
      }
      if (t == 0) {
        sel = idx;
        perm[k] = idx;
        if (!(A[idx * ld + k] != 0.0)) bad = 1;
      }
    }
    __syncthreads();
    if (bad) break;   // uniform across the workgroup
    const int p = sel;
    if (p != k)
      for (int j = t; j < n; j += kGjThreads) {
        const double v = A[k * ld + j];
        A[k * ld + j] = A[p * ld + j];
        A[p * ld + j] = v;
      }
    __syncthreads();
    const double pk = 1.0 / A[k * ld + k];
    for (int j = t; j < n; j += kGjThreads)
      if (j != k) A[k * ld + j] *= pk;
    __syncthreads();
    for (int e = t; e < n * n; e += kGjThreads) {
      const int i = e / n, j = e - (e / n) * n;
      if (i != k && j != k) A[i * ld + j] -= A[i * ld + k] * A[k * ld + j];
    }
    __syncthreads();
    for (int i = t; i < n; i += kGjThreads) A[i * ld + k] = i == k ? pk : -A[i * ld + k] * pk;
    __syncthreads();
  }
  if (bad) {
    if (t == 0) flags[0] = OPM_ESINGULAR;
    return;
  }
  for (int k = n - 1; k >= 0; --k) {
    const int p = perm[k];
    if (p != k)
      for (int i = t; i < n; i += kGjThreads) {
        const double v = A[i * ld + k];
        A[i * ld + k] = A[i * ld + p];
        A[i * ld + p] = v;
      }
    __syncthreads();
  }
  for (int e = t; e < n * n; e += kGjThreads) inv[e] = A[(e / n) * ld + e % n];
}

// Where a level's right-hand side comes from.
enum BSrc { kFromR = 0, kGiven = 1, kChildren = 2 };

struct BArgs {
  const double* w;           // kFromR: weights and residual
  const double* r;
  const double* b0;          // kGiven
  const int32_t* child_ptr;  // kChildren: the finer level's aggregates and residuals
  const int32_t* child;
  const double* res;
};

// The in-order sum of a coarse unknown's children, eight loads at a time (an
// aggregate of 2 x 2 x 2 cells has at most eight).
template <typename Res>
__device__ __forceinline__ double child_sum(const int32_t* child, int t0, int t1, Res res) {
  constexpr int kKids = 8;
  double v = 0.0;
  for (int t = t0; t < t1; t += kKids) {
    int c[kKids];
    double x[kKids];
#pragma unroll
    for (int e = 0; e < kKids; ++e) c[e] = child[min(t + e, t1 - 1)];
#pragma unroll
    for (int e = 0; e < kKids; ++e) x[e] = res(c[e]);
#pragma unroll
    for (int e = 0; e < kKids; ++e)
      if (t + e < t1) v += x[e];
  }
  return v;
}

template <int SRC>
__device__ __forceinline__ double bval(const BArgs& s, int i) {
  if (SRC == kFromR) {
    double v = s.w[3 * i] * s.r[3 * i];
    v += s.w[3 * i + 1] * s.r[3 * i + 1];
    v += s.w[3 * i + 2] * s.r[3 * i + 2];
    return v;
  } else if (SRC == kGiven) {
    return s.b0[i];
  } else {
    return child_sum(s.child, s.child_ptr[i], s.child_ptr[i + 1],
                     [&](int c) { return s.res[c]; });
  }
}

// Down at one level: b and x = omega D^{-1} b.
template <int SRC>
__global__ __launch_bounds__(kBlock) void k_cpr_rhs(int n, BArgs src, const double* d, double* b,
                                                     double* x, const int32_t* skip) {
  const int off = skip ? *skip : 0;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const double di = d[i];
  if (SRC == kChildren && off != 0) return;
  const double bi = bval<SRC>(src, i);
  if (off != 0) return;
  b[i] = bi;
  x[i] = kOmega * bi / di;
}

// Down at one level: the residual b - A x.  Each lane forms x of its neighbour
// from b once and not seven times: with the right-hand side in the same kernel
// (neighbours' weights, residuals and divisions by each lane that needs them)
// 30.2 us at 500,000 cells, as two kernels 6.2 + 13.5 us (36 and 56 MB).
template <int U>
__global__ __launch_bounds__(kBlock) void k_cpr_res(int n, const int32_t* row_ptr,
                                                     const int32_t* col, const double* a,
                                                     const double* b, const double* x,
                                                     double* res, const int32_t* skip) {
  const int off = skip ? *skip : 0;
  RowSets<U> s;
  s.bounds(n, row_ptr, wave_sets<U>());
  if (off != 0) return;
  s.columns(col);
  s.values(a);
  double bi[U], xj[U];
#pragma unroll
  for (int u = 0; u < U; ++u) bi[u] = b[s.row[u]];
#pragma unroll
  for (int u = 0; u < U; ++u) xj[u] = x[s.col[u]];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    double p = s.in[u] ? 0.0 + s.a[u] * xj[u] : 0.0;
    if (s.live[u])
      for (int q = s.q[u] + kRowLanes; q < s.q1[u]; q += kRowLanes) p += a[q] * x[col[q]];
    const double sum = row_sum(p);
    if (s.live[u] && s.k == 0) res[s.row[u]] = bi[u] - sum;
  }
}

// A hierarchy of one level: b from its source, x = A^{-1} b (one workgroup, a
// lane per row).
template <int SRC>
__global__ __launch_bounds__(OPM_AMG_COARSE) void k_cpr_coarse(int n, const double* inv,
                                                                BArgs src, double* x,
                                                                const int32_t* skip) {
  __shared__ double sb[OPM_AMG_COARSE];
  if (skip && *skip != 0) return;
  const int i = threadIdx.x;
  if (i < n) sb[i] = bval<SRC>(src, i);
  __syncthreads();
  if (i >= n) return;
  double s = 0.0;
  for (int c = 0; c < n; ++c) s += inv[i * n + c] * sb[c];
  x[i] = s;
}

// Up at one level: y = x + omega D^{-1} (b - A x) with the corrected
// x = x_l + x_c[agg].  500,000 cells: 18.4 us, 61 MB.
template <int U>
__global__ __launch_bounds__(kBlock) void k_cpr_up(int n, const int32_t* row_ptr,
                                                    const int32_t* col, const double* a,
                                                    const double* d, const double* b,
                                                    const double* x, const int32_t* agg,
                                                    const double* xc, double* y,
                                                    const int32_t* skip) {
  const int off = skip ? *skip : 0;
  RowSets<U> s;
  s.bounds(n, row_ptr, wave_sets<U>());
  if (off != 0) return;
  s.columns(col);
  s.values(a);
  double bi[U], di[U], xj[U];
  int g[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bi[u] = b[s.row[u]];
    di[u] = d[s.row[u]];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    g[u] = agg[s.col[u]];
    xj[u] = x[s.col[u]];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) xj[u] += xc[g[u]];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    double p = s.in[u] ? 0.0 + s.a[u] * xj[u] : 0.0;
    if (s.live[u])
      for (int q = s.q[u] + kRowLanes; q < s.q1[u]; q += kRowLanes)
        p += a[q] * (x[col[q]] + xc[agg[col[q]]]);
    const double sum = row_sum(p);
    const int own = s.diag_lane(u);
    double xi = __shfl(xj[u], max(own, 0), kWave);
    if (s.live[u] && s.k == 0) {
      const int i = s.row[u];
      if (own < 0) xi = x[i] + xc[agg[i]];
      y[i] = xi + kOmega * (bi[u] - sum) / di[u];
    }
  }
}

// The bottom levels: from the first of at most kTailRows unknowns.  Their part
// of the cycle is linear in the right-hand side of the first of them; column c
// of its matrix is the cycle of unit vector c, by one workgroup with the levels'
// vectors in LDS.
constexpr int kTailRows = 2048, kTailThreads = 1024;
constexpr size_t kTailLds = 64 * 1024;   // (what a kernel may use without asking for more)
struct TailLevel {
  const int32_t *row_ptr, *col, *child_ptr, *child, *agg;
  const double *a, *d;
  int n, at;   // LDS: b, x and the residual (on the way up: y), n values each from `at`
};
struct Tail {
  TailLevel l[OPM_AMG_MAX_LEVELS];
  int levels;
  const double* inv;   // of the last level
  double* m;           // [n][n] of the first level
};

__global__ __launch_bounds__(kTailThreads) void k_cpr_tail(Tail t) {
  extern __shared__ __attribute__((aligned(16))) double tail_lds[];
  typedef __attribute__((address_space(3))) double lds_double;
  lds_double* lds = (lds_double*)tail_lds;
  constexpr int kSets = 3, kWaves = kTailThreads / kWave;
  const int wave = threadIdx.x / kWave;
  for (int l = 0; l < t.levels; ++l) {
    const TailLevel& v = t.l[l];
    lds_double *b = lds + v.at, *x = b + v.n, *res = x + v.n;
    const lds_double* up = l > 0 ? lds + t.l[l - 1].at + 2 * t.l[l - 1].n : lds;
    const bool last = l + 1 == t.levels;
    for (int i = threadIdx.x; i < v.n; i += kTailThreads) {
      const double di = v.d[i];
      double bi = i == (int)blockIdx.x ? 1.0 : 0.0;
      if (l > 0)
        bi = child_sum(v.child, v.child_ptr[i], v.child_ptr[i + 1],
                       [&](int c) { return (double)up[c]; });
      b[i] = bi;
      if (!last) x[i] = kOmega * bi / di;
    }
    __syncthreads();
    if (last) break;
    for (int g = wave * kSets; g * kWaveRows < v.n; g += kWaves * kSets) {
      RowSets<kSets> s;
      s.bounds(v.n, v.row_ptr, g);
      s.columns(v.col);
      s.values(v.a);
#pragma unroll
      for (int u = 0; u < kSets; ++u) {
        double p = s.in[u] ? 0.0 + s.a[u] * x[s.col[u]] : 0.0;
        if (s.live[u])
          for (int q = s.q[u] + kRowLanes; q < s.q1[u]; q += kRowLanes)
            p += v.a[q] * x[v.col[q]];
        const double sum = row_sum(p);
        if (s.live[u] && s.k == 0) res[s.row[u]] = b[s.row[u]] - sum;
      }
    }
    __syncthreads();
  }
  {   // the coarsest level by its inverse, a thread per row
    const TailLevel& v = t.l[t.levels - 1];
    const lds_double* b = lds + v.at;
    lds_double* y = lds + v.at + 2 * v.n;
    if ((int)threadIdx.x < v.n) {
      double s = 0.0;
      for (int c = 0; c < v.n; ++c) s += t.inv[(size_t)threadIdx.x * v.n + c] * b[c];
      y[threadIdx.x] = s;
    }
    __syncthreads();
  }
  for (int l = t.levels - 2; l >= 0; --l) {
    const TailLevel& v = t.l[l];
    lds_double *b = lds + v.at, *x = b + v.n, *y = x + v.n;
    const lds_double* xc = lds + t.l[l + 1].at + 2 * t.l[l + 1].n;
    // the corrected x first: every lane's neighbours read it
    for (int i = threadIdx.x; i < v.n; i += kTailThreads) x[i] += xc[v.agg[i]];
    __syncthreads();
    for (int g = wave * kSets; g * kWaveRows < v.n; g += kWaves * kSets) {
      RowSets<kSets> s;
      s.bounds(v.n, v.row_ptr, g);
      s.columns(v.col);
      s.values(v.a);
      double di[kSets];
#pragma unroll
      for (int u = 0; u < kSets; ++u) di[u] = v.d[s.row[u]];
#pragma unroll
      for (int u = 0; u < kSets; ++u) {
        double p = s.in[u] ? 0.0 + s.a[u] * x[s.col[u]] : 0.0;
        if (s.live[u])
          for (int q = s.q[u] + kRowLanes; q < s.q1[u]; q += kRowLanes)
            p += v.a[q] * x[v.col[q]];
        const double sum = row_sum(p);
        if (s.live[u] && s.k == 0) {
          const double yi = x[s.row[u]] + kOmega * (b[s.row[u]] - sum) / di[u];
          y[s.row[u]] = yi;
        }
      }
    }
    __syncthreads();
  }
  const TailLevel& v = t.l[0];
  for (int i = threadIdx.x; i < v.n; i += kTailThreads)
    t.m[(size_t)i * v.n + blockIdx.x] = lds[v.at + 2 * v.n + i];
}

// y = M b of the bottom levels, b the sums of the children's residuals: a
// wavefront per row, its matrix entries asked for ahead of the right-hand side,
// which every workgroup forms for itself.  1183 unknowns (11 MB): 9.0 us; the
// three levels behind it took 26 us by one workgroup that went through them,
// and five launches of 4 to 6 us as kernels of their own.
constexpr int kDenseThreads = 512, kDenseLoads = 16;
__global__ __launch_bounds__(kDenseThreads) void k_cpr_dense(int n, const double* m, BArgs src,
                                                              double* y, const int32_t* skip) {
  __shared__ double b[kTailRows];
  const int off = skip ? *skip : 0;
  const int lane = threadIdx.x & (kWave - 1);
  const int i = blockIdx.x * (kDenseThreads / kWave) + threadIdx.x / kWave;
  const double* row = m + (size_t)min(i, n - 1) * n;
  if (off != 0) return;
  double v[kDenseLoads];
#pragma unroll
  for (int e = 0; e < kDenseLoads; ++e) v[e] = row[min(lane + e * kWave, n - 1)];
  for (int j = threadIdx.x; j < n; j += kDenseThreads) b[j] = bval<kChildren>(src, j);
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < kDenseLoads; ++e)
    if (lane + e * kWave < n) s += v[e] * b[lane + e * kWave];
  for (int j = lane + kDenseLoads * kWave; j < n; j += kWave) s += row[j] * b[j];
#pragma unroll
  for (int w = kWave / 2; w >= 1; w /= 2) s += __shfl_xor(s, w, kWave);
  if (lane == 0 && i < n) y[i] = s;
}

// Second-stage residual r2 = r - A x1 with x1 = (x_p, 0, 0) per cell, from
// the compact pressure column of J: seven lanes per row (one entry each,
// its three values in one 24-byte run), summed in entry order.
template <int U>
__global__ __launch_bounds__(kBlock) void k_cpr_r2(int n, const int32_t* row_ptr,
                                                    const int32_t* col, const double* jp,
                                                    const double* r, const double* xp,
                                                    double* r2, const int32_t* skip) {
  const int off = skip ? *skip : 0;
  RowSets<U> s;
  s.bounds(n, row_ptr, wave_sets<U>());
  if (off != 0) return;
  s.columns(col);
  double B[U][3], xj[U], ri[U];
  const int c = min(s.k, 2);   // lane c < 3 of a row writes its component c
#pragma unroll
  for (int u = 0; u < U; ++u) {
#pragma unroll
    for (int e = 0; e < 3; ++e) B[u][e] = jp[3 * (size_t)s.entry(u) + e];
    ri[u] = r[3 * (size_t)s.row[u] + c];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) xj[u] = xp[s.col[u]];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    double p[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) p[e] = s.in[u] ? 0.0 + B[u][e] * xj[u] : 0.0;
    if (s.live[u])
      for (int q = s.q[u] + kRowLanes; q < s.q1[u]; q += kRowLanes)
#pragma unroll
        for (int e = 0; e < 3; ++e) p[e] += jp[3 * (size_t)q + e] * xp[col[q]];
    const double t0 = row_sum(p[0]), t1 = row_sum(p[1]), t2 = row_sum(p[2]);
    if (s.live[u] && s.k < 3) r2[3 * (size_t)s.row[u] + c] = ri[u] - (c == 0 ? t0 : c == 1 ? t1 : t2);
  }
}

// z += x1.
__global__ __launch_bounds__(kBlock) void k_cpr_add(int n, const double* xp, double* z,
                                                     const int32_t* skip) {
  if (skip && *skip != 0) return;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) z[3 * i] += xp[i];
}

const int32_t* level_rows(const opm_problem* pb, int l) {
  return l == 0 ? pb->row_ptr : pb->amg->row_ptr[l];
}
const int32_t* level_cols(const opm_problem* pb, int l) {
  return l == 0 ? pb->col_idx : pb->amg->col[l];
}

}  // namespace

// First of the bottom levels (never level 0; n_levels: there is none, the
// hierarchy is one level) and the LDS of their cycle.  With 2048 unknowns the
// product reads 34 MB, about 7 us; a level of its own takes four launches, not
// under 14 us.
struct Bottom {
  int first;
  size_t lds;
};
static Bottom bottom_of(const opm_amg* g) {
  Bottom b{g->n_levels, 0};
  while (b.first > 1 && g->n[b.first - 1] <= kTailRows &&
         b.lds + 24 * (size_t)g->n[b.first - 1] <= kTailLds)
    b.lds += 24 * (size_t)g->n[--b.first];
  return b;
}

size_t cpr_bytes(const opm_problem* pb) {
  const opm_amg* g = pb->amg;
  if (!g) return 0;
  const int L = g->n_levels, nc = g->n[L - 1];
  size_t s = 2 * al256(8 * 3 * (size_t)pb->n_cells) + al256(8 * 3 * (size_t)pb->nnzb) +
             al256(8 * (size_t)nc * nc);
  for (int l = 0; l < L; ++l) s += al256(8 * (size_t)g->nnz[l]) + 5 * al256(8 * (size_t)g->n[l]);
  const int lt = bottom_of(g).first;
  if (lt < L) s += al256(8 * (size_t)g->n[lt] * g->n[lt]);
  return s;
}

CprWork cpr_carve(const opm_problem* pb, void* p) {
  const opm_amg* g = pb->amg;
  CprWork w;
  std::memset(&w, 0, sizeof w);
  char* c = (char*)p;
  auto take = [&](size_t bytes) {
    char* r = c;
    c += al256(bytes);
    return (double*)r;
  };
  const int L = g->n_levels, nc = g->n[L - 1];
  w.w = take(8 * 3 * (size_t)pb->n_cells);
  w.jp = take(8 * 3 * (size_t)pb->nnzb);
  for (int l = 0; l < L; ++l) {
    w.a[l] = take(8 * (size_t)g->nnz[l]);
    w.d[l] = take(8 * (size_t)g->n[l]);
    w.b[l] = take(8 * (size_t)g->n[l]);
    w.x[l] = take(8 * (size_t)g->n[l]);
    w.res[l] = take(8 * (size_t)g->n[l]);
    w.y[l] = take(8 * (size_t)g->n[l]);
  }
  w.inv = take(8 * (size_t)nc * nc);
  const int lt = bottom_of(g).first;
  w.tail = lt < L ? take(8 * (size_t)g->n[lt] * g->n[lt]) : nullptr;
  w.r2 = take(8 * 3 * (size_t)pb->n_cells);
  return w;
}

int cpr_setup(const opm_problem* pb, const double* J, const CprWork& w, int32_t* flags,
              hipStream_t s) {
  const opm_amg* g = pb->amg;
  const int n = pb->n_cells, L = g->n_levels;
  hipLaunchKernelGGL(k_cpr_weights, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, n,
                     pb->diag_pos, J, w.w, w.d[0], flags);
  hipLaunchKernelGGL(k_cpr_pressure, dim3(row_blocks(n)), dim3(kBlock), 0, s, n, pb->row_ptr, J,
                     w.w, w.a[0], w.jp);
  for (int l = 1; l < L; ++l) {
    hipLaunchKernelGGL(k_cpr_galerkin, dim3(blocks_for(g->nnz[l], kBlock)), dim3(kBlock), 0, s,
                       g->nnz[l], g->gmap_ptr[l], g->gmap[l], w.a[l - 1], w.a[l]);
    hipLaunchKernelGGL(k_cpr_diag, dim3(blocks_for(g->n[l], kBlock)), dim3(kBlock), 0, s,
                       g->n[l], g->dpos[l], w.a[l], w.d[l]);
  }
  hipLaunchKernelGGL(k_cpr_inverse, dim3(1), dim3(kGjThreads), 0, s, g->n[L - 1],
                     level_rows(pb, L - 1), level_cols(pb, L - 1), w.a[L - 1], w.inv, flags);
  const Bottom bt = bottom_of(g);
  if (bt.first < L) {
    Tail t{};
    t.levels = L - bt.first;
    t.inv = w.inv;
    t.m = w.tail;
    int at = 0;
    for (int l = bt.first; l < L; ++l) {
      t.l[l - bt.first] = TailLevel{level_rows(pb, l), level_cols(pb, l), g->child_ptr[l - 1],
                                    g->child[l - 1], g->agg[l], w.a[l], w.d[l], g->n[l], at};
      at += 3 * g->n[l];
    }
    hipLaunchKernelGGL(k_cpr_tail, dim3(g->n[bt.first]), dim3(kTailThreads), bt.lds, s, t);
  }
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

int cpr_vcycle(const opm_problem* pb, const CprWork& w, const double* r, const double* b0,
               hipStream_t s, const int32_t* skip) {
  const opm_amg* g = pb->amg;
  const int L = g->n_levels;
  auto src_of = [&](int l) {
    BArgs a{};
    if (l == 0) {
      a.w = w.w;
      a.r = r;
      a.b0 = b0;
    } else {
      a.child_ptr = g->child_ptr[l - 1];
      a.child = g->child[l - 1];
      a.res = w.res[l - 1];
    }
    return a;
  };
  const int lt = bottom_of(g).first;
  const int own = std::min(lt, L - 1);   // levels with kernels of their own
  for (int l = 0; l < own; ++l) {
    const int n = g->n[l];
    const BArgs src = src_of(l);
#define OPM_CPR_RHS(SRC)                                                                      \
  hipLaunchKernelGGL(k_cpr_rhs<SRC>, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, n, src, \
                     w.d[l], w.b[l], w.x[l], skip)
#define OPM_CPR_RES(U)                                                                        \
  hipLaunchKernelGGL(k_cpr_res<U>, dim3(row_blocks(n, U)), dim3(kBlock), 0, s, n,             \
                     level_rows(pb, l), level_cols(pb, l), w.a[l], w.b[l], w.x[l], w.res[l],  \
                     skip)
    if (l > 0)
      OPM_CPR_RHS(kChildren);
    else if (r)
      OPM_CPR_RHS(kFromR);
    else
      OPM_CPR_RHS(kGiven);
    if (n >= kManyRows)
      OPM_CPR_RES(4);
    else
      OPM_CPR_RES(1);
#undef OPM_CPR_RHS
#undef OPM_CPR_RES
  }
  if (L == 1) {
    const BArgs src = src_of(0);
    if (r)
      hipLaunchKernelGGL(k_cpr_coarse<kFromR>, dim3(1), dim3(OPM_AMG_COARSE), 0, s, g->n[0],
                         w.inv, src, w.y[0], skip);
    else
      hipLaunchKernelGGL(k_cpr_coarse<kGiven>, dim3(1), dim3(OPM_AMG_COARSE), 0, s, g->n[0],
                         w.inv, src, w.y[0], skip);
  } else {
    const int n = g->n[lt];
    hipLaunchKernelGGL(k_cpr_dense, dim3(blocks_for(n, kDenseThreads / kWave)),
                       dim3(kDenseThreads), 0, s, n, w.tail, src_of(lt), w.y[lt], skip);
  }
  for (int l = own - 1; l >= 0; --l) {
    const int n = g->n[l];
#define OPM_CPR_UP(U)                                                                         \
  hipLaunchKernelGGL(k_cpr_up<U>, dim3(row_blocks(n, U)), dim3(kBlock), 0, s, n,              \
                     level_rows(pb, l), level_cols(pb, l), w.a[l], w.d[l], w.b[l], w.x[l],    \
                     g->agg[l], w.y[l + 1], w.y[l], skip)
    if (n >= kManyRows)
      OPM_CPR_UP(4);
    else
      OPM_CPR_UP(1);
#undef OPM_CPR_UP
  }
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

int cpr_apply(const opm_problem* pb, const double* J, void* ilu, int precision, const CprWork& w,
              const double* r, double* z, hipStream_t s, const int32_t* skip) {
  (void)J;
  const int n = pb->n_cells;
  OPM_TRY(cpr_vcycle(pb, w, r, nullptr, s, skip));
  if (n >= kManyRows)
    hipLaunchKernelGGL(k_cpr_r2<4>, dim3(row_blocks(n, 4)), dim3(kBlock), 0, s, n, pb->row_ptr,
                       pb->col_idx, w.jp, r, w.y[0], w.r2, skip);
  else
    hipLaunchKernelGGL(k_cpr_r2<1>, dim3(row_blocks(n)), dim3(kBlock), 0, s, n, pb->row_ptr,
                       pb->col_idx, w.jp, r, w.y[0], w.r2, skip);
  OPM_TRY_HIP(hipGetLastError());
  OPM_TRY(ilu_apply(pb, ilu, precision, w.r2, z, s, skip));
  hipLaunchKernelGGL(k_cpr_add, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, n, w.y[0], z,
                     skip);
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

}  // namespace opm
