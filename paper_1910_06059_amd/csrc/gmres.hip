// Restarted GMRes, right preconditioned (paper sec. 2.3.1: the alternative
// Krylov method to the default BiCGStab), on the block-CSR SpMV and the
// ILU(0) / block-ILU0 solves of the other files.
//
// x0 = 0; each cycle starts from the residual r = b - A x, builds an
// orthonormal basis v_0 .. v_k of the Krylov space of A M^{-1} (at most
// `restart` vectors), reduces the Hessenberg least-squares problem with
// Givens rotations (|g_{j+1}| is the residual norm of the iterate), and ends
// with x += M^{-1} V y, R y = g.  Stop on |g_{j+1}| <= rtol ||b||, at the
// iteration cap, or on an exact breakdown h_{j+1,j} = 0.
//
// The preconditioned vectors z_j = M^{-1} v_j of the cycle are kept and the
// update is formed as Z y (the flexible form): for a linear M the same
// iterate as M^{-1} (V y), one preconditioner solve per cycle fewer, and with
// FP32 factors, whose solve is linear only up to FP32 rounding, an iterate
// whose residual is the one the rotations minimised.
//
// Orthogonalisation is classical Gram-Schmidt applied twice (CGS2): the
// j + 1 projections of a pass are one fused reduction, where modified
// Gram-Schmidt would need j + 1 dependent ones; the second pass restores the
// orthogonality modified Gram-Schmidt reaches.  Per inner iteration six
// launches: the preconditioner solve, the SpMV, the first projections, the
// first update + second projections, the second update + norm, and the
// rotations + the next basis vector.
//
// All scalars stay on the device.  A reducing kernel writes one partial per
// workgroup (at most kGmGrid of them); the kernel that consumes the sum adds
// the partials in its prologue, in the same fixed order in every workgroup,
// so all workgroups hold the same bits and take the same decisions, and
// every run gives the same result.  A state word (running / cycle end /
// done), read once per workgroup, lets the kernels of iterations that are no
// longer needed return at once; the host enqueues a cycle's iterations in
// chunks and reads the state between chunks.
#include <algorithm>

#include "cpr_dev.h"
#include "solver_dev.h"

namespace opm {

int ilu_apply(const opm_problem* pb, void* ilu, int precision, const double* r, double* x,
              hipStream_t s, const int32_t* skip);

namespace {

constexpr int kMaxRestart = 32;   // basis vectors per cycle
constexpr int kGmGrid = 256;      // largest grid of the reducing kernels (partials per sum)
constexpr int kGmBlock = 512;     // threads of the vector kernels (8 wavefronts)

enum GmState : int32_t { kGmRunning = 0, kGmCycleEnd = 1, kGmDone = 2 };

struct GmScalars {
  double H[(kMaxRestart + 1) * kMaxRestart];   // H[i * kMaxRestart + j], rotated
  double cs[kMaxRestart], sn[kMaxRestart];
  double gr[kMaxRestart];           // rotated right-hand side of the least-squares problem
  double gres[kMaxRestart + 1];     // gres[j]: residual estimate after j iterations of the cycle
  double h1[kMaxRestart + 1], h2[kMaxRestart + 1];   // projections of the two passes
  // the part read by the host between chunks starts here
  double bnorm, tol, relres, scale;
  int32_t state;       // GmState
  int32_t status, its, k_used, maxit, m, its0, pad;
};

struct GmHostView {   // mirrors GmScalars from bnorm on
  double bnorm, tol, relres, scale;
  int32_t state, status, its, k_used, maxit, m, its0, pad;
};

struct GmWork {
  double* V;      // [m + 1][Np] basis
  double* Z;      // [m][Np] preconditioned basis vectors
  double* w;      // [Np]
  double* pa;     // [kGmGrid][kMaxRestart] partials
  double* pb;     // [kGmGrid][kMaxRestart] partials
  double* pn;     // [kGmGrid] partials of a norm
  GmScalars* sc;
  int Np;
};

inline size_t np_of(int n) { return (3 * (size_t)n + 31) / 32 * 32; }

size_t gm_bytes(int n, int m) {
  const size_t Np = np_of(n);
  return sizeof(double) * ((size_t)(2 * m + 2) * Np + 2 * (kMaxRestart + 1) * kGmGrid + kGmGrid) +
         sizeof(GmScalars) + 256;
}

GmWork gm_carve(int n, int m, void* work) {
  GmWork w;
  w.Np = (int)np_of(n);
  double* d = (double*)work;
  w.V = d;
  d += (size_t)(m + 1) * w.Np;
  w.Z = d;
  d += (size_t)m * w.Np;
  w.w = d;
  d += w.Np;
  w.pa = d;
  d += (size_t)(kMaxRestart + 1) * kGmGrid;
  w.pb = d;
  d += (size_t)(kMaxRestart + 1) * kGmGrid;
  w.pn = d;
  d += kGmGrid;
  w.sc = (GmScalars*)d;
  return w;
}

inline int vec_grid(int N) { return std::min(kGmGrid, std::max(1, blocks_for(N, kGmBlock))); }

// The sums over the wavefront of acc[0 .. JB), JB a power of two: each step
// gives half of a lane's rows to the lane they are exchanged with and adds the
// other half, so JB - 1 exchanges leave one row per lane (64 / JB lanes hold
// the same one, added last) where JB separate sums take 6 JB.  Lane l returns
// the sum of row l / (64 / JB).
// With distance 32 or 16 the swap instructions of the lane halves or rows
// exchange a pair in place; below, a shuffle.
template <int W>
__device__ __forceinline__ double halve_pair(double a, double b) {
  if constexpr (W >= 16) {
    const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
    const unsigned long long ub = __builtin_bit_cast(unsigned long long, b);
    auto swap = [](unsigned p, unsigned q) {
      if constexpr (W == 32)
        return __builtin_amdgcn_permlane32_swap(p, q, false, false);
      else
        return __builtin_amdgcn_permlane16_swap(p, q, false, false);
    };
    const auto lo = swap((unsigned)ua, (unsigned)ub);
    const auto hi = swap((unsigned)(ua >> 32), (unsigned)(ub >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
  } else {
    const bool up = (threadIdx.x & W) != 0;
    return (up ? b : a) + __shfl_xor(up ? a : b, W, kWave);
  }
}
template <int HALF, int W, int JB>
__device__ __forceinline__ double halve_rows(double (&acc)[JB]) {
  if constexpr (HALF >= 1) {
#pragma unroll
    for (int i = 0; i < HALF; ++i) acc[i] = halve_pair<W>(acc[i], acc[i + HALF]);
    return halve_rows<HALF / 2, W / 2, JB>(acc);
  } else {
    double v = acc[0];
#pragma unroll
    for (int w = W; w >= 1; w /= 2) v += __shfl_xor(v, w, kWave);
    return v;
  }
}
template <int JB>
__device__ __forceinline__ double wave_rows(double (&acc)[JB]) {
  return halve_rows<JB / 2, kWave / 2, JB>(acc);
}

// The workgroup's sums of acc[i] (i <= j) into part[blockIdx.x][i].
template <int JB>
__device__ __forceinline__ void store_rows(double (&acc)[JB], int j, double* part,
                                           double (*red)[JB]) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const double v = wave_rows<JB>(acc);
  if (lane % (kWave / JB) == 0) red[wv][lane / (kWave / JB)] = v;
  __syncthreads();
  if ((int)threadIdx.x <= j) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kGmBlock / kWave; ++q) s += red[q][threadIdx.x];
    part[(size_t)blockIdx.x * kMaxRestart + threadIdx.x] = s;
  }
}

// The sums h[i], i < JB, of the partials part[0 .. G)[i] (zero for i > j), in
// the same fixed order in every workgroup: thread t adds row t % JB of the
// partials t / JB, t / JB + 512 / JB, ..., then the wavefront and the
// workgroup.  The first kFirst of a thread are loaded by `first`, to be issued
// ahead of other loads.
template <int JB>
struct RowSums {
  static constexpr int kStep = kGmBlock / JB, kFirst = 4;
  double v[kFirst];
  __device__ __forceinline__ void first(const double* part, int G) {
    const int row = threadIdx.x % JB, q0 = threadIdx.x / JB;
#pragma unroll
    for (int u = 0; u < kFirst; ++u)
      v[u] = part[(size_t)min(q0 + u * kStep, G - 1) * kMaxRestart + row];
  }
  __device__ __forceinline__ void finish(const double* part, int G, int j, double (*red)[JB],
                                         double* h) {
    const int row = threadIdx.x % JB, q0 = threadIdx.x / JB;
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < kFirst; ++u) t += q0 + u * kStep < G ? v[u] : 0.0;
    for (int q = q0 + kFirst * kStep; q < G; q += kStep) t += part[(size_t)q * kMaxRestart + row];
#pragma unroll
    for (int w = JB; w < kWave; w *= 2) t += __shfl_xor(t, w, kWave);
    const int lane = threadIdx.x & (kWave - 1);
    if (lane < JB) red[threadIdx.x / kWave][lane] = t;
    __syncthreads();
    if ((int)threadIdx.x < JB) {
      double sum = 0.0;
#pragma unroll
      for (int q = 0; q < kGmBlock / kWave; ++q) sum += red[q][threadIdx.x];
      h[threadIdx.x] = (int)threadIdx.x <= j ? sum : 0.0;
    }
    __syncthreads();
  }
};

// The sum of the partials part[0 .. G), G <= kGmGrid, in every lane of every
// wavefront (in the same order): loads and end of it.
struct NormSum {
  static constexpr int kLoads = kGmGrid / kWave;
  double v[kLoads];
  __device__ __forceinline__ void first(const double* part, int G) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int u = 0; u < kLoads; ++u) v[u] = part[min(lane + u * kWave, G - 1)];
  }
  __device__ __forceinline__ double finish(int G) {
    const int lane = threadIdx.x & (kWave - 1);
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) t += lane + u * kWave < G ? v[u] : 0.0;
#pragma unroll
    for (int w = kWave / 2; w >= 1; w /= 2) t += __shfl_xor(t, w, kWave);
    return t;
  }
};

// Keeps loads issued before this point, ahead of the tests and the arithmetic
// after it.
__device__ __forceinline__ void loads_issued() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ int read_state(const GmScalars* sc, int* word) {
  if (threadIdx.x == 0) *word = sc->state;
  __syncthreads();
  return *word;
}

// x = 0 and the partials of <b, b>.
__global__ __launch_bounds__(kGmBlock) void k_gm_init(int N, const double* b, double* x,
                                                       GmWork w) {
  __shared__ double sh[kGmBlock / kWave];
  double bb = 0.0;
  for (int k = blockIdx.x * kGmBlock + threadIdx.x; k < N; k += gridDim.x * kGmBlock) {
    x[k] = 0.0;
    bb += b[k] * b[k];
  }
  const double s = block_sum<kGmBlock>(bb, sh);
  if (threadIdx.x == 0) w.pn[blockIdx.x] = s;
}

__global__ __launch_bounds__(kGmBlock) void k_gm_init2(GmWork w, int G, double rtol, int maxit,
                                                        int m) {
  NormSum ns;
  ns.first(w.pn, G);
  const double t = ns.finish(G);
  if (threadIdx.x == 0) {
    GmScalars& c = *w.sc;
    c.bnorm = sqrt(t);
    c.tol = rtol * c.bnorm;
    c.relres = t == 0.0 ? 0.0 : 1.0;
    c.its = 0;
    c.its0 = 0;
    c.maxit = maxit;
    c.m = m;
    c.k_used = 0;
    c.status = t == 0.0 ? OPM_OK : OPM_ENOTCONV;
    c.state = t == 0.0 ? kGmDone : kGmCycleEnd;
  }
}

// y = A x (one group of three block rows per wavefront, the grid of the
// plain SpMV) while the state is `want`; with RES, y = b - A x.
template <bool RES>
__global__ __launch_bounds__(kBlock) void k_gm_spmv(int n, const int32_t* row_ptr,
                                                     const int32_t* col, const double* J,
                                                     const double* x, const double* b, double* y,
                                                     const GmScalars* sc, int want, WellCorr wc) {
  const int st = sc->state;   // (not changed by this kernel)
  if (RES ? st == kGmDone : st != want) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int group = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  if (group >= ilu::spmv_groups(n)) return;   // whole wavefront
  int row, comp;
  double yv;
  if (ilu::spmv_group(n, row_ptr, col, J, x, group, lane, row, comp, yv, wc))
    y[3 * row + comp] = RES ? b[3 * row + comp] - yv : yv;
}

// Partials of ||v_0||^2 at the start of a cycle.
__global__ __launch_bounds__(kGmBlock) void k_gm_norm0(int N, GmWork w) {
  __shared__ double sh[kGmBlock / kWave];
  __shared__ int word;
  if (read_state(w.sc, &word) == kGmDone) return;
  double ss = 0.0;
  for (int k = blockIdx.x * kGmBlock + threadIdx.x; k < N; k += gridDim.x * kGmBlock)
    ss += w.V[k] * w.V[k];
  const double s = block_sum<kGmBlock>(ss, sh);
  if (threadIdx.x == 0) w.pn[blockIdx.x] = s;
}

// Start of a cycle (one workgroup): beta = ||r||; the iteration cap (only
// with maxit = 0, since a cycle that reaches it ends the solve), convergence,
// or g = beta e_0 and run.
__global__ __launch_bounds__(kGmBlock) void k_gm_start(GmWork w, int G) {
  __shared__ int word;
  if (read_state(w.sc, &word) == kGmDone) return;
  NormSum ns;
  ns.first(w.pn, G);
  const double tot = ns.finish(G);
  if (threadIdx.x != 0) return;
  GmScalars& c = *w.sc;
  const double beta = sqrt(tot);
  c.relres = c.bnorm > 0.0 ? beta / c.bnorm : 0.0;
  c.k_used = 0;
  c.its0 = c.its;
  if (c.its >= c.maxit) {
    c.status = OPM_ENOTCONV;
    c.state = kGmDone;
  } else if (beta <= c.tol) {
    c.status = OPM_OK;
    c.state = kGmDone;
  } else {
    c.gres[0] = beta;
    c.scale = 1.0 / beta;
    c.state = kGmRunning;
  }
}

// v_0 *= 1 / beta, while running.
__global__ __launch_bounds__(kGmBlock) void k_gm_scale0(int N, GmWork w) {
  __shared__ int word;
  if (read_state(w.sc, &word) != kGmRunning) return;
  const double f = w.sc->scale;
  for (int k = blockIdx.x * kGmBlock + threadIdx.x; k < N; k += gridDim.x * kGmBlock)
    w.V[k] *= f;
}

// The three kernels of the orthogonalisation are latencies more than bytes
// (9000 cells: 7 MB of basis vectors from the caches), so each asks for all it
// needs first, the state word, the partials of the sums and the first element's
// vectors, and then waits once.  The basis rows are read for all JB rows without
// a branch (rows past j as row j, a cache hit, and weighted by zero).  9000
// cells, 16 to 32 rows: dots 12.1 -> 5.7 us, cgs1 13.5 -> 5.9 us, cgs2 6.7 -> 4.9 us
// (before: sums one row after another, and after the state and the partials).
template <int JB>
__device__ __forceinline__ void load_rows(const GmWork& w, int j, int k, double (&vk)[JB]) {
#pragma unroll
  for (int i = 0; i < JB; ++i) vk[i] = w.V[(size_t)min(i, j) * w.Np + k];
}

// Partials of the first projections h1_i = <v_i, w>, i <= j.
template <int JB>
__global__ __launch_bounds__(kGmBlock) void k_gm_dots(int N, GmWork w, int j) {
  __shared__ double red[kGmBlock / kWave][JB];
  const int state = w.sc->state;   // (not changed by this kernel)
  const int k0 = blockIdx.x * kGmBlock + threadIdx.x;
  double acc[JB], vk[JB];
  load_rows<JB>(w, j, min(k0, N - 1), vk);
  double wk = w.w[min(k0, N - 1)];
  loads_issued();
  if (state != kGmRunning) return;
  if (k0 >= N) wk = 0.0;
#pragma unroll
  for (int i = 0; i < JB; ++i) acc[i] = k0 < N ? vk[i] * wk : 0.0;
  for (int k = k0 + gridDim.x * kGmBlock; k < N; k += gridDim.x * kGmBlock) {
    load_rows<JB>(w, j, k, vk);
    wk = w.w[k];
    __builtin_amdgcn_sched_barrier(0);   // every load of the element issued before the arithmetic
#pragma unroll
    for (int i = 0; i < JB; ++i) acc[i] += vk[i] * wk;
  }
  store_rows<JB>(acc, j, w.pa, red);
}

// First update w -= V h1 (h1 summed from the partials; workgroup 0 keeps
// it) and the partials of the second projections h2_i = <v_i, w>.
template <int JB>
__global__ __launch_bounds__(kGmBlock) void k_gm_cgs1(int N, GmWork w, int j, int G) {
  __shared__ double h[JB];
  __shared__ double red[kGmBlock / kWave][JB];
  const int state = w.sc->state;
  RowSums<JB> rs;
  rs.first(w.pa, G);
  const int k0 = blockIdx.x * kGmBlock + threadIdx.x;
  double acc[JB], vk[JB];
  load_rows<JB>(w, j, min(k0, N - 1), vk);
  double v = w.w[min(k0, N - 1)];
  loads_issued();
  if (state != kGmRunning) return;
  rs.finish(w.pa, G, j, red, h);
  if (blockIdx.x == 0 && (int)threadIdx.x <= j) w.sc->h1[threadIdx.x] = h[threadIdx.x];
#pragma unroll
  for (int i = 0; i < JB; ++i) v -= h[i] * vk[i];
  if (k0 < N) w.w[k0] = v;
#pragma unroll
  for (int i = 0; i < JB; ++i) acc[i] = k0 < N ? vk[i] * v : 0.0;
  for (int k = k0 + gridDim.x * kGmBlock; k < N; k += gridDim.x * kGmBlock) {
    load_rows<JB>(w, j, k, vk);
    v = w.w[k];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < JB; ++i) v -= h[i] * vk[i];
    w.w[k] = v;
#pragma unroll
    for (int i = 0; i < JB; ++i) acc[i] += vk[i] * v;
  }
  store_rows<JB>(acc, j, w.pb, red);
}

// Second update w -= V h2 (workgroup 0 keeps h2) and the partials of ||w||^2.
template <int JB>
__global__ __launch_bounds__(kGmBlock) void k_gm_cgs2(int N, GmWork w, int j, int G) {
  __shared__ double h[JB];
  __shared__ double red[kGmBlock / kWave][JB];
  __shared__ double sh[kGmBlock / kWave];
  const int state = w.sc->state;
  RowSums<JB> rs;
  rs.first(w.pb, G);
  const int k0 = blockIdx.x * kGmBlock + threadIdx.x;
  double vk[JB];
  load_rows<JB>(w, j, min(k0, N - 1), vk);
  double v = w.w[min(k0, N - 1)];
  loads_issued();
  if (state != kGmRunning) return;
  rs.finish(w.pb, G, j, red, h);
  if (blockIdx.x == 0 && (int)threadIdx.x <= j) w.sc->h2[threadIdx.x] = h[threadIdx.x];
#pragma unroll
  for (int i = 0; i < JB; ++i) v -= h[i] * vk[i];
  if (k0 < N) w.w[k0] = v;
  double ss = k0 < N ? v * v : 0.0;
  for (int k = k0 + gridDim.x * kGmBlock; k < N; k += gridDim.x * kGmBlock) {
    load_rows<JB>(w, j, k, vk);
    v = w.w[k];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < JB; ++i) v -= h[i] * vk[i];
    w.w[k] = v;
    ss += v * v;
  }
  const double s = block_sum<kGmBlock>(ss, sh);
  if (threadIdx.x == 0) w.pn[blockIdx.x] = s;
}

__device__ __forceinline__ double lane_value(double v, int lane) {   // uniform `lane`
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Column j of H (h1 + h2, then h_{j+1,j} = ||w||), the earlier rotations and
// the new one, the residual estimate and the decision: converged or an
// exact breakdown (end the cycle, then the solve), end of the cycle (restart
// length or iteration cap), or go on with v_{j+1} = w / h_{j+1,j}.  Every
// wavefront computes the rotation from values this kernel does not write
// (lane i holds entry i of the column and rotation i), so all take the same
// decision; workgroup 0 records it (the state only when the cycle ends, where a
// wavefront that reads it late has nothing to do either).  9000 cells: 4.4 us
// (one thread going through LDS: 4.6 us).
__global__ __launch_bounds__(kGmBlock) void k_gm_rotate(int N, GmWork w, int j, int G) {
  GmScalars& c = *w.sc;
  const int lane = threadIdx.x & (kWave - 1), li = min(lane, kMaxRestart - 1);
  const int state = c.state;
  NormSum ns;
  ns.first(w.pn, G);
  const double a1 = c.h1[li], a2 = c.h2[li], cs = c.cs[li], sn = c.sn[li];
  const double gj = c.gres[j], tol = c.tol, bnorm = c.bnorm;
  const int its = c.its0 + j + 1, m = c.m, maxit = c.maxit;
  const int k0 = blockIdx.x * kGmBlock + threadIdx.x;
  const double w0 = w.w[min(k0, N - 1)];
  loads_issued();
  if (state != kGmRunning) return;
  const double hn = sqrt(ns.finish(G));
  const double col = a1 + a2;
  double h = 0.0;                          // lane i < j: entry i of the rotated column
  double d = lane_value(col, 0);           // the entry the next rotation takes first
  for (int i = 0; i < j; ++i) {
    const double ci = lane_value(cs, i), si = lane_value(sn, i), e = lane_value(col, i + 1);
    const double up = ci * d + si * e;
    d = -si * d + ci * e;
    if (lane == i) h = up;
  }
  const double len = hypot(d, hn);
  const double cj = len > 0.0 ? d / len : 1.0, sj = len > 0.0 ? hn / len : 0.0;
  const double gnext = -sj * gj;
  const bool conv = fabs(gnext) <= tol || hn == 0.0;
  const bool more = !conv && j + 1 < m && its < maxit;
  if (blockIdx.x == 0 && threadIdx.x < kWave) {
    if (lane < j) c.H[lane * kMaxRestart + j] = h;
    if (lane == 0) {
      c.H[j * kMaxRestart + j] = len;
      c.cs[j] = cj;
      c.sn[j] = sj;
      c.gr[j] = cj * gj;
      c.gres[j + 1] = gnext;
      c.its = its;
      c.k_used = j + 1;
      c.relres = fabs(gnext) / bnorm;
      if (conv) c.status = OPM_OK;
      if (!more) c.state = kGmCycleEnd;
    }
  }
  if (!more) return;
  const double f = 1.0 / hn;
  double* vn = w.V + (size_t)(j + 1) * w.Np;
  if (k0 < N) vn[k0] = w0 * f;
  for (int k = k0 + gridDim.x * kGmBlock; k < N; k += gridDim.x * kGmBlock)
    vn[k] = w.w[k] * f;
}

// End of a cycle: y = R^{-1} g over the k columns used (every workgroup
// solves the small triangular system from LDS, identically) and x += Z y,
// unless R is singular.  Lane i holds entry i: a column of R per step, where a
// row per step on one thread took 32^2 / 2 dependent products (20 -> 9 us with
// 32 columns, 9000 cells).
template <int JB>
__global__ __launch_bounds__(kGmBlock) void k_gm_finish(int N, double* x, GmWork w) {
  constexpr int kLd = kMaxRestart + 1;   // (a column's entries in different banks)
  __shared__ double R[kMaxRestart * kLd];
  __shared__ double y[kMaxRestart];
  __shared__ int word, singular;
  if (read_state(w.sc, &word) == kGmDone) return;
  const GmScalars& c = *w.sc;
  const int k = c.k_used;
  for (int q = threadIdx.x; q < k * kMaxRestart; q += kGmBlock)
    R[q / kMaxRestart * kLd + q % kMaxRestart] = c.H[q];
  const int li = min((int)threadIdx.x, kMaxRestart - 1);
  double t = c.gr[li];
  __syncthreads();
  if (threadIdx.x < kWave) {
    const bool zero = (int)threadIdx.x < k && R[li * kLd + li] == 0.0;
    const bool bad = __builtin_amdgcn_ballot_w64(zero) != 0;
    double yi = 0.0;
    for (int q = bad ? -1 : k - 1; q >= 0; --q) {
      const double yq = lane_value(t, q) / R[q * kLd + q];
      if ((int)threadIdx.x == q) yi = yq;
      t -= R[li * kLd + q] * yq;   // (lanes past row q hold nothing that is read again)
    }
    if (threadIdx.x < kMaxRestart) y[threadIdx.x] = yi;
    if (threadIdx.x == 0) singular = bad;
  }
  __syncthreads();
  if (singular || k == 0) return;
  // y is zero past k - 1: rows past k - 1 are read as row k - 1
  for (int e = blockIdx.x * kGmBlock + threadIdx.x; e < N; e += gridDim.x * kGmBlock) {
    double zk[JB];
#pragma unroll
    for (int i = 0; i < JB; ++i) zk[i] = w.Z[(size_t)min(i, k - 1) * w.Np + e];
    const double xe = x[e];
    __builtin_amdgcn_sched_barrier(0);
    double u = 0.0;
#pragma unroll
    for (int i = 0; i < JB; ++i) u += y[i] * zk[i];
    x[e] = xe + u;
  }
}

// After the update (one thread): a singular R ends the solve with
// OPM_EBREAKDOWN (x keeps the previous cycles); convergence or the iteration
// cap end it; otherwise the next cycle starts.
__global__ void k_gm_close(GmWork w) {
  if (threadIdx.x != 0) return;
  GmScalars& c = *w.sc;
  if (c.state == kGmDone) return;
  for (int i = 0; i < c.k_used; ++i)
    if (c.H[i * kMaxRestart + i] == 0.0) {
      c.status = OPM_EBREAKDOWN;
      c.state = kGmDone;
      return;
    }
  if (c.status == OPM_OK || c.its >= c.maxit) c.state = kGmDone;
}

template <int JB>
void launch_projections(const GmWork& w, int j, int N, int G, hipStream_t st) {
  hipLaunchKernelGGL(k_gm_dots<JB>, dim3(G), dim3(kGmBlock), 0, st, N, w, j);
  hipLaunchKernelGGL(k_gm_cgs1<JB>, dim3(G), dim3(kGmBlock), 0, st, N, w, j, G);
  hipLaunchKernelGGL(k_gm_cgs2<JB>, dim3(G), dim3(kGmBlock), 0, st, N, w, j, G);
}

template <int JB>
void launch_finish(const GmWork& w, double* x, int N, int G, hipStream_t st) {
  hipLaunchKernelGGL(k_gm_finish<JB>, dim3(G), dim3(kGmBlock), 0, st, N, x, w);
}

int read_view(const GmWork& w, GmHostView* v, hipStream_t st) {
  OPM_TRY_HIP(hipMemcpyAsync(v, &w.sc->bnorm, sizeof(GmHostView), hipMemcpyDeviceToHost, st));
  OPM_TRY_HIP(hipStreamSynchronize(st));
  return OPM_OK;
}

}  // namespace

size_t gmres_bytes(const opm_problem* pb, int restart) {
  return gm_bytes(pb->n_cells, std::min(std::max(restart, 1), kMaxRestart));
}

// cpr (may be null): CPR-AMG set up for J, with ilu as its second stage.
// ws (may be null): standard wells, solved through their Schur complement
// (the operator subtracts sum_w C_w D_w^{-1} B_w of its argument).
int gmres(const opm_problem* pb, const double* J, void* ilu, int precision, const double* b,
          double* x, double rtol, int maxit, int restart, void* work, opm_solve_report* rep,
          hipStream_t st, const CprWork* cpr, const WellSchur* ws) {
  if (restart < 1 || restart > kMaxRestart || maxit < 0) return OPM_EINVAL;
  const int n = pb->n_cells, N = 3 * n, m = restart;
  GmWork w = gm_carve(n, m, work);
  const int G = vec_grid(N);
  const int Gs = std::max(1, blocks_for(ilu::spmv_groups(n), kBlock / kWave));
  hipLaunchKernelGGL(k_gm_init, dim3(G), dim3(kGmBlock), 0, st, N, b, x, w);
  hipLaunchKernelGGL(k_gm_init2, dim3(1), dim3(kGmBlock), 0, st, w, G, rtol, maxit, m);
  OPM_TRY_HIP(hipGetLastError());
  const int chunk = 6;
  GmHostView v{};
  const WellCorr wc = ws ? ws->wc() : WellCorr{nullptr, nullptr, nullptr};
  for (int cycle = 0;; ++cycle) {
    if (ws) OPM_TRY(well_op(*ws, x, nullptr, st));
    hipLaunchKernelGGL(k_gm_spmv<true>, dim3(Gs), dim3(kBlock), 0, st, n, pb->row_ptr,
                       pb->col_idx, J, x, b, w.V, w.sc, 0, wc);
    hipLaunchKernelGGL(k_gm_norm0, dim3(G), dim3(kGmBlock), 0, st, N, w);
    hipLaunchKernelGGL(k_gm_start, dim3(1), dim3(kGmBlock), 0, st, w, G);
    hipLaunchKernelGGL(k_gm_scale0, dim3(G), dim3(kGmBlock), 0, st, N, w);
    OPM_TRY_HIP(hipGetLastError());
    for (int j0 = 0; j0 < m; j0 += chunk) {
      for (int j = j0; j < std::min(m, j0 + chunk); ++j) {
        double* zj = w.Z + (size_t)j * w.Np;
        const double* vj = w.V + (size_t)j * w.Np;
        if (cpr)
          OPM_TRY(cpr_apply(pb, J, ilu, precision, *cpr, vj, zj, st, &w.sc->state));
        else
          OPM_TRY(ilu_apply(pb, ilu, precision, vj, zj, st, &w.sc->state));
        if (ws) OPM_TRY(well_op(*ws, zj, &w.sc->state, st));
        hipLaunchKernelGGL(k_gm_spmv<false>, dim3(Gs), dim3(kBlock), 0, st, n, pb->row_ptr,
                           pb->col_idx, J, zj, nullptr, w.w, w.sc, (int)kGmRunning, wc);
        if (j < 4)
          launch_projections<4>(w, j, N, G, st);
        else if (j < 8)
          launch_projections<8>(w, j, N, G, st);
        else if (j < 16)
          launch_projections<16>(w, j, N, G, st);
        else
          launch_projections<32>(w, j, N, G, st);
        hipLaunchKernelGGL(k_gm_rotate, dim3(G), dim3(kGmBlock), 0, st, N, w, j, G);
        OPM_TRY_HIP(hipGetLastError());
      }
      OPM_TRY(read_view(w, &v, st));
      if (v.state != kGmRunning) break;
    }
    // the state was read after the last chunk: k_used is final
    if (v.k_used <= 4)
      launch_finish<4>(w, x, N, G, st);
    else if (v.k_used <= 8)
      launch_finish<8>(w, x, N, G, st);
    else if (v.k_used <= 16)
      launch_finish<16>(w, x, N, G, st);
    else
      launch_finish<32>(w, x, N, G, st);
    hipLaunchKernelGGL(k_gm_close, dim3(1), dim3(64), 0, st, w);
    OPM_TRY_HIP(hipGetLastError());
    OPM_TRY(read_view(w, &v, st));
    if (v.state == kGmDone) break;
    if (cycle > maxit + 1) {   // cannot happen: every cycle adds an iteration or stops
      v.status = OPM_ENOTCONV;
      break;
    }
  }
  if (rep) {
    rep->status = v.status;
    rep->half = 0;
    rep->its = v.its;
    rep->rel_res = v.relres;
  }
  return OPM_OK;
}

}  // namespace opm
