// Column sweeps: the ILU(0) factorisation and triangular solves of a box of
// lattice columns by one workgroup (paper sec. 2.3.1), shared by the kernels
// of cols.hip.
//
// A workgroup owns a box of bx x by columns of up to bz cells.  Four lanes (a
// quad) hold one column, lane eq < 3 its equation eq, and walk it one cell per
// level: on level l the column (ci, cj) of the box is at cell k = l - ci - cj,
// so its three lower neighbours are its own previous cell (its value is still
// in the quad's registers), and the cells that the columns ci - 1 and cj - 1
// handled on the previous level (their values are in LDS).  The backward sweep
// walks the levels down.  Every address of a lane (records, neighbour rows,
// exchange slots) is a constant plus a multiple of the level: there is no
// neighbour index to load and no row position to compute.
//
// Why this shape: a sweep is a chain of dependent levels, and one wavefront per
// SIMD pays for each instruction of a level.  With rows found by position (the
// sweeps of ilu0.hip) most of a level is index arithmetic and nine LDS reads per
// lane; here it is one LDS write, four reads, 12 fused multiply-adds and the
// loads of a later level (about 55 instructions, 0.11-0.14 us per level of a
// 4x4 box, against 0.24 us).  One application, both sweeps, by HIP events:
// 9000 cells in 4x4x15 boxes 10.6 -> 6.7 us FP64, 10.1 -> 5.8 us FP32; 500k
// cells in 4x4x50 boxes 56.8 -> 48.3 us (bound by bandwidth: 63 values per row
// instead of 72), FP32 33.8 -> 24.4 us.  The dynamic LDS must be declared
// 16-byte aligned: behind a static 4-byte word its 8-byte reads were misaligned
// and split (8x8x60 cells, FP64: 131 against 43 us).
//
// Storage: slot (box, l, c) for every level and column, also where the column
// has no cell: the index is 0 there, the value zero, and the records are not read.
// Record of (slot, equation): forward the three scaled lower blocks' rows (k, j, i) and the row of D^{-1}, 12 values in 16-byte chunks;
// backward the scaled upper blocks' rows (i, j, k), 9 values, the last one in
// an array of its own.  A level of a box is one contiguous piece.
//
// HALO: the boxes are tiles of one system (the ILU(0) of the whole lattice):
// a tile's western and southern columns need the values of the eastern and
// northern columns of its neighbours.  Those go through exchange arrays that
// hold a marker (a signalling NaN, which no arithmetic returns) until they are
// written through to the device's coherence point.  Two wavefronts of a tile's
// own store and load them (tile_send, tile_receive), the loads two levels ahead
// and again while a value still holds the marker (bounded; a wait that gives up
// takes NaN, so that the solve returns NaN instead of hanging).  Workgroups are dispatched in index order
// and wait only on lower indices.  The forward launch refills the exchange
// arrays of the backward one with the marker and the other way round.
#pragma once

#include "krylov_dev.h"
#include "solver_dev.h"

namespace opm {
namespace ilu {

constexpr int kColsPerWave = 16;
constexpr int kMaxColThreads = 512;   // (FP64 spills registers at 1024)
constexpr int kHaloRows = 32;   // most exchange rows (bx + by) of a tile

struct ColGrid {
  int nx, ny, nz;      // the lattice
  int bx, by, bz;      // cells of a box per axis
  int nbx, nby, nbz;   // boxes per axis
  int C;               // columns of a box, padded to whole wavefronts
  int L;               // levels of a box
  int n;               // cells
  int halo;            // the boxes are tiles of one system
  __host__ __device__ int boxes() const { return nbx * nby * nbz; }
  __host__ __device__ size_t slots() const { return (size_t)boxes() * L * C; }
};

// What the factorisation finds about a slot: byte offsets of the blocks of its
// row in the Jacobian (lower k-, j-, i-, diagonal, upper i+, j+, k+; past its
// end where there is none) and its position.
struct alignas(16) FacSlot {
  unsigned lo[3], diag, up[3];
  int pos;
};

template <typename T>
struct ColView {
  ColGrid g;
  T* rec_f;            // [box][L][12 values as chunks][C][3]
  T* rec_b;            // [box][L][8 values as chunks, then one][C][3]
  int32_t* idx;        // [box][L][C] 24 (cell + 1): past the cell's values, 0: none
  FacSlot* fac;        // [box][L][C]
  T* z;                // HALO: [box][L][C][3] forward results
  T* ex[2];            // HALO: [box][bz][by][3] of the forward / backward sweep
  T* ey[2];            // HALO: [box][bz][bx][3]
  double* eux;         // HALO: [box][bz][by][9] scaled upper blocks
  double* euy;         // HALO: [box][bz][bx][9]
  int32_t* gave_up;    // HALO: [3] a wait of the forward / backward sweep or the factorisation gave up
  unsigned spin;       // polls of a wait before it gives up (0: at once)
};

// A value in LDS (address space 3: 32-bit addresses).
template <typename T>
using Lds = __attribute__((address_space(3))) T;
// Word 3 of a raw buffer resource on gfx9 (32-bit data format, no swizzle).
constexpr int kBufferWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t col_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0,
                                           (int)(unsigned)(bytes < 0xffffffffu ? bytes : 0xffffffffu),
                                           kBufferWord3);
}

template <typename T>
__device__ __forceinline__ T col_load(__amdgpu_buffer_rsrc_t r, int off, int soff = 0) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
__device__ __forceinline__ void col_store(double x, __amdgpu_buffer_rsrc_t r, int off, int soff = 0) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), r, off, soff, 0);
}
__device__ __forceinline__ void col_store(float x, __amdgpu_buffer_rsrc_t r, int off, int soff = 0) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, off, soff, 0);
}

// the marker of a value not yet written (signalling NaNs: arithmetic
// returns quiet ones)
__device__ __forceinline__ void unset_value(double& v) {
  v = __builtin_bit_cast(double, 0x7FF4A5A5A5A5A5A5ull);
}
__device__ __forceinline__ void unset_value(float& v) { v = __builtin_bit_cast(float, 0x7FA5A5A5u); }
__device__ __forceinline__ bool is_unset(double v) {
  return __builtin_bit_cast(unsigned long long, v) == 0x7FF4A5A5A5A5A5A5ull;
}
__device__ __forceinline__ bool is_unset(float v) {
  return __builtin_bit_cast(unsigned, v) == 0x7FA5A5A5u;
}

// Value of lane K of the lane's quad (DPP quad permutation: a VALU move, no
// LDS round trip).
template <int K>
__device__ __forceinline__ double quad_lane(double x) {
  constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, ctrl, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
template <int K>
__device__ __forceinline__ float quad_lane(float x) {
  constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), ctrl, 0xf, 0xf, false));
}

// The end of a level: a workgroup barrier, or for a one-wavefront
// workgroup a wavefront-scope fence (the wavefront's LDS operations are
// performed in order, so the next level's reads see this level's writes
// without waiting for them to complete).
template <int NT>
__device__ __forceinline__ void level_barrier() {
  if (NT == 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Forward right-hand side of a sweep: r itself, or (fused with BiCGStab)
// p = r + beta (p - omega v) or s = r - alpha v, written back for the rows
// of the level.
struct BlockRhs {
  const double* r;
  kry::Fused f;
  double beta, omega, alpha;
};

// The lane's place in its box: column c = (ci, cj), equation eq (lane 3 of a
// quad holds none).
struct ColLane {
  int c, eq, ci, cj;
  int lag;       // level of the column's first cell (far past the last level: no column)
  __device__ __forceinline__ explicit ColLane(const ColGrid& g) {
    const int tid = (int)threadIdx.x;
    c = tid >> 2;
    eq = tid & 3;
    cj = c / g.bx;
    ci = c - cj * g.bx;
    lag = c < g.bx * g.by ? ci + cj : 1 << 29;
  }
  // the column has a place on level l
  __device__ __forceinline__ bool at(int l, int bz) const {
    return (unsigned)(l - lag) < (unsigned)bz;
  }
};

// Rows of the LDS exchange between levels: 4 values per column (equation eq
// at eq), a zero row, then the exchange rows (HALO); two of these, used in
// turn by even and odd levels.
template <int NT, bool HALO>
struct ColRows {
  static constexpr int kZero = NT / 4, kHalo = NT / 4 + 1,
                       kRows = NT / 4 + 1 + (HALO ? kHaloRows : 0);
};
template <typename T, int NT, bool HALO>
constexpr size_t col_rows_bytes() {
  return sizeof(T) * 2 * 4 * ColRows<NT, HALO>::kRows;
}

// Bytes of one level of the records.
template <typename T, bool FWD>
__host__ __device__ inline int col_rec_bytes(int C) {
  return C * 3 * (FWD ? 12 : 9) * (int)sizeof(T);
}

template <typename T>
struct ColJob {
  T a[9];       // rows of the three scaled neighbour blocks
  T d[3];       // forward: row of D^{-1}
  T z;          // backward, HALO: the forward result
  double u[3];  // forward: the vector values the right-hand side is made of
};

// The exchange of a tile with its neighbours, by two wavefronts beside those
// that compute: at most 24 values towards x and 24 towards y per level, one per
// lane.  The sender stores a level's values of the edge columns as soon as the
// level is done; the receiver asks for the neighbours' values two levels ahead
// and has them in the LDS rows of a level before that level starts.  They meet
// the others at the barrier of each level, and a level of those is then that of
// a box on its own: with the exchange in the computing wavefronts (its loads,
// tests and stores in every lane) a level of 256 threads took 0.5 us, where a
// box's takes 0.28 us.  30 x 30 x 10 cells: application 114 -> 69 us, 100 x 100 x
// 50: 441 -> 391 us (FP32 factors 328 -> 252 us).  Levels ahead: every one adds to
// the distance between neighbouring tiles, and none leaves a round trip (0.6 to
// 1 us) on every level; 8, 4, 3, 2, 1 of them: 81, 74.5, 69.7, 69.3, 78 us.
constexpr int kExchange = 128;   // threads of the two wavefronts
template <typename T>
struct TileEdge {
  T* base;
  int off, step, size;   // of level l: off + l step, if in [0, size)
  int row, a;            // LDS row of a level, equation
  bool x;                // towards x (else y)
  __device__ __forceinline__ bool has(int l) const {
    return (unsigned)(off + l * step) < (unsigned)size;
  }
};
// W values per cell (of a sweep 3, of the factorisation 9; the lane's W / 3 are
// consecutive, its first one is here), exchanged through x and y
template <typename T, int W, bool FWD, bool SEND, typename R>
__device__ __forceinline__ TileEdge<T> tile_edge(const ColGrid& g, T* ex, T* ey, int box) {
  const int lane = threadIdx.x & 63, I = box % g.nbx, Jt = box / g.nbx % g.nby;
  const bool x = lane < 3 * g.by;
  const int k = x ? lane : lane - 3 * g.by, p = k / 3, a = k - 3 * p;
  constexpr bool up = FWD == SEND;   // the edge towards higher columns
  const int at = x ? (up ? g.bx - 1 : 0) : (up ? g.by - 1 : 0);
  const int ci = x ? at : p, cj = x ? p : at, per = x ? g.by : g.bx;
  const bool on = (x || k < 3 * g.bx) &&
                  (x ? (up ? I + 1 < g.nbx : I > 0) : (up ? Jt + 1 < g.nby : Jt > 0));
  TileEdge<T> e;
  e.step = W * per;
  e.size = g.bz * e.step;
  const int other = (up ? 1 : -1) * (x ? 1 : g.nbx);
  T* const all = x ? ex : ey;
  e.base = all + (on ? (size_t)(box + (SEND ? 0 : other)) * e.size : 0);
  e.off = (p - (ci + cj) * per) * W + a * (W / 3);
  e.row = SEND ? cj * g.bx + ci : R::kHalo + (W == 3 ? (x ? cj : g.by + ci) : p);
  e.a = a;
  e.x = x;
  if (!on) e.size = 0;
  return e;
}

template <typename T, bool FWD, typename R>
__device__ __forceinline__ void tile_send(const ColView<T>& v, int box, const Lds<T>* nb) {
  const TileEdge<T> e =
      tile_edge<T, 3, FWD, true, R>(v.g, v.ex[FWD ? 0 : 1], v.ey[FWD ? 0 : 1], box);
  const int L = v.g.L;
  __syncthreads();
  for (int s = 0; s < L; ++s) {
    __syncthreads();   // level s is done: its values are in the rows the next one reads
    const int l = FWD ? s : L - 1 - s;
    if (e.has(l))
      __hip_atomic_store(e.base + e.off + l * e.step, (T)nb[((s + 1) & 1) * 4 * R::kRows + 4 * e.row + e.a],
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A value not yet written holds the marker: the receiver polls for it (with the
// levels behind it, in the same round trip), at most v.spin times.
template <typename T, bool FWD, typename R>
__device__ __forceinline__ void tile_receive(const ColView<T>& v, int box, Lds<T>* nb) {
  const TileEdge<T> e =
      tile_edge<T, 3, FWD, false, R>(v.g, v.ex[FWD ? 0 : 1], v.ey[FWD ? 0 : 1], box);
  const int L = v.g.L;
  constexpr int D = 2;
  auto level = [&](int s) { return FWD ? min(s, L - 1) : L - 1 - min(s, L - 1); };
  auto load = [&](int s) {   // (a lane without a value there: the array's first, not used)
    const int l = level(s);
    return __hip_atomic_load(e.has(l) ? e.base + e.off + l * e.step : e.base, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  };
  T h[D];
#pragma unroll
  for (int u = 0; u < D; ++u) h[u] = load(u);
  bool lost = false;
  auto get = [&](int s, int slot) __attribute__((always_inline)) {
    const bool want = s < L && e.has(level(s));
    bool miss = want && (is_unset(h[slot]) || v.spin == 0);
    for (unsigned it = 0; __builtin_amdgcn_ballot_w64(miss) != 0; ++it) {
      if (it >= v.spin || lost) {
        lost = true;
        if (miss) h[slot] = (T)__builtin_nan("");
        __hip_atomic_store(v.gave_up + (FWD ? 0 : 1), 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
#pragma unroll
      for (int u = 0; u < D; ++u) h[(slot + u) % D] = load(s + u);
      miss = want && is_unset(h[slot]);
      if ((it & 63) == 63 && __hip_atomic_load(v.gave_up + (FWD ? 0 : 1), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) != 0)
        lost = true;
    }
    if (want) nb[(s & 1) * 4 * R::kRows + 4 * e.row + e.a] = h[slot];
    h[slot] = load(s + D);
  };
  get(0, 0);
  __syncthreads();
  int s = 1;   // level s is received while level s - 1 is computed
  for (; s + D - 1 <= L; s += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      get(s + u, (1 + u) % D);
      __syncthreads();
    }
  }
#pragma unroll
  for (int u = 0; u < D; ++u) {
    if (s + u > L) return;
    get(s + u, (1 + u) % D);
    __syncthreads();
  }
}

// One sweep of box `box` by the workgroup of NT threads.
//   nb: LDS rows (col_rows_bytes), all zero on entry to the forward sweep
//   zl: !HALO: the box's forward results in LDS, [L][C][3] and one value more
//   (written by the lanes that hold none)
// DEPTH levels of loads are in flight while a level is computed.
// No branch separates a load from its use: what a lane does not need lies
// past the end of its buffer, reads zero and costs no traffic.
template <typename T, int NT, int DEPTH, bool FWD, int MODE, bool HALO, typename Gate>
__device__ __forceinline__ bool col_sweep(const ColView<T>& v, int box, BlockRhs& q, Lds<T>* nb,
                                          Lds<T>* zl, double* x, double& ss, Gate gate) {
  typedef typename Vec16<T>::type V;
  typedef ColRows<NT, HALO> R;
  constexpr int ts = (int)sizeof(T), kV = 16 / ts;
  // jobs in a ring of ND steps, indices in one of 2 ND (an index is loaded ND
  // steps ahead of the loads that need it, so it is older than any load they
  // wait for, and kept until its level is computed); the steps are unrolled
  // over 2 ND, so that every ring slot is a register of its own
  constexpr int ND = DEPTH + 1, P = 2 * ND;
  const ColGrid& g = v.g;
  // (one and two wavefronts: every column of the workgroup, so that the
  // distances between the chunks of a record are constants of the loads)
  const int L = g.L, C = NT <= 128 ? NT / 4 : g.C;
  const ColLane ln(g);
  const int a = min(ln.eq, 2);
  constexpr int kOut = (int)0x80000000;   // an offset past the end of any buffer here
  const bool stored = ln.c < C && ln.eq < 3;
  const int rb = col_rec_bytes<T, FWD>(C);
  const __amdgpu_buffer_rsrc_t rrec =
      col_rsrc((FWD ? v.rec_f : v.rec_b) + (size_t)box * L * C * 3 * (FWD ? 12 : 9),
               (size_t)L * rb);
  const __amdgpu_buffer_rsrc_t ridx = col_rsrc(v.idx + (size_t)box * L * C, (size_t)L * C * 4);
  const int vrec = stored ? (ln.c * 3 + a) * 16 : kOut;
  const int vlast = stored ? (ln.c * 3 + a) * ts : kOut;   // backward: the ninth value
  const int vidx = stored ? ln.c * 4 : kOut;
  const int vcell = a * 8 - 24;           // + its index: this equation of the cell
  const size_t vec_bytes = 24 * (size_t)g.n;
  const __amdgpu_buffer_rsrc_t rz =
      col_rsrc(HALO ? v.z + (size_t)box * L * C * 3 : nullptr, HALO ? (size_t)L * C * 3 * ts : 0);
  const int vz = stored ? (ln.c * 3 + a) * ts : kOut;
  // neighbour rows: the column before (forward) or after (backward) in i and j
  const bool edge_i = FWD ? ln.ci == 0 : ln.ci == g.bx - 1;
  const bool edge_j = FWD ? ln.cj == 0 : ln.cj == g.by - 1;
  const bool col = ln.c < g.bx * g.by;
  int row_i = R::kZero, row_j = R::kZero;
  if (col) {
    row_i = !edge_i ? (FWD ? ln.c - 1 : ln.c + 1) : HALO ? R::kHalo + ln.cj : R::kZero;
    row_j = !edge_j ? (FWD ? ln.c - g.bx : ln.c + g.bx)
                    : HALO ? R::kHalo + g.by + ln.ci : R::kZero;
  }
  auto level = [&](int s) {   // of step s (past the last one: the last one)
    const int sc = min(s, L - 1);
    return FWD ? sc : L - 1 - sc;
  };
  // With one wavefront a step is its instructions more than anything else (156
  // ns of 70 instructions; 53 of them, the loads' chunks at constant distances
  // and these offsets carried along, take 138 ns), so what can be carried from one to the next is: the byte offsets of
  // the next level to load (the last one again past the end) and the place of its
  // forward result.  Nothing is loaded where there is no cell (index 0): on levels
  // above and below a column, of which a box has bx + by - 2 more than bz (6 of 56
  // for 4 x 4 x 50 cells), and at the inactive cells of a masked lattice, whose
  // records would be most of what a sweep reads (100 x 100 x 50, a quarter active,
  // 4 x 4 columns: application 42.0 -> 24.5 us, 30.6 us by the position lists).
  const int last_idx = (L - 1) * C * 4, last_rec = (L - 1) * rb;
  int so_idx = 0, so_rec = 0;   // (backward: from the last level down)
  auto load_idx = [&]() __attribute__((always_inline)) {
    const int i = col_load<int>(ridx, vidx, FWD ? so_idx : last_idx - so_idx);
    so_idx = min(so_idx + C * 4, last_idx);
    return i;
  };
  Lds<T>* zp = HALO ? nullptr
                    : zl + (stored ? ((FWD ? 0 : L - 1) * C + ln.c) * 3 + a : L * C * 3);
  const int zstep = HALO || !stored ? 0 : FWD ? C * 3 : -C * 3;
  auto data = [&](int s, bool at, int ix, ColJob<T>& j, auto next_idx)
      __attribute__((always_inline)) {
    const int l = level(s), so = FWD ? so_rec : last_rec - so_rec;   // (l: HALO)
    const int vr = at ? vrec : kOut;
    so_rec = min(so_rec + rb, last_rec);
    next_idx();
    // 8 or 12 values in whole chunks (backward: the ninth follows them)
#pragma unroll
    for (int c = 0; c < (FWD ? 12 : 8) / kV; ++c) {
      const V w = __builtin_bit_cast(
          V, NT <= 128
                 ? __builtin_amdgcn_raw_buffer_load_b128(rrec, vr + c * C * 48, so, 0)
                 : __builtin_amdgcn_raw_buffer_load_b128(rrec, vr, so + c * C * 48, 0));
#pragma unroll
      for (int e = 0; e < kV; ++e) {
        if (c * kV + e < 9)
          j.a[c * kV + e] = w[e];
        else
          j.d[c * kV + e - 9] = w[e];
      }
    }
    if (!FWD) j.a[8] = col_load<T>(rrec, at ? vlast : kOut, so + 8 * C * 3 * ts);
    if (FWD) {
      const int off = ix + vcell;
      auto ld = [&](const double* base) { return col_load<double>(col_rsrc(base, vec_bytes), off); };
      if (MODE == kry::kFuseNone) j.u[0] = ld(q.r);
      if (MODE == kry::kFuseBegin) {
        j.u[0] = ld(q.f.r);
        j.u[1] = ld(q.f.p);
        j.u[2] = ld(q.f.v);
      }
      if (MODE == kry::kFuseS) {
        j.u[0] = ld(q.f.r);
        j.u[1] = ld(q.f.v);
      }
    } else if (HALO) {
      j.z = col_load<T>(rz, at ? vz : kOut, l * C * 3 * ts);
    }
    // keep every load of the stage here, ahead of the computation of the
    // current level, and the arithmetic on them after this point
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  ColJob<T> jobs[ND];
  int idx[P];
  // prologue: the data of steps 0 .. DEPTH-1, their indices and the ND after
  // (records by the column's range, so that they do not wait for the indices: a
  // round trip per sweep; what an inactive cell's place holds is not used)
#pragma unroll
  for (int s = 0; s < DEPTH + ND; ++s) idx[s] = load_idx();
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) data(s, ln.at(level(s), g.bz), idx[s], jobs[s], []() {});
  // with the first levels' loads in flight: the decisions that need the
  // iteration's scalars (their loads overlap those of the sweep)
  if (!gate(q)) return false;
  T out = (T)0;
  level_barrier<HALO ? 2 * NT : NT>();
  // step s reads the rows of parity s % 2 and writes the others
  auto step = [&](int s, int qq) __attribute__((always_inline)) {
    const Lds<T>* rd = nb + (qq & 1) * 4 * R::kRows;
    const Lds<T>* wi = rd + 4 * row_i;
    const Lds<T>* wj = rd + 4 * row_j;
    const T xi0 = wi[0], xi1 = wi[1], xi2 = wi[2];
    const T xj0 = wj[0], xj1 = wj[1], xj2 = wj[2];
    __builtin_amdgcn_sched_barrier(0);
    const int next = idx[(qq + DEPTH) % P];
    data(s + DEPTH, next != 0, next, jobs[(qq + DEPTH) % ND],
         [&]() { idx[(qq + DEPTH + ND) % P] = load_idx(); });
    const ColJob<T>& j = jobs[qq % ND];
    const int ix = idx[qq];
    const int l = level(s);
    const T xk0 = quad_lane<0>(out), xk1 = quad_lane<1>(out), xk2 = quad_lane<2>(out);
    // the same expressions as the unfused vector kernels of the iteration
    double u = j.u[0];
    if (FWD && MODE == kry::kFuseBegin) u = j.u[0] + q.beta * (j.u[1] - q.omega * j.u[2]);
    if (FWD && MODE == kry::kFuseS) u = j.u[0] - q.alpha * j.u[1];
    T o;
    if (FWD) {
      const T r = (T)u;
      o = dot3(j.d[0], quad_lane<0>(r), j.d[1], quad_lane<1>(r), j.d[2], quad_lane<2>(r));
      o = sub_dot3(o, j.a, xk0, xk1, xk2);
      o = sub_dot3(o, j.a + 3, xj0, xj1, xj2);
      o = sub_dot3(o, j.a + 6, xi0, xi1, xi2);
    } else {
      o = HALO ? j.z : *zp;
      if (!HALO) zp += zstep;
      o = sub_dot3(o, j.a, xi0, xi1, xi2);
      o = sub_dot3(o, j.a + 3, xj0, xj1, xj2);
      o = sub_dot3(o, j.a + 6, xk0, xk1, xk2);
    }
    out = ix != 0 ? o : (T)0;
    nb[((qq & 1) ^ 1) * 4 * R::kRows + 4 * ln.c + ln.eq] = out;
    const int off = ix + vcell;
    if (HALO) {
      if (FWD) col_store(out, rz, ix != 0 ? vz : kOut, l * C * 3 * ts);
    } else if (FWD) {
      *zp = out;
      zp += zstep;
    }
    if (!FWD) col_store((double)out, col_rsrc(x, vec_bytes), off);
    if (FWD && MODE == kry::kFuseBegin) col_store(u, col_rsrc(q.f.p, vec_bytes), off);
    if (FWD && MODE == kry::kFuseS) {
      col_store(u, col_rsrc(q.f.s, vec_bytes), off);
      ss += ix != 0 ? u * u : 0.0;
    }
    level_barrier<HALO ? 2 * NT : NT>();
  };
  // (the last levels apart: an exit inside the loop meets its back edge in the
  // compiled code, which then waits there as for the loads of the shortest way)
  int s = 0;
#pragma clang loop unroll(disable)
  for (; s + P <= L; s += P) {
#pragma unroll
    for (int qq = 0; qq < P; ++qq) step(s + qq, qq);
  }
#pragma unroll
  for (int qq = 0; qq < P; ++qq) {
    if (s + qq >= L) return true;
    step(s + qq, qq);
  }
  return true;
}

}  // namespace ilu
}  // namespace opm
