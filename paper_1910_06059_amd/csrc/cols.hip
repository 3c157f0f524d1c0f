// ILU(0) preconditioner by columns: the factorisation and the triangular
// solves of the boxes of a lattice, one workgroup per box (cols_dev.h has the
// shape of the sweeps and the storage).  Two uses:
//  - the block ILU0 (paper sec. 2.5), a box per subdomain, and the ILU(0) of
//    a whole system of few columns, one box: both sweeps in one launch, the
//    forward results in LDS;
//  - the ILU(0) of a whole lattice (sec. 2.3.1) cut into tiles that exchange
//    the values of their boundary columns while they run (HALO): one launch
//    per sweep.  The chain of dependent levels is the whole system's, but all
//    tiles walk it at once, a few levels behind each other.
#include <algorithm>

#include "cols_dev.h"

namespace opm {

extern int g_plane_spin;

namespace {

using namespace ilu;

constexpr size_t kMaxColLds = 150 * 1024;

inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }

// ---------------------------------------------------------- factorisation
// Three launches (and the exchange arrays' reset for tiles):
//  - k_cols_slots finds where the blocks of every slot's row lie, all slots at
//    once, so that the recursion loads one 32-byte index record per slot
//    instead of following a chain of three loads;
//  - k_cols_pivots walks the levels: D_i = A_ii - sum_k A_ik (D_k^{-1} A_ki)
//    takes the scaled upper blocks that the three lower neighbours have just
//    formed (its own column's from the quad's registers, the others' from
//    LDS), inverts, scales the row's upper blocks and passes them on.  Only
//    what the next level waits for is in this chain.  Lane eq of a quad holds
//    row eq of the lower blocks and of D, and column eq of the upper blocks, so
//    that each product needs either only its own values or the whole D^{-1},
//    which every lane forms;
//  - k_cols_records scales the blocks and writes the sweeps' records, all
//    slots at once (it reads the matrix a second time: cheaper than its stores
//    and its products in the chain).
// Factorisation with its records, by HIP events, against the recursion by
// position and a packing pass: 9000 cells 40.2 -> 27.7 us, 500k cells
// (4x4x50 boxes) 304 -> 207 us FP64.  Whole lattices, the exchange in the
// computing wavefronts -> beside them: 30 x 30 x 10 165 -> 109 us, 100 x 100 x 50
// 875 -> 745 us.
struct FacIn {
  const double* J;
  const int32_t* row_ptr;
  const int32_t* box_cell;
  const int32_t* iperm;
  // the neighbours of a block topology, by position (null: nothing to compare)
  const int32_t *lo_blk, *up_blk;
  int32_t* status;
  double* dinv64;
  void* dinv;   // in the sweeps' precision (FP32: an array of its own)
  int ns, nnzb;
};

// In a slot's index record: no such block (past the end of the matrix, with
// room for the offsets added to it).
constexpr unsigned kNoBlock = 0xffffff00u;

// The neighbours that the box gives a row, and those of the topology: the same
// blocks, in any order.
__device__ __forceinline__ bool same_blocks(const unsigned* at, const int32_t* list) {
  const int l[3] = {list[0], list[1], list[2]};
  int found = 0, listed = 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    listed += l[q] >= 0 ? 1 : 0;
#pragma unroll
    for (int e = 0; e < 3; ++e) found += l[e] >= 0 && (unsigned)l[e] * 72u == at[q] ? 1 : 0;
  }
  int wanted = 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) wanted += at[q] != kNoBlock ? 1 : 0;
  return found == wanted && listed == wanted;
}

template <typename T>
__global__ __launch_bounds__(256) void k_cols_slots(ColView<T> v, FacIn f) {
  const ColGrid& g = v.g;
  const unsigned slot = blockIdx.x * 256u + threadIdx.x;
  if (blockIdx.x == 0)   // the padding of the inverse pivots
    for (int e = threadIdx.x; e < 9 * (f.ns - g.n); e += 256) {
      const size_t at = (size_t)(e / (f.ns - g.n)) * f.ns + g.n + e % (f.ns - g.n);
      f.dinv64[at] = 0.0;
      if (sizeof(T) != sizeof(double)) ((T*)f.dinv)[at] = (T)0;
    }
  if (slot >= g.slots()) return;
  const int row = (int)(slot / (unsigned)g.C), c = (int)(slot - (unsigned)row * (unsigned)g.C);
  const int box = row / g.L, s = row - box * g.L;
  const int cj = c / g.bx, ci = c - cj * g.bx, kk = s - ci - cj;
  const int gi = box % g.nbx * g.bx + ci, gj = box / g.nbx % g.nby * g.by + cj;
  const int k = box / (g.nbx * g.nby) * g.bz + kk;
  FacSlot rec{{kNoBlock, kNoBlock, kNoBlock}, kNoBlock, {kNoBlock, kNoBlock, kNoBlock}, 0};
  int cell = -1;
  if (c < g.bx * g.by && gi < g.nx && gj < g.ny && kk >= 0 && kk < g.bz && k < g.nz) {
    const int sxy = g.nx * g.ny;
    const int32_t* b = f.box_cell + gi + g.nx * gj + (size_t)sxy * k;
    cell = b[0];
    if (cell >= 0) {
      const bool in[6] = {k > 0, gj > 0, gi > 0, gi + 1 < g.nx, gj + 1 < g.ny, k + 1 < g.nz};
      const int step[6] = {-sxy, -g.nx, -1, 1, g.nx, sxy};
      const bool h = g.halo != 0;
      const bool own[6] = {kk > 0, h || cj > 0, h || ci > 0, h || ci + 1 < g.bx,
                           h || cj + 1 < g.by, kk + 1 < g.bz};
      unsigned at = (unsigned)f.row_ptr[cell] * 72u;   // the row's blocks in column order
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        if (q == 3) {
          rec.diag = at;
          at += 72u;
        }
        const bool act = in[q] && b[in[q] ? step[q] : 0] >= 0;
        if (act && own[q]) (q < 3 ? rec.lo[q] : rec.up[q - 3]) = at;
        at += act ? 72u : 0u;
      }
      rec.pos = f.iperm[cell];
      // a box that is not the topology's: OPM_EINVAL, and no factors of this
      // row (its records are NaN).  The comparison reads 24 bytes per cell: the
      // factorisation of 500,000 cells 203 -> 207 us, of 9000 cells 27.0 -> 27.7 us
      if (f.lo_blk && !(same_blocks(rec.lo, f.lo_blk + 3 * (size_t)rec.pos) &&
                        same_blocks(rec.up, f.up_blk + 3 * (size_t)rec.pos))) {
        rec = FacSlot{{kNoBlock, kNoBlock, kNoBlock}, kNoBlock, {kNoBlock, kNoBlock, kNoBlock}, -1};
        if (f.status) *f.status = OPM_EINVAL;
      }
    }
  }
  v.fac[slot] = rec;
  v.idx[slot] = 24 * (cell + 1);
}

// three consecutive doubles
__device__ __forceinline__ void load3(__amdgpu_buffer_rsrc_t r, unsigned off, double* x) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 w = __builtin_bit_cast(v2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
  x[0] = w[0];
  x[1] = w[1];
  x[2] = col_load<double>(r, (int)off + 16);
}

struct FacRow {
  double lo[3][3], D[3];   // row a of the lower blocks (k-, j-, i-) and of the diagonal
  double up[3][3];         // column a of the upper blocks (i+, j+, k+)
};
// The exchange of a tile's factorisation, by two wavefronts as in the sweeps
// (tile_send, tile_receive): the scaled upper blocks of the edge columns, three
// values per lane.
template <typename R, int kB>
__device__ __forceinline__ void factor_send(const ColGrid& g, double* eux, double* euy, int box,
                                            const Lds<double>* ui, const Lds<double>* uj) {
  const TileEdge<double> e = tile_edge<double, 9, true, true, R>(g, eux, euy, box);
  const Lds<double>* u = (e.x ? ui : uj) + e.row * kB + 3 * e.a;
  __syncthreads();
  for (int s = 0; s < g.L; ++s) {
    __syncthreads();
    if (e.has(s))
#pragma unroll
      for (int k = 0; k < 3; ++k)
        __hip_atomic_store(e.base + e.off + s * e.step + k,
                           (double)u[((s + 1) & 1) * R::kRows * kB + k], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  }
}
template <typename R, int kB>
__device__ __forceinline__ void factor_receive(const ColGrid& g, double* eux, double* euy,
                                               int box, int32_t* gave_up, unsigned spin,
                                               int32_t* status, Lds<double>* ui,
                                               Lds<double>* uj) {
  const TileEdge<double> e = tile_edge<double, 9, true, false, R>(g, eux, euy, box);
  Lds<double>* u = (e.x ? ui : uj) + e.row * kB + 3 * e.a;
  bool lost = false;
  for (int s = 0; s <= g.L; ++s) {   // level s before its barrier
    const bool want = s < g.L && e.has(s);
    const double* p = want ? e.base + e.off + s * e.step : e.base;   // (or the array's first)
    double h[3];
    bool miss = want;
    for (unsigned it = 0; __builtin_amdgcn_ballot_w64(miss) != 0; ++it) {
      if (it > spin || spin == 0 || lost) {
        lost = true;
        __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (status) *status = OPM_EHIP;
        if (miss) h[0] = h[1] = h[2] = 0.0;
        break;
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
        h[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      miss = want && (is_unset(h[0]) || is_unset(h[1]) || is_unset(h[2]));
      if ((it & 63) == 63 &&
          __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
        lost = true;
    }
    if (want)
#pragma unroll
      for (int k = 0; k < 3; ++k) u[(s & 1) * R::kRows * kB + k] = h[k];
    __syncthreads();
  }
}

template <typename T, int NT, bool HALO>
__global__ __launch_bounds__(NT + (HALO ? kExchange : 0)) void k_cols_pivots(ColView<T> v, FacIn f) {
  typedef ColRows<NT, HALO> R;
  constexpr int kB = 10;   // doubles of a block's place in LDS
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // scaled upper blocks towards i + 1 and j + 1 of every column, column by
  // column: two levels
  Lds<double>* ui = (Lds<double>*)reinterpret_cast<double*>(smem);
  Lds<double>* uj = ui + 2 * kB * R::kRows;
  const ColGrid& g = v.g;
  const int box = (int)blockIdx.x, L = g.L, C = g.C;
  const ColLane ln(g);
  const int a = min(ln.eq, 2);
  for (int e = threadIdx.x; e < 4 * kB * R::kRows; e += NT + (HALO ? kExchange : 0)) ui[e] = 0.0;
  __syncthreads();
  if (HALO) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    if (wave == NT / 64) {
      factor_send<R, kB>(g, v.eux, v.euy, box, ui, uj);
      return;
    }
    if (wave > NT / 64) {
      factor_receive<R, kB>(g, v.eux, v.euy, box, v.gave_up + 2, v.spin, f.status, ui, uj);
      return;
    }
  }
  constexpr int kOut = (int)0x80000000;
  const __amdgpu_buffer_rsrc_t rslot = col_rsrc(v.fac + (size_t)box * L * C, (size_t)L * C * 32);
  const __amdgpu_buffer_rsrc_t rj = col_rsrc(f.J, (size_t)f.nnzb * 72);
  const int vslot = ln.c < C ? ln.c * 32 : kOut;
  auto slot_at = [&](int s) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const int l = min(s, L - 1), so = l * C * 32, vs = ln.at(l, g.bz) ? vslot : kOut;
    const u4 p = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rslot, vs, so, 0));
    const u4 q = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rslot, vs, so + 16, 0));
    return FacSlot{{p[0], p[1], p[2]}, p[3], {q[0], q[1], q[2]}, (int)q[3]};
  };
  auto data = [&](int s, const FacSlot& r, FacRow& b) __attribute__((always_inline)) {
    const unsigned none = ln.at(min(s, L - 1), g.bz) ? 0u : kNoBlock;   // (sets every bit that matters)
    load3(rj, (r.diag | none) + 24u * a, b.D);
#pragma unroll
    for (int q = 0; q < 3; ++q) load3(rj, (r.lo[q] | none) + 24u * a, b.lo[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int e = 0; e < 3; ++e)
        b.up[q][e] = col_load<double>(rj, (int)((r.up[q] | none) + 8u * a) + 24 * e);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int row_i = R::kZero, row_j = R::kZero;
  if (ln.c < g.bx * g.by) {
    row_i = ln.ci > 0 ? ln.c - 1 : HALO ? R::kHalo + ln.cj : R::kZero;
    row_j = ln.cj > 0 ? ln.c - g.bx : HALO ? R::kHalo + ln.ci : R::kZero;
  }
  double uk[9];   // the column's scaled block towards k + 1 on the previous level
#pragma unroll
  for (int e = 0; e < 9; ++e) uk[e] = 0.0;
  // level s: the rows of the next DEPTH levels and the indices of the levels
  // up to s + 5 in flight (512 threads, and 256 beside the exchange, have
  // registers for one level of rows)
  constexpr int DEPTH = NT < (HALO ? 256 : 512) ? 2 : 1, ND = DEPTH + 1;
  FacRow rows[ND];
  FacSlot slots[6];
#pragma unroll
  for (int s = 0; s < 5; ++s) slots[s] = slot_at(s);
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) data(s, slots[s], rows[s]);
  level_barrier<HALO ? 2 * NT : NT>();
  auto step = [&](int s, int qq) __attribute__((always_inline)) {
    const int par = qq & 1;
    double Ui[9], Uj[9];   // column by column
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      Uj[e] = uj[(par * R::kRows + row_j) * kB + e];
      Ui[e] = ui[(par * R::kRows + row_i) * kB + e];
    }
    __builtin_amdgcn_sched_barrier(0);
    slots[(qq + 5) % 6] = slot_at(s + 5);
    data(s + DEPTH, slots[(qq + DEPTH) % 6], rows[(qq + DEPTH) % ND]);
    const FacRow& b = rows[qq % ND];
    const FacSlot& r = slots[qq % 6];
    const bool live = ln.at(s, g.bz) && r.diag != kNoBlock;
    double D[3] = {b.D[0], b.D[1], b.D[2]};
    auto update = [&](const double* A, const double* U) {
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double upd = dot3(A[0], U[3 * e], A[1], U[3 * e + 1], A[2], U[3 * e + 2]);
        D[e] -= upd;
      }
    };
    update(b.lo[0], uk);
    update(b.lo[1], Uj);
    update(b.lo[2], Ui);
    double full[9], inv[9];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      full[e] = quad_lane<0>(D[e]);
      full[3 + e] = quad_lane<1>(D[e]);
      full[6 + e] = quad_lane<2>(D[e]);
    }
    const bool ok = inverse3(full, inv);
    if (!ok && live && f.status) *f.status = OPM_ESINGULAR;
#pragma unroll
    for (int e = 0; e < 9; ++e) inv[e] = ok && live ? inv[e] : 0.0;
    // column a of D^{-1} A for the upper blocks
    double U[3][3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int e = 0; e < 3; ++e)
        U[q][e] = dot3(inv[3 * e], b.up[q][0], inv[3 * e + 1], b.up[q][1], inv[3 * e + 2],
                       b.up[q][2]);
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      if (ln.eq < 3) {
        ui[((par ^ 1) * R::kRows + ln.c) * kB + 3 * a + e] = U[0][e];
        uj[((par ^ 1) * R::kRows + ln.c) * kB + 3 * a + e] = U[1][e];
      }
      uk[e] = quad_lane<0>(U[2][e]);
      uk[3 + e] = quad_lane<1>(U[2][e]);
      uk[6 + e] = quad_lane<2>(U[2][e]);
    }
    if (live && ln.eq < 3) {
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double di = a == 0 ? inv[e] : a == 1 ? inv[3 + e] : inv[6 + e];
        const size_t at = (size_t)(3 * a + e) * f.ns + r.pos;
        f.dinv64[at] = di;
        if (sizeof(T) != sizeof(double)) ((T*)f.dinv)[at] = (T)di;
      }
    }
    level_barrier<HALO ? 2 * NT : NT>();
  };
  for (int s = 0;; s += 6) {
#pragma unroll
    for (int qq = 0; qq < 6; ++qq) {
      step(s + qq, qq);
      if (s + qq + 1 >= L) return;
    }
  }
}

// The sweeps' records: row a of D^{-1} A for the lower blocks and of D^{-1}
// (forward), of D^{-1} A for the upper blocks (backward).
template <typename T>
__global__ __launch_bounds__(256) void k_cols_records(ColView<T> v, FacIn f) {
  typedef typename Vec16<T>::type V;
  constexpr int ts = (int)sizeof(T), kV = 16 / ts;
  const ColGrid& g = v.g;
  const size_t slot = (size_t)blockIdx.x * 64 + threadIdx.x / 4;
  const int a = (int)(threadIdx.x & 3u);
  if (slot >= g.slots() || a == 3) return;
  const FacSlot r = v.fac[slot];
  const bool live = r.diag != kNoBlock;
  // (a wait of the recursion gave up: the pivots that went on from zeros are no
  // factors of this matrix, and every solve with them returns NaN; so does one
  // with a box that is not the topology's)
  const bool lost = r.pos < 0 || (live && g.halo && v.gave_up[2] != 0);
  // (sixteen slots without a cell: nobody reads their records, and they are whole
  // cache lines; single ones are written, 110 -> 131 us at 500,000 cells otherwise)
  if (__builtin_amdgcn_ballot_w64(live || lost) == 0) return;
  double di[3];
#pragma unroll
  for (int e = 0; e < 3; ++e)
    di[e] = lost  ? __builtin_nan("")
            : live ? f.dinv64[(size_t)(3 * a + e) * f.ns + r.pos]
                   : 0.0;
  const __amdgpu_buffer_rsrc_t rj = col_rsrc(f.J, (size_t)f.nnzb * 72);
  auto scaled = [&](unsigned o, T* S) {
    double A[9];
#pragma unroll
    for (int e = 0; e < 3; ++e) load3(rj, o + 24u * e, A + 3 * e);
#pragma unroll
    for (int e = 0; e < 3; ++e) S[e] = (T)dot3(di[0], A[e], di[1], A[3 + e], di[2], A[6 + e]);
  };
  T wf[12], wb[9];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    scaled(r.lo[q], wf + 3 * q);
    scaled(r.up[q], wb + 3 * q);
    wf[9 + q] = (T)di[q];
  }
  const size_t c = slot % g.C, level = slot / g.C;
  char* pf = (char*)v.rec_f + level * col_rec_bytes<T, true>(g.C) + (c * 3 + a) * 16;
  char* pb = (char*)v.rec_b + level * col_rec_bytes<T, false>(g.C);
#pragma unroll
  for (int q = 0; q < 12 / kV; ++q) {
    V w;
#pragma unroll
    for (int e = 0; e < kV; ++e) w[e] = wf[q * kV + e];
    *reinterpret_cast<V*>(pf + (size_t)q * g.C * 48) = w;
  }
#pragma unroll
  for (int q = 0; q < 8 / kV; ++q) {
    V w;
#pragma unroll
    for (int e = 0; e < kV; ++e) w[e] = wb[q * kV + e];
    *reinterpret_cast<V*>(pb + (size_t)q * g.C * 48 + (c * 3 + a) * 16) = w;
  }
  *reinterpret_cast<T*>(pb + (size_t)8 * g.C * 3 * ts + (c * 3 + a) * ts) = wb[8];
}

// Fills `n` values with the marker of a value not yet written.
template <typename T>
__device__ __forceinline__ void mark(T* p, size_t n, size_t first, size_t stride) {
  T u;
  unset_value(u);
  for (size_t e = first; e < n; e += stride) p[e] = u;
}

// Before a factorisation: every exchange array holds the marker, no wait gave up.
template <typename T>
__global__ __launch_bounds__(256) void k_cols_reset(ColView<T> v) {
  const size_t first = blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  const size_t nx = (size_t)v.g.boxes() * v.g.bz * v.g.by, ny = (size_t)v.g.boxes() * v.g.bz * v.g.bx;
  for (int q = 0; q < 2; ++q) {
    mark(v.ex[q], 3 * nx, first, stride);
    mark(v.ey[q], 3 * ny, first, stride);
  }
  mark(v.eux, 9 * nx, first, stride);
  mark(v.euy, 9 * ny, first, stride);
  if (first < 3) v.gave_up[first] = 0;
}

// --------------------------------------------------------------- sweeps
// Start of a sweep kernel: the skip flag or the iteration's state word (read
// once for the workgroup) and the LDS rows cleared.  Returns false if the
// sweep does not run.
template <typename T, int NT, bool HALO, int MODE>
__device__ __forceinline__ bool cols_begin(Lds<T>* nb, const int32_t* skip, const kry::Fused& f,
                                           int* word, int& state) {
  int w = 0;
  if (threadIdx.x == 0) w = MODE != kry::kFuseNone ? f.sc->state : skip ? *skip : 0;
  for (int e = threadIdx.x; e < 8 * ColRows<NT, HALO>::kRows; e += NT + (HALO ? kExchange : 0))
    nb[e] = (T)0;
  if (threadIdx.x == 0) *word = w;
  __syncthreads();
  state = *word;
  if (MODE == kry::kFuseNone) return state == 0;
  if (state != kry::kRunning) {
    if (MODE == kry::kFuseBegin && state == kry::kHalfPending && blockIdx.x == 0 &&
        threadIdx.x == 0)
      f.sc->state = kry::kDone;
    return false;
  }
  return true;
}

// The iteration's tests and scalars (every workgroup on the same partials).
// What they need is asked for at the start of the kernel, ahead of the sweep's
// first levels: loaded behind those, the sums waited for all of them (9000
// cells: p update and application 9.42 -> 8.93 us, s update and application 9.99
// -> 8.80 us).
template <int NT, int MODE>
struct ColsGate {
  kry::Shares<NT> a, b;
  kry::IterScalars c;
  __device__ __forceinline__ void load(const kry::Fused& f) {
    if (MODE == kry::kFuseNone) return;
    a.load(f.part_a, f.n_part);
    if (MODE == kry::kFuseBegin) b.load(f.part_b, f.n_part);
    c.load(*f.sc);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ bool pass(const kry::Fused& f, int state, double* red,
                                       BlockRhs& q) const {
    if (MODE == kry::kFuseBegin)
      return kry::begin_iteration_share<NT>(*f.sc, state, c, a.share(f.n_part), b.share(f.n_part),
                                            red, q.beta, q.omega);
    if (MODE == kry::kFuseS)
      return kry::alpha_step_share<NT>(*f.sc, state, c.rho, a.share(f.n_part), red, q.alpha);
    return true;
  }
};

// The box of this workgroup: workgroups go to the 8 XCDs in turn, and each
// XCD gets a contiguous range of boxes, because the cells of boxes next to
// each other in x share cache lines of the vectors (a row of 4 cells is 96
// bytes): one L2 then holds both sides of a line.  500,000 cells in 4x4 columns:
// p update and application 76.9 -> 75.8 us, s update and application 72.1 ->
// 70.5 us, application 54.3 -> 52.8 us.
__device__ __forceinline__ int xcd_box(int boxes) {
  const int w = (int)blockIdx.x, q = boxes / 8, r = boxes % 8;
  const int xcd = w % 8;
  return xcd * q + min(xcd, r) + w / 8;
}

// x = M^{-1} r of one box per workgroup, both sweeps.  MODE (kry::FusedMode):
// the forward right-hand side is r, or the p or s update of a BiCGStab
// iteration, preceded by the tests of that iteration; with the s update the
// workgroup's partial of <s, s> goes to f.part_out.
template <typename T, int NT, int DEPTH, int MODE>
__global__ __launch_bounds__(NT) void k_cols_apply(ColView<T> v, const double* r, double* x,
                                                    const int32_t* skip, kry::Fused f) {
  __shared__ double red[2 * NT / 64];
  __shared__ int word;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  Lds<T>* nb = (Lds<T>*)reinterpret_cast<T*>(smem);
  Lds<T>* zl = nb + 8 * ColRows<NT, false>::kRows;
  int state;
  ColsGate<NT, MODE> gate;
  gate.load(f);
  if (!cols_begin<T, NT, false, MODE>(nb, skip, f, &word, state)) return;
  BlockRhs q{r, f, 0.0, 0.0, 0.0};
  double ss = 0.0;
  const int box = xcd_box(v.g.boxes());
  if (!col_sweep<T, NT, DEPTH, true, MODE, false>(
          v, box, q, nb, zl, x, ss,
          [&](BlockRhs& qq) { return gate.pass(f, state, red, qq); }))
    return;
  if (MODE == kry::kFuseS) {
    const double tot = block_sum<NT>(ss, red);
    if (threadIdx.x == 0) f.part_out[box] = tot;
  }
  col_sweep<T, NT, DEPTH, false, MODE, false>(v, box, q, nb, zl, x, ss,
                                              [](BlockRhs&) { return true; });
}

// One sweep of the tiles of a whole lattice.  Backward workgroups take the
// tiles in descending order, so that they too wait on lower indices only.
template <typename T, int NT, int DEPTH, bool FWD, int MODE>
__global__ __launch_bounds__(NT + kExchange) void k_cols_tiles(ColView<T> v, const double* r,
                                                                double* x, const int32_t* skip,
                                                                kry::Fused f) {
  typedef ColRows<NT, true> R;
  constexpr int kAll = NT + kExchange;
  __shared__ double red[2 * kAll / 64];
  __shared__ int word;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  Lds<T>* nb = (Lds<T>*)reinterpret_cast<T*>(smem);
  int state;
  // (the backward launch of a fused pair is skipped like its forward one: by
  // the iteration's state, as `skip`)
  constexpr int M = FWD ? MODE : kry::kFuseNone;
  ColsGate<kAll, M> sums;
  sums.load(f);
  if (!cols_begin<T, NT, true, M>(nb, skip, f, &word, state)) return;
  BlockRhs q{r, f, 0.0, 0.0, 0.0};
  double ss = 0.0;
  const int box = FWD ? (int)blockIdx.x : v.g.boxes() - 1 - (int)blockIdx.x;
  // (every wavefront of the workgroup takes the same decision, and the same
  // number of barriers)
  auto gate = [&](BlockRhs& qq) { return sums.pass(f, state, red, qq); };
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  if (wave < NT / 64) {
    if (!col_sweep<T, NT, DEPTH, FWD, M, true>(v, box, q, nb, (Lds<T>*)nullptr, x, ss, gate))
      return;
  } else {
    if (!gate(q)) return;
    if (wave == NT / 64)
      tile_send<T, FWD, R>(v, box, nb);
    else
      tile_receive<T, FWD, R>(v, box, nb);
  }
  if (FWD && MODE == kry::kFuseS) {
    const double tot = block_sum<kAll>(ss, red);
    if (threadIdx.x == 0) f.part_out[box] = tot;
  }
  // the other sweep's exchange arrays of this tile, and its give-up word
  constexpr int o = FWD ? 1 : 0;
  const size_t nx = (size_t)3 * v.g.bz * v.g.by, ny = (size_t)3 * v.g.bz * v.g.bx;
  mark(v.ex[o] + box * nx, nx, threadIdx.x, kAll);
  mark(v.ey[o] + box * ny, ny, threadIdx.x, kAll);
  if (blockIdx.x == 0 && threadIdx.x == 0) v.gave_up[o] = 0;
}

// ------------------------------------------------------------ host side
// one flag per kernel instantiation
bool g_cols_lds_set[64] = {};

template <typename K>
int allow_lds(K kernel, int slot) {
  if (!g_cols_lds_set[slot]) {
    hipFuncAttributes at;
    OPM_TRY_HIP(hipFuncGetAttributes(&at, reinterpret_cast<const void*>(kernel)));
    OPM_TRY_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024 - (int)at.sharedSizeBytes));
    g_cols_lds_set[slot] = true;
  }
  return OPM_OK;
}

// threads for a level of that many rows, and of a box's workgroup: a power of
// two of wavefronts
int threads_of_rows(int rows) {
  int nt = 64;
  while (nt / 64 * kColsPerWave < rows) nt *= 2;
  return nt;
}
int threads_of(const ColGrid& g) { return threads_of_rows(g.C); }

ColGrid make_grid(const opm_problem* pb, int bx, int by, int bz, bool halo) {
  ColGrid g;
  g.nx = pb->nx;
  g.ny = pb->ny;
  g.nz = pb->nz;
  g.bx = std::min(bx, g.nx);
  g.by = std::min(by, g.ny);
  g.bz = std::min(bz, g.nz);
  g.nbx = (g.nx + g.bx - 1) / g.bx;
  g.nby = (g.ny + g.by - 1) / g.by;
  g.nbz = (g.nz + g.bz - 1) / g.bz;
  g.C = (int)((long)((long)g.bx * g.by + kColsPerWave - 1) / kColsPerWave * kColsPerWave);
  g.L = g.bx + g.by + g.bz - 2;
  g.n = pb->n_cells;
  g.halo = halo && g.boxes() > 1;
  return g;
}

template <typename T>
size_t apply_lds(const ColGrid& g) {
  const size_t rows = threads_of(g) / 4 + 1 + (g.halo ? kHaloRows : 0);
  return sizeof(T) * 8 * rows + (g.halo ? 0 : sizeof(T) * (3 * (size_t)g.L * g.C + 1));
}
size_t factor_lds(const ColGrid& g) {
  const size_t rows = threads_of(g) / 4 + 1 + (g.halo ? kHaloRows : 0);
  return sizeof(double) * 4 * 10 * rows;
}

bool fits(const ColGrid& g) {
  // (LDS for FP64, so that both precisions take the same boxes; the
  // records' and vectors' byte offsets stay below 2^31)
  return (long)g.bx * g.by * 4 <= kMaxColThreads && (!g.halo || 3 * (g.bx + g.by) <= 64) && apply_lds<double>(g) <= kMaxColLds &&
         factor_lds(g) <= kMaxColLds && (size_t)g.L * g.C * 288 < ((size_t)1 << 30) &&
         (!g.halo || (g.bx + g.by <= kHaloRows && g.nbz == 1)) && g.n < (1 << 26) &&
         g.slots() < ((size_t)1 << 31);   // (32-bit slot numbers)
}

bool lattice(const opm_problem* pb) {
  return pb->n_cells > 0 && pb->nx > 0 && pb->ny > 0 && pb->nz > 0 && pb->box_cell &&
         pb->cell_box && pb->row_ptr && pb->iperm && (long)pb->nx * pb->ny < (1 << 28) &&
         (size_t)pb->nnzb * 72 < 0xfffffe00u;   // (byte offsets into the Jacobian)
}

// The storage has a slot for every level and column of a box, with a cell or
// without: 604 bytes each (FP64, tiles; FP32 340), the position lists 1170 (670)
// per cell.  How many slots there may be, by what was measured:
constexpr size_t kFewSlots = (size_t)1 << 20;   // 0.6 GB

// The whole system by columns was faster at every share of active cells: the
// other shapes walk its levels one after another in one workgroup or by launches
// (an iteration of BiCGStab, 100 x 100 x 50 all active / 40 % / 15 % / 4 %: 1133 / 802 /
// 574 / 555 us against 2479 / 4569 / 2265 / 1003; 50 x 50 x 12, 2.7 slots per cell, 318
// against 960; 200 x 200 x 5, 3.8 slots per cell, 1244 against 5701).  32 slots per
// cell, the sparsest of these, keep the storage in proportion.
bool worth_whole(const ColGrid& g) { return g.slots() <= std::max(32 * (size_t)g.n, kFewSlots); }

// Subdomains: the position lists serve them with one workgroup each, too.
bool worth_blocks(const opm_problem* pb, const ColGrid& g, int precision) {
  // A level costs a barrier over the workgroup, so columns do not pay where the
  // widest level would need half their wavefronts: an iteration with 8 x 8 x 3
  // boxes (22 rows) 43 us against 36, 11 x 11 x 3 (31 rows) 74 against 47, 8 x 8 x 30 at
  // 12 % active (30 rows) 80 against 69; at 15 % (37 rows) 81 against 85.  Two
  // wavefronts against one: equal within 5 %.
  const int nt = threads_of(g);
  if (nt > 128 && threads_of_rows(pb->max_width) < nt) return false;
  // What is left in the 256 MB last-level cache between two sweeps (J and the
  // records, about 1 kB per cell, and the vectors) is bound by its levels, and
  // columns have the cheaper ones: 125,000 of 500,000 places active, 4.5 slots
  // per cell, 103 us against 114; 120 x 100 x 10 in 2 x 2 x 10, 4.8 slots per cell, 103
  // against 103.
  if (g.n <= (1 << 17) && g.slots() <= kFewSlots) return true;
  // Larger systems are bound by bytes, of which a place without a cell beside
  // one with a cell costs its share of a cache line: 100 x 100 x 50 in 4 x 4 columns, 70 %
  // active (1.6 slots per cell) 242 us against 243 and 250 against 259, 60 % (1.9)
  // 218 against 214, 40 % (2.8) 153 against 140; 8 x 8 columns, 70 % (2.0) 270
  // against 270 and 278 against 294, 40 % (3.5) 184 against 153; full ones, 3 x 3 x 50
  // (2.0) 334 against 331 with the factorisation 345 against 445, 8 x 8 x 10 (2.6)
  // 370 against 362, 4 x 4 x 4 (2.6) 371 against 333.  FP32 factors take half of
  // these: 40 % active 106 against 126 and 128 against 140; 4 x 4 x 4 292 against 278.
  return g.slots() <= 2 * (size_t)g.nx * g.ny * g.nz &&
         g.slots() <= (precision == OPM_PREC_MIXED ? 4 : 2) * (size_t)g.n;
}

// The box given with a block topology, as far as the host can tell it from another
// (k_cols_slots compares every row): false where the topology's counts cannot be
// those of this box, as with a field that was never set.
bool given_box(const opm_problem* pb, int& bx, int& by, int& bz) {
  bx = pb->ilu_box & 1023;
  by = (pb->ilu_box >> 10) & 1023;
  bz = (pb->ilu_box >> 20) & 1023;
  if (((unsigned)pb->ilu_box >> 30) != 0 || bx < 1 || by < 1 || bz < 1 || bx > pb->nx ||
      by > pb->ny || bz > pb->nz || !pb->lo_blk || !pb->up_blk)
    return false;
  const long cells = (long)bx * by * bz, levels = (long)bx + by + bz - 2;
  const long boxes = (((long)pb->nx + bx - 1) / bx) * (((long)pb->ny + by - 1) / by) *
                     (((long)pb->nz + bz - 1) / bz);
  if ((long)pb->n_cells == (long)pb->nx * pb->ny * pb->nz)
    return pb->n_sub == boxes && pb->n_levels == levels && pb->max_sub == cells;
  return pb->n_sub <= boxes && pb->n_levels <= levels && pb->max_sub <= cells &&
         pb->n_cells <= pb->n_sub * cells;
}

// The boxes of a problem's preconditioner; false: not by columns.
bool grid_of(const opm_problem* pb, int precision, ColGrid& g) {
  if (!lattice(pb)) return false;
  if (pb->n_sub > 1) {
    int bx, by, bz;
    if (!given_box(pb, bx, by, bz)) return false;
    g = make_grid(pb, bx, by, bz, false);
    return fits(g) && worth_blocks(pb, g, precision);
  }
  // the whole system: one box of at most 128 columns (300 cells: an
  // application 28 -> 24 us, and the updates of BiCGStab fused into it, 8
  // launches per iteration -> 5), else tiles of 8x8 columns (500k cells: an
  // application 1120 us by planes -> 386 us; factored 1900 -> 745 us)
  if ((long)pb->nx * pb->ny <= 128) {
    g = make_grid(pb, pb->nx, pb->ny, pb->nz, false);
    if (fits(g) && worth_whole(g)) return true;
  }
  g = make_grid(pb, 8, 8, pb->nz, true);
  return fits(g) && worth_whole(g);
}

template <typename T>
size_t view_bytes_of(const ColGrid& g) {
  const size_t s = g.slots();
  size_t b = al256(sizeof(T) * 36 * s) + al256(sizeof(T) * 27 * s) + al256(4 * s) +
             al256(sizeof(FacSlot) * s);
  if (g.halo) {
    const size_t nx = (size_t)g.boxes() * g.bz * g.by, ny = (size_t)g.boxes() * g.bz * g.bx;
    b += al256(sizeof(T) * 3 * s) + 2 * (al256(sizeof(T) * 3 * nx) + al256(sizeof(T) * 3 * ny)) +
         al256(72 * nx) + al256(72 * ny) + 256;
  }
  return b;
}

template <typename T>
ColView<T> view_of(const ColGrid& g, void* base) {
  ColView<T> v{};
  v.g = g;
  const size_t s = g.slots();
  char* c = (char*)base;
  auto take = [&](size_t bytes) {
    char* p = c;
    c += al256(bytes);
    return p;
  };
  v.rec_f = (T*)take(sizeof(T) * 36 * s);
  v.rec_b = (T*)take(sizeof(T) * 27 * s);
  v.idx = (int32_t*)take(4 * s);
  v.fac = (FacSlot*)take(sizeof(FacSlot) * s);
  if (g.halo) {
    const size_t nx = (size_t)g.boxes() * g.bz * g.by, ny = (size_t)g.boxes() * g.bz * g.bx;
    v.z = (T*)take(sizeof(T) * 3 * s);
    for (int q = 0; q < 2; ++q) {
      v.ex[q] = (T*)take(sizeof(T) * 3 * nx);
      v.ey[q] = (T*)take(sizeof(T) * 3 * ny);
    }
    v.eux = (double*)take(72 * nx);
    v.euy = (double*)take(72 * ny);
    v.gave_up = (int32_t*)take(256);
  }
  v.spin = (unsigned)g_plane_spin;
  return v;
}

// The column arrays follow the inverse pivots (the other shapes' arrays lie
// there too: an ILU buffer is swept by the shape that factored it).
template <typename T>
size_t pivot_bytes(const opm_problem* pb) {
  return al256((sizeof(double) + (sizeof(T) != sizeof(double) ? sizeof(T) : 0)) * 9 *
               ilu_padded(pb->n_cells));
}

template <typename T>
int factor_impl(const opm_problem* pb, const ColGrid& g, const double* J, void* ilu,
                int32_t* status, hipStream_t s) {
  const ColView<T> v = view_of<T>(g, (char*)ilu + pivot_bytes<T>(pb));
  const size_t ns = ilu_padded(pb->n_cells);
  double* d64 = (double*)ilu;
  const bool blocks = pb->n_sub > 1;
  const FacIn f{J, pb->row_ptr, pb->box_cell, pb->iperm, blocks ? pb->lo_blk : nullptr,
                blocks ? pb->up_blk : nullptr, status, d64,
                sizeof(T) == sizeof(double) ? (void*)d64 : (void*)(d64 + 9 * ns), (int)ns,
                pb->nnzb};
  if (g.halo)
    hipLaunchKernelGGL(k_cols_reset<T>, dim3(256), dim3(256), 0, s, v);
  const long slots = (long)g.slots();
  hipLaunchKernelGGL(k_cols_slots<T>, dim3(blocks_for(slots, 256)), dim3(256), 0, s, v, f);
  const size_t lds = factor_lds(g);
  const int slot = (sizeof(T) == 8 ? 0 : 5);
#define OPM_COLS_FACTOR(NT, SL)                                                              \
  do {                                                                                       \
    if (g.halo) {                                                                            \
      hipLaunchKernelGGL((k_cols_pivots<T, (NT < 512 ? NT : 256), true>), dim3(g.boxes()),   \
                         dim3(NT + kExchange), lds, s, v, f);                                \
    } else {                                                                                 \
      OPM_TRY(allow_lds(k_cols_pivots<T, NT, false>, slot + SL));                            \
      hipLaunchKernelGGL((k_cols_pivots<T, NT, false>), dim3(g.boxes()), dim3(NT), lds, s, v, \
                         f);                                                                 \
    }                                                                                        \
  } while (0)
  switch (threads_of(g)) {
    case 64: OPM_COLS_FACTOR(64, 0); break;
    case 128: OPM_COLS_FACTOR(128, 1); break;
    case 256: OPM_COLS_FACTOR(256, 2); break;
    default: OPM_COLS_FACTOR(512, 3); break;
  }
#undef OPM_COLS_FACTOR
  hipLaunchKernelGGL(k_cols_records<T>, dim3(blocks_for(slots, 64)), dim3(256), 0, s, v, f);
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

template <typename T, int MODE>
int apply_impl(const opm_problem* pb, const ColGrid& g, void* ilu, const double* r, double* x,
               const int32_t* skip, const kry::Fused& f, hipStream_t s) {
  const ColView<T> v = view_of<T>(g, (char*)ilu + pivot_bytes<T>(pb));
  const size_t lds = apply_lds<T>(g);
  const int slot = 10 + (sizeof(T) == 8 ? 0 : 15) + 5 * MODE;
  const int32_t* skip2 = MODE == kry::kFuseNone ? skip : &f.sc->state;
#define OPM_COLS(NT, D, SL)                                                                  \
  do {                                                                                       \
    if (g.halo) {                                                                            \
      /* (forward FP64: with three levels in flight the fused forms spill) */                \
      constexpr int NTT = NT < 512 ? NT : 256, DF = sizeof(T) == 8 ? 2 : 3;                  \
      hipLaunchKernelGGL((k_cols_tiles<T, NTT, DF, true, MODE>), dim3(g.boxes()),            \
                         dim3(NT + kExchange), lds, s, v, r, x, skip, f);                    \
      hipLaunchKernelGGL((k_cols_tiles<T, NTT, 3, false, kry::kFuseNone>), dim3(g.boxes()),  \
                         dim3(NT + kExchange), lds, s, v, r, x, skip2, f);                   \
    } else {                                                                                 \
      OPM_TRY(allow_lds(k_cols_apply<T, NT, D, MODE>, slot + SL));                           \
      hipLaunchKernelGGL((k_cols_apply<T, NT, D, MODE>), dim3(g.boxes()), dim3(NT), lds, s,  \
                         v, r, x, skip, f);                                                  \
    }                                                                                        \
  } while (0)
  switch (threads_of(g)) {
    case 64: OPM_COLS(64, 3, 0); break;
    case 128: OPM_COLS(128, 3, 1); break;
    case 256: OPM_COLS(256, 3, 2); break;
    default: OPM_COLS(512, 3, 3); break;
  }
#undef OPM_COLS
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

}  // namespace

// The preconditioner of pb is factored and applied by columns.
bool cols_capable(const opm_problem* pb, int precision) {
  ColGrid g;
  return grid_of(pb, precision, g);
}

// Workgroups of a sweep (the partial sums of a fused one).
int cols_boxes(const opm_problem* pb, int precision) {
  ColGrid g;
  return grid_of(pb, precision, g) ? g.boxes() : 0;
}

size_t cols_bytes(const opm_problem* pb, int precision) {
  ColGrid g;
  if (!grid_of(pb, precision, g)) return 0;
  return precision == OPM_PREC_MIXED ? pivot_bytes<float>(pb) + view_bytes_of<float>(g)
                                     : pivot_bytes<double>(pb) + view_bytes_of<double>(g);
}

int cols_factor(const opm_problem* pb, const double* J, void* ilu, int precision,
                int32_t* status, hipStream_t s) {
  ColGrid g;
  if (!grid_of(pb, precision, g)) return OPM_EINVAL;
  return precision == OPM_PREC_MIXED ? factor_impl<float>(pb, g, J, ilu, status, s)
                                     : factor_impl<double>(pb, g, J, ilu, status, s);
}

// mode: kry::FusedMode; skip (may be null, mode kFuseNone only): the sweeps
// return at once while *skip != 0.
int cols_apply(const opm_problem* pb, void* ilu, int precision, int mode, const double* r,
               double* x, const int32_t* skip, const kry::Fused& f, hipStream_t s) {
  ColGrid g;
  if (!grid_of(pb, precision, g)) return OPM_EINVAL;
  if (precision == OPM_PREC_MIXED) {
    switch (mode) {
      case kry::kFuseBegin: return apply_impl<float, kry::kFuseBegin>(pb, g, ilu, r, x, skip, f, s);
      case kry::kFuseS: return apply_impl<float, kry::kFuseS>(pb, g, ilu, r, x, skip, f, s);
      default: return apply_impl<float, kry::kFuseNone>(pb, g, ilu, r, x, skip, f, s);
    }
  }
  switch (mode) {
    case kry::kFuseBegin: return apply_impl<double, kry::kFuseBegin>(pb, g, ilu, r, x, skip, f, s);
    case kry::kFuseS: return apply_impl<double, kry::kFuseS>(pb, g, ilu, r, x, skip, f, s);
    default: return apply_impl<double, kry::kFuseNone>(pb, g, ilu, r, x, skip, f, s);
  }
}

}  // namespace opm
