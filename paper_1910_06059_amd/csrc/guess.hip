// Learned Newton initial guess: a three-layer 3-D convolutional network
// (3x3x3 kernels, 16 channels, zero padding, ReLU after layers 1 and 2) maps
// the last two states, the log-permeability and the well terms of each cell
// to a predicted state change over one report step: the last change
// y_n - y_{n-1} (a skip connection, linear extrapolation) plus the network's
// correction of the saturations away from wells (the pressure keeps the
// extrapolation: an error of a few psi in the slightly compressible system
// raises the CNV far above the extrapolation's).  The paper always starts
// Newton from the previous state (sec. 2.3); here the prediction replaces
// that start only when its CNV is lower, and the convergence test is left
// as it is, so converged states do not depend on the network.
//
// Convolutions are implicit GEMMs on the BF16 matrix cores of gfx950
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation) over 16x4x4 tiles of the box
// staged in LDS: 16 cells along x by 16 output channels accumulate 14 products
// of 16x16x32, each reducing over the 16 input channels of two taps.
// Activations and their gradients are stored channels-last in BF16
// ([box cell][16], rounded to nearest even); weights exist as an FP32 master
// copy (updated by Adam) and as BF16 operand copies in the two layouts that
// the forward and backward-data products read.
#include <cmath>

#include "common.h"

namespace opm {

// y_guess = learned guess; if y_extrap is given it receives a pointer into
// the workspace holding the extrapolation alone (valid until the next call).
int guess_infer(const opm_problem* pb, const opm_guess_net* net, const double* y_n,
                const double* y_nm1, double* y_guess, void* work, hipStream_t s,
                const double** y_extrap = nullptr);
size_t guess_work_bytes(const opm_problem* pb, const opm_guess_net* net);

namespace {

constexpr int kCh = OPM_GUESS_CHANNELS;
constexpr int kTaps = 27;
constexpr int kLayerW = kTaps * kCh * kCh;        // W[27][cout][cin]
constexpr int kLayerParams = kLayerW + kCh;       // + bias[cout]
constexpr int kParams = 3 * kLayerParams;
constexpr int kTX = 16, kTY = 4, kTZ = 4;         // cells of a convolution tile
constexpr int kConvWgs = 768;                     // workgroups of a convolution
constexpr int kGradWgs = 512;                     // workgroups of the weight gradient
constexpr int kReduceGroup = 32;                  // workgroups per stage-1 sum of the partials
static_assert(kParams == OPM_GUESS_PARAMS, "parameter count");

typedef short short8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// v_mfma_f32_16x16x32_bf16 (gfx950): D[16][16] += A[16][32] B[32][16] in
// FP32; lane l holds A[l % 16][k] and B[k][l % 16] for the eight k of lane
// group l / 16, and D[4 (l / 16) + r][l % 16].  A product sums over k, so
// any assignment of the (tap, channel) or cell pairs to k that A and B
// share gives the same sum.
__device__ __forceinline__ floatx4 mfma32(const short8& a, const short8& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ unsigned short f2bf(float f) {   // round to nearest even
  unsigned u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);   // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) {
  return __uint_as_float(((unsigned)h) << 16);
}

struct Grid {
  int nx, ny, nz, nbox;
};

inline int tiles_of(const Grid& g) { return (g.nbox + 15) / 16; }
inline size_t al(size_t b) { return (b + 255) / 256 * 256; }
inline size_t act_bytes(const Grid& g) { return al(sizeof(unsigned short) * (size_t)tiles_of(g) * 16 * kCh); }
__host__ __device__ inline int ctiles_x(const Grid& g) { return (g.nx + kTX - 1) / kTX; }
__host__ __device__ inline int ctiles_y(const Grid& g) { return (g.ny + kTY - 1) / kTY; }
inline int ctiles_of(const Grid& g) {
  return ctiles_x(g) * ctiles_y(g) * ((g.nz + kTZ - 1) / kTZ);
}
inline int grad_wgs(const Grid& g) { return ctiles_of(g) < kGradWgs ? ctiles_of(g) : kGradWgs; }
inline int groups_of(const Grid& g) { return (grad_wgs(g) + kReduceGroup - 1) / kReduceGroup; }
// per-workgroup partials, then the stage-1 sums of groups of them
inline size_t partial_bytes(const Grid& g) {
  return al(sizeof(float) * (size_t)grad_wgs(g) * kLayerParams) +
         al(sizeof(float) * (size_t)groups_of(g) * kLayerParams);
}

// -------------------------------------------------------------- features
// Channel scales: pressures as (p - 4800 psi) / 1000 psi, saturations as
// they are, log10(k_h / 1 mD) - 2, injection rates per 10 m^3/day, the
// producer term log(1 + WI (p - p_bhp)^+ / 1 cP per 10 m^3/day).  Outputs:
// dp per 100 psi, ds_w and ds_g per 0.1 (comparable magnitudes in the loss).
constexpr double kPsi = 6894.757293168;
constexpr double kP0 = 4800.0 * kPsi;
constexpr double kPS = 1000.0 * kPsi;
constexpr double kQS = 86400.0 / 10.0;
constexpr double kMuRef = 1e-3;
constexpr double kDPS = 100.0 * kPsi;
constexpr double kDSS = 0.1;
constexpr double kMilliDarcy = 9.869233e-16;

// channels: 0-2 y_n, 3-5 the last change y_n - y_{n-1} (per 100 psi and
// per 0.1, so BF16 keeps it to 3 digits), 6 log-permeability, 7-9 injection
// of water, oil, gas, 10 producer term, 11-15 zero.  Inactive box cells stay 0.
// near (may be null; zero on entry): marks the cells near a well: a cell and
// its 26 box neighbours where it carries a non-zero well channel (7-10, as
// stored; +0 and -0 both count as zero).  The learned correction is neither
// trained nor applied there.
__global__ __launch_bounds__(kBlock) void k_features(Grid g, opm_problem pb,
                                                      const int32_t* cell_box, const double* yn,
                                                      const double* ynm1, const double* perm,
                                                      unsigned short* feats, unsigned char* near) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= pb.n_cells) return;
  float f[kCh];
#pragma unroll
  for (int k = 0; k < kCh; ++k) f[k] = 0.f;
  const double p = yn[3 * c];
  f[0] = (float)((p - kP0) / kPS);
  f[1] = (float)yn[3 * c + 1];
  f[2] = (float)yn[3 * c + 2];
  f[3] = (float)((p - ynm1[3 * c]) / kDPS);
  f[4] = (float)((yn[3 * c + 1] - ynm1[3 * c + 1]) / kDSS);
  f[5] = (float)((yn[3 * c + 2] - ynm1[3 * c + 2]) / kDSS);
  f[6] = (float)(log10(perm[c] / kMilliDarcy) - 2.0);
  const int t0 = pb.cell_conn_ptr[c], t1 = pb.cell_conn_ptr[c + 1];
  if (t0 < t1) {
    double inj[3] = {0.0, 0.0, 0.0}, prod = 0.0;
    for (int t = t0; t < t1; ++t) {
      const int k = pb.cell_conn[t];
      if (pb.conn_kind[k] == OPM_WELL_RATE_INJ) {
        const int ph = pb.conn_phase[k];
#pragma unroll
        for (int a = 0; a < 3; ++a)   // conn_rate is an outflux: negative for injection
          if (a == ph) inj[a] -= pb.conn_rate[k];
      } else {
        const double dd = p - pb.conn_bhp[k];
        if (dd > 0.0) prod += pb.conn_wi[k] * dd;
      }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) f[7 + a] = (float)(inj[a] * kQS);
    f[10] = (float)log1p(prod / kMuRef * kQS);
  }
  const int b = cell_box[c];
  short8 o[2];
#pragma unroll
  for (int k = 0; k < kCh; ++k) o[k / 8][k % 8] = (short)f2bf(f[k]);
  short8* out = reinterpret_cast<short8*>(feats + (size_t)b * kCh);
  out[0] = o[0];
  out[1] = o[1];
  if (near && t0 < t1 && ((o[0][7] | o[1][0] | o[1][1] | o[1][2]) & 0x7fff)) {
    const int i = b % g.nx, j = (b / g.nx) % g.ny, k = b / (g.nx * g.ny);
    for (int dz = -1; dz <= 1; ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const int ii = i + dx, jj = j + dy, kk = k + dz;
          if (ii >= 0 && ii < g.nx && jj >= 0 && jj < g.ny && kk >= 0 && kk < g.nz)
            near[ii + g.nx * (jj + g.ny * kk)] = 1;
        }
  }
}

__global__ __launch_bounds__(kBlock) void k_zero_bytes(uint4* p, size_t count) {
  for (size_t k = blockIdx.x * (size_t)kBlock + threadIdx.x; k < count;
       k += (size_t)gridDim.x * kBlock)
    p[k] = uint4{0, 0, 0, 0};
}

// ---------------------------------------------------- convolution (MFMA)
// Tap t covers the offset (t % 3 - 1, t / 3 % 3 - 1, t / 9 - 1) in (x, y, z).
//
// A workgroup owns a tile of 16x4x4 box cells, staged in LDS with its one-cell
// halo (18x6x6 cells, zero outside the box), so that each input is read from
// memory about 2.5 times (by neighbouring tiles) instead of 27, and each
// wavefront keeps the 14 operand pairs of the weights in registers for the four
// rows of its z-slab.  One product per pair of taps: A rows are the 16 cells of
// a row, A columns the 16 input channels of the cell at each of the two tap
// offsets (mirrored when FLIP); B the two taps' weights wt[t] as [n][k] rows of
// 16.  Lane group kb takes tap t + kb / 2 and channels 8 (kb % 2) .. + 7 in both
// operands; the 27th tap pairs with zeros.  kConvWgs workgroups (three per
// compute unit) go through the tiles with the next one's loads in flight, so
// that the weights are loaded three times per unit and not once per tile.  Per
// layer of 500k cells 41.7 us (16 cells per wavefront, every neighbour read from
// memory) -> 24.6 us staged -> 20.6 us with the weights kept; the bytes alone
// take 7 us.  The gradient form reads one more box, the layer inputs that mask
// its result; asked for ahead of the products: 28.2 -> 22.7 us.
constexpr int kHX = kTX + 2, kHY = kTY + 2, kHZ = kTZ + 2;   // a tile with its halo
enum ConvOut : int { kOutRelu, kOutAll, kOutThree, kOutGrad };

struct ConvTile {
  int x0, y0, z0;
  __device__ __forceinline__ ConvTile(const Grid& g, int t) {
    const int tx = ctiles_x(g), ty = ctiles_y(g);
    x0 = t % tx * kTX;
    y0 = t / tx % ty * kTY;
    z0 = t / (tx * ty) * kTZ;
  }
};

// OUT kOutRelu: out_bf = BF16 of ReLU(conv(in) + bias); kOutAll: out_f = the
// sum itself, [cell][16]; kOutThree: its first three channels, [cell][4];
// kOutGrad: out_bf = conv^T(in) where the layer input act_in is positive.
template <int OUT>
__global__ __launch_bounds__(256) void k_conv(Grid g, const unsigned short* in,
                                              const unsigned short* wt, const float* bias,
                                              const unsigned short* act_in,
                                              unsigned short* out_bf, float* out_f, int ntiles) {
  constexpr bool FLIP = OUT == kOutGrad;
  __shared__ __attribute__((aligned(16))) unsigned short tile[kHX * kHY * kHZ * kCh];
  constexpr int kChunks = kHX * kHY * kHZ * 2, kU = (kChunks + 255) / 256;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int m = lane & 15, kb = lane >> 4;
  const int half = kb >> 1, c8 = (kb & 1) * 8;
  constexpr int kPairs = (kTaps + 1) / 2;
  short8 b[kPairs];
  int at[kPairs];   // this lane's A operand of the first row
#pragma unroll
  for (int p = 0; p < kPairs; ++p) {
    const int t = 2 * p + half, tc = t < kTaps ? t : kTaps - 1;
    b[p] = *reinterpret_cast<const short8*>(wt + (tc * kCh + m) * kCh + c8);
    if (t >= kTaps) b[p] = short8{0, 0, 0, 0, 0, 0, 0, 0};
    int dx = tc % 3 - 1, dy = (tc / 3) % 3 - 1, dz = tc / 9 - 1;
    if (FLIP) {
      dx = -dx;
      dy = -dy;
      dz = -dz;
    }
    at[p] = (((w + 1 + dz) * kHY + 1 + dy) * kHX + m + 1 + dx) * kCh + c8;
  }
  const float bs = OUT == kOutGrad ? 0.f : bias[m];
  // a tile's loads, all in flight together
  short8 stage[kU];
  auto fetch = [&](int t) {
    const ConvTile ct(g, t);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int q = u * 256 + threadIdx.x, cell = q >> 1;
      const int x = ct.x0 + cell % kHX - 1, y = ct.y0 + cell / kHX % kHY - 1,
                z = ct.z0 + cell / (kHX * kHY) - 1;
      stage[u] = short8{0, 0, 0, 0, 0, 0, 0, 0};
      if (q < kChunks && x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz)
        stage[u] = *reinterpret_cast<const short8*>(
            in + (unsigned)(x + g.nx * (y + g.ny * z)) * kCh + (q & 1) * 8);
    }
  };
  if ((int)blockIdx.x < ntiles) fetch(blockIdx.x);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const ConvTile ct(g, t);
    __syncthreads();   // the previous tile has been read
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int q = u * 256 + threadIdx.x;
      if (q < kChunks) *reinterpret_cast<short8*>(tile + q * 8) = stage[u];
    }
    __syncthreads();
    if (t + (int)gridDim.x < ntiles) fetch(t + gridDim.x);
    const int z = ct.z0 + w;
    if (z >= g.nz) continue;   // whole wavefront: MFMA needs all lanes
    // the layer inputs that mask the gradient, ahead of the products (clamped)
    unsigned short av[kTY][4];
    if (OUT == kOutGrad)
#pragma unroll
      for (int ly = 0; ly < kTY; ++ly)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int x = min(ct.x0 + 4 * kb + r, g.nx - 1), y = min(ct.y0 + ly, g.ny - 1);
          av[ly][r] = act_in[(size_t)(x + g.nx * (y + g.ny * z)) * kCh + m];
        }
#pragma unroll
    for (int ly = 0; ly < kTY; ++ly) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kPairs; ++p) {
        short8 a = *reinterpret_cast<const short8*>(tile + at[p] + ly * kHX * kCh);
        // (the last pair's second tap: zeros, also against a non-finite input)
        if (p == kPairs - 1 && half) a = short8{0, 0, 0, 0, 0, 0, 0, 0};
        acc = mfma32(a, b[p], acc);
      }
      const int y = ct.y0 + ly;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = ct.x0 + 4 * kb + r;
        if (x >= g.nx || y >= g.ny) continue;
        const size_t cell = (size_t)(x + g.nx * (y + g.ny * z));
        const float v = acc[r] + bs;
        if (OUT == kOutRelu) out_bf[cell * kCh + m] = f2bf(v > 0.f ? v : 0.f);
        if (OUT == kOutAll) out_f[cell * kCh + m] = v;
        if (OUT == kOutThree && m < 4) out_f[cell * 4 + m] = v;
        if (OUT == kOutGrad)
          out_bf[cell * kCh + m] = f2bf(bf2f(av[ly][r]) > 0.f ? acc[r] : 0.f);
      }
    }
  }
}

// Weight-gradient partials of one workgroup over its tiles:
// dW[t][cout][cin] = sum_cells in[cell + off_t][cin] d_out[cell][cout] as
// 16x16x32 products whose reduction runs over 32 cells, two rows of 16 (A =
// in^T with rows cin, B = d_out with columns cout; lane group kb takes cells
// 8 (kb % 2) .. + 7 of row kb / 2 in both operands); bias[cout] = sum_cells
// d_out[cell][cout].  Both operands need eight consecutive cells of one
// channel, so the tile is staged channel by channel (pairs of cells as 4-byte
// words): a lane reads the twelve cells x - 2 .. x + 9 of a row once and shifts
// them by a cell for dx = -1 and + 1.  Each of the three wavefronts takes one
// dz (nine taps, 36 accumulators).  A layer of 500k cells: 424 us (operands
// gathered two bytes at a time from memory) -> 27.7 us.
constexpr int kGX = kTX + 4;                        // cells of a staged row, x - 2 .. x + 17
constexpr int kInCh = kHY * kHZ * kGX + 4;          // values of a channel (padded against
constexpr int kDoCh = kTY * kTZ * kTX + 8;          //   bank conflicts between channels)
__global__ __launch_bounds__(192) void k_conv_wgrad(Grid g, const unsigned short* in,
                                                    const unsigned short* dout, int ntiles,
                                                    float* partials) {
  __shared__ __attribute__((aligned(16))) unsigned short ti[kCh * kInCh];
  __shared__ __attribute__((aligned(16))) unsigned short td[kCh * kDoCh];
  const int tid = threadIdx.x, lane = tid & 63, dzi = tid >> 6;
  const int m = lane & 15, kb = lane >> 4;
  floatx4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  auto fetch = [&](const unsigned short* src, int x, int y, int z, int h) {
    short8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if (x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz)
      v = *reinterpret_cast<const short8*>(src + (unsigned)(x + g.nx * (y + g.ny * z)) * kCh +
                                           h * 8);
    return v;
  };
  // two cells' eight channels, as one word per channel
  auto put = [](unsigned short* dst, int stride, const short8& lo, const short8& hi) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      *reinterpret_cast<unsigned*>(dst + e * stride) =
          (unsigned)(unsigned short)lo[e] | (unsigned)(unsigned short)hi[e] << 16;
  };
  constexpr int kInTasks = kHY * kHZ * (kGX / 2) * 2, kDoTasks = kTY * kTZ * (kTX / 2) * 2;
  constexpr int kInU = (kInTasks + 191) / 192, kDoU = (kDoTasks + 191) / 192;
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const ConvTile ct(g, t);
    short8 lo[kInU + kDoU], hi[kInU + kDoU];
#pragma unroll
    for (int u = 0; u < kInU; ++u) {
      const int q = u * 192 + tid, h = q & 1, pr = (q >> 1) % (kGX / 2), row = (q >> 1) / (kGX / 2);
      const int x = ct.x0 + 2 * pr - 2, y = ct.y0 + row % kHY - 1,
                z = q < kInTasks ? ct.z0 + row / kHY - 1 : -1;
      lo[u] = fetch(in, x, y, z, h);
      hi[u] = fetch(in, x + 1, y, z, h);
    }
#pragma unroll
    for (int u = 0; u < kDoU; ++u) {
      const int q = u * 192 + tid, h = q & 1, pr = (q >> 1) % (kTX / 2), row = (q >> 1) / (kTX / 2);
      const int x = ct.x0 + 2 * pr, y = ct.y0 + row % kTY, z = q < kDoTasks ? ct.z0 + row / kTY : -1;
      lo[kInU + u] = fetch(dout, x, y, z, h);
      hi[kInU + u] = fetch(dout, x + 1, y, z, h);
    }
    __syncthreads();   // the previous tile's products have been formed
#pragma unroll
    for (int u = 0; u < kInU; ++u) {
      const int q = u * 192 + tid, h = q & 1, pr = (q >> 1) % (kGX / 2), row = (q >> 1) / (kGX / 2);
      if (q < kInTasks) put(ti + 8 * h * kInCh + row * kGX + 2 * pr, kInCh, lo[u], hi[u]);
    }
#pragma unroll
    for (int u = 0; u < kDoU; ++u) {
      const int q = u * 192 + tid, h = q & 1, pr = (q >> 1) % (kTX / 2), row = (q >> 1) / (kTX / 2);
      if (q < kDoTasks)
        put(td + 8 * h * kDoCh + row * kTX + 2 * pr, kDoCh, lo[kInU + u], hi[kInU + u]);
    }
    __syncthreads();
    const bool partial = ct.x0 + kTX > g.nx || ct.y0 + kTY > g.ny || ct.z0 + kTZ > g.nz;
    // rows (z, y) and (z, y + 1) of the tile per product
#pragma unroll 2
    for (int kq = 0; kq < kTZ * kTY / 2; ++kq) {
      const int row = 2 * kq + (kb >> 1), ly = row % kTY, lz = row / kTY, x0 = 8 * (kb & 1);
      const short8 b = *reinterpret_cast<const short8*>(td + m * kDoCh + row * kTX + x0);
      u32x4 mask = {0, 0, 0, 0};
      if (partial && ct.y0 + ly < g.ny && ct.z0 + lz < g.nz) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (ct.x0 + x0 + e < g.nx) mask[e / 2] |= 0xffffu << (16 * (e % 2));
      }
      if (dzi == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bsum += bf2f((unsigned short)b[e]);
      }
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        const uint2* src = reinterpret_cast<const uint2*>(
            ti + m * kInCh + ((lz + dzi) * kHY + ly + dy) * kGX + x0);
        unsigned d[6];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const uint2 v = src[e];
          d[2 * e] = v.x;
          d[2 * e + 1] = v.y;
        }
        u32x4 am, ap;
#pragma unroll
        for (int e = 0; e < 4; ++e) {   // cells x - 1 .. x + 6 and x + 1 .. x + 8
          am[e] = __builtin_amdgcn_alignbyte(d[e + 1], d[e], 2);
          ap[e] = __builtin_amdgcn_alignbyte(d[e + 2], d[e + 1], 2);
        }
        u32x4 a0 = {d[1], d[2], d[3], d[4]};
        if (partial) {   // cells outside the box: no product, also of a non-finite input
          am &= mask;
          a0 &= mask;
          ap &= mask;
        }
        acc[3 * dy] = mfma32(__builtin_bit_cast(short8, am), b, acc[3 * dy]);
        acc[3 * dy + 1] = mfma32(__builtin_bit_cast(short8, a0), b, acc[3 * dy + 1]);
        acc[3 * dy + 2] = mfma32(__builtin_bit_cast(short8, ap), b, acc[3 * dy + 2]);
      }
    }
  }
  float* P = partials + (size_t)blockIdx.x * kLayerParams;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) P[((9 * dzi + t) * kCh + m) * kCh + 4 * kb + r] = acc[t][r];
  // lanes m, m+16, m+32, m+48 hold the four cell groups of channel m
  bsum += __shfl_xor(bsum, 16, 64);
  bsum += __shfl_xor(bsum, 32, 64);
  if (dzi == 0 && kb == 0) P[kLayerW + m] = bsum;
}

// Sum of the per-workgroup partials in two fixed-order stages: stage 1 adds
// groups of kReduceGroup workgroups (grid: parameter blocks x groups), stage 2
// adds the groups (deterministic).

__global__ __launch_bounds__(256) void k_reduce_stage1(const float* partials, int nwaves,
                                                       float* stage) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= kLayerParams) return;
  const int w0 = blockIdx.y * kReduceGroup, w1 = min(w0 + kReduceGroup, nwaves);
  float s = 0.f;
#pragma unroll 8
  for (int w = w0; w < w1; ++w) s += partials[(size_t)w * kLayerParams + e];
  stage[(size_t)blockIdx.y * kLayerParams + e] = s;
}

__global__ __launch_bounds__(256) void k_reduce_partials(const float* stage, int ngroups,
                                                         float* grad) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= kLayerParams) return;
  float s = 0.f;
#pragma unroll 8
  for (int gr = 0; gr < ngroups; ++gr) s += stage[(size_t)gr * kLayerParams + e];
  grad[e] = s;
}

// -------------------------------------------------------------- training
// Squared error of the two saturation outputs against the scaled correction
// of the step to the extrapolated one, (y_next - y_n) - (y_n - y_{n-1})
// (ds / 0.1), summed over active cells away from wells and divided by
// 2 n_cells; d_out = dL/d out in BF16 (channels 1-2; channel 0, the unused
// pressure output, and cells near wells get zero).
// out: [box cell][4] (k_conv's kOutThree); d_out rows are written whole.
__global__ __launch_bounds__(kBlock) void k_loss(int n, const int32_t* cell_box,
                                                 const unsigned char* near, const float* out,
                                                 const double* yn, const double* ynm1,
                                                 const double* ynext, unsigned short* dout,
                                                 double* partials) {
  __shared__ double sh[kBlock / kWave];
  const int c = blockIdx.x * kBlock + threadIdx.x;
  double se = 0.0;
  if (c < n) {
    const size_t b = (size_t)cell_box[c];
    const float4 o = reinterpret_cast<const float4*>(out)[b];
    short8 d = {0, 0, 0, 0, 0, 0, 0, 0};   // (channel 0: neither trained nor used)
    if (!near[b]) {
      const float ov[3] = {o.x, o.y, o.z};
#pragma unroll
      for (int k = 1; k < 3; ++k) {
        const double tgt =
            ((ynext[3 * c + k] - yn[3 * c + k]) - (yn[3 * c + k] - ynm1[3 * c + k])) / kDSS;
        const double e = (double)ov[k] - tgt;
        se += e * e;
        d[k] = (short)f2bf((float)(2.0 * e / (2.0 * n)));
      }
    }
    short8* dst = reinterpret_cast<short8*>(dout + b * kCh);
    dst[0] = d;
    dst[1] = short8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  const double s = block_sum<kBlock>(se, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ __launch_bounds__(kBlock) void k_loss_final(const double* partials, int nblk, int n,
                                                       double* loss) {
  __shared__ double sh[kBlock / kWave];
  double v = 0.0;
  for (int k = threadIdx.x; k < nblk; k += kBlock) v += partials[k];
  v = block_sum<kBlock>(v, sh);
  if (threadIdx.x == 0) *loss = v / (2.0 * n);
}

// Adam (Kingma and Ba) on the FP32 master parameters; step is 1-based.
__global__ __launch_bounds__(256) void k_adam(float* w, const float* grad, float* m1, float* m2,
                                              int count, float lr, float b1, float b2, float eps,
                                              int step) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= count) return;
  const float gr = grad[e];
  const float a = b1 * m1[e] + (1.f - b1) * gr;
  const float b = b2 * m2[e] + (1.f - b2) * gr * gr;
  m1[e] = a;
  m2[e] = b;
  const float ah = a / (1.f - powf(b1, (float)step));
  const float bh = b / (1.f - powf(b2, (float)step));
  w[e] -= lr * ah / (sqrtf(bh) + eps);
}

// BF16 operand copies of the master weights: forward wf[l][t][cout][cin],
// backward-data wb[l][t][cin][cout].
__global__ __launch_bounds__(256) void k_pack_weights(const float* master, unsigned short* wf,
                                                      unsigned short* wb) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= 3 * kLayerW) return;
  const int layer = e / kLayerW, r = e % kLayerW;
  const int t = r / (kCh * kCh), co = (r / kCh) % kCh, ci = r % kCh;
  const unsigned short v = f2bf(master[(size_t)layer * kLayerParams + r]);
  wf[(size_t)layer * kLayerW + r] = v;
  wb[(size_t)layer * kLayerW + (t * kCh + ci) * kCh + co] = v;
}

// y_guess = y_n + (y_n - y_{n-1}) + the correction of the two saturations
// (the skip connection is applied in FP64; the pressure keeps the
// extrapolation, output 0 is unused); the correction is used only away from
// wells and only if all three outputs are finite, and not at all when out is
// null (the extrapolation alone); saturations clamped to [0, 1] with
// s_w + s_g <= 1 (s_g reduced first).
__global__ __launch_bounds__(kBlock) void k_guess_apply(int n, const int32_t* cell_box,
                                                        const unsigned char* near,
                                                        const double* yn, const double* ynm1,
                                                        const float* out, double* yg) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n) return;
  const size_t b = (size_t)cell_box[c];
  float o0 = 0.f, o1 = 0.f, o2 = 0.f;
  bool ok = false;
  if (out) {
    const float4 o = reinterpret_cast<const float4*>(out)[b];
    o0 = o.x;
    o1 = o.y;
    o2 = o.z;
    ok = isfinite(o0) && isfinite(o1) && isfinite(o2) && !near[b];
  }
  const double p = yn[3 * c] + (yn[3 * c] - ynm1[3 * c]);
  double sw = yn[3 * c + 1] + (yn[3 * c + 1] - ynm1[3 * c + 1]) + (ok ? kDSS * (double)o1 : 0.0);
  double sg = yn[3 * c + 2] + (yn[3 * c + 2] - ynm1[3 * c + 2]) + (ok ? kDSS * (double)o2 : 0.0);
  sw = fmin(fmax(sw, 0.0), 1.0);
  sg = fmin(fmax(sg, 0.0), 1.0);
  if (sw + sg > 1.0) sg = 1.0 - sw;
  yg[3 * c] = p;
  yg[3 * c + 1] = sw;
  yg[3 * c + 2] = sg;
}

// ------------------------------------------------------------ host side
bool valid_grid(int nx, int ny, int nz) {
  return nx > 0 && ny > 0 && nz > 0 && (long)nx * ny * nz * kCh < (1L << 31);
}

template <int OUT>
void conv_launch(const Grid& g, const unsigned short* in, const unsigned short* wt,
                 const float* bias, const unsigned short* act_in, unsigned short* out_bf,
                 float* out_f, hipStream_t s) {
  const int nt = ctiles_of(g);
  hipLaunchKernelGGL(k_conv<OUT>, dim3(nt < kConvWgs ? nt : kConvWgs), dim3(256), 0, s, g, in, wt,
                     bias, act_in, out_bf, out_f, nt);
}

void backward_launch(const Grid& g, const unsigned short* in, const unsigned short* dout,
                     const unsigned short* wb, const unsigned short* act_in, unsigned short* din,
                     float* grad, float* partials, hipStream_t s) {
  const int nw = grad_wgs(g), ng = groups_of(g);
  float* stage = partials + al(sizeof(float) * (size_t)nw * kLayerParams) / sizeof(float);
  hipLaunchKernelGGL(k_conv_wgrad, dim3(nw), dim3(192), 0, s, g, in, dout, ctiles_of(g),
                     partials);
  hipLaunchKernelGGL(k_reduce_stage1, dim3((kLayerParams + 255) / 256, ng), dim3(256), 0, s,
                     partials, nw, stage);
  hipLaunchKernelGGL(k_reduce_partials, dim3((kLayerParams + 255) / 256), dim3(256), 0, s, stage,
                     ng, grad);
  if (din) conv_launch<kOutGrad>(g, dout, wb, nullptr, act_in, din, nullptr, s);
}

// Zero the rows of a box buffer that no active cell writes: all of them where
// the box has inactive cells, else the rows past its end.
void zero_unwritten(const Grid& g, int n, unsigned short* rows, hipStream_t s) {
  const size_t total = (size_t)tiles_of(g) * 16, first = n < g.nbox ? 0 : (size_t)g.nbox;
  if (first == total) return;
  const size_t words = (total - first) * kCh * sizeof(unsigned short) / sizeof(uint4);
  hipLaunchKernelGGL(k_zero_bytes, dim3((unsigned)(words < 256 * kBlock ? blocks_for((long)words, kBlock) : 256)),
                     dim3(kBlock), 0, s, reinterpret_cast<uint4*>(rows + first * kCh), words);
}

// Workspace of infer / train: activations a0 (features), a1, a2, output,
// gradients d3, d2, d1, weight partials, gradient, loss partials, guess.
struct Bufs {
  unsigned short *a0, *a1, *a2, *d3, *d2, *d1;
  float* out;
  float* partials;
  float* grad;
  double* lpart;
  double* yg;
  unsigned char* near;   // [box] cells near a well
};

size_t bufs_bytes(const Grid& g, int n) {
  return 6 * act_bytes(g) + al(sizeof(float) * 4 * (size_t)g.nbox) + al((size_t)g.nbox) +
         partial_bytes(g) + al(sizeof(float) * kParams) +
         al(sizeof(double) * (blocks_for(n, kBlock) + 1)) + al(sizeof(double) * 3 * (size_t)n);
}

Bufs carve(const Grid& g, int n, void* work) {
  char* c = (char*)work;
  Bufs b;
  unsigned short** acts[6] = {&b.a0, &b.a1, &b.a2, &b.d3, &b.d2, &b.d1};
  for (auto* p : acts) {
    *p = (unsigned short*)c;
    c += act_bytes(g);
  }
  b.out = (float*)c;
  c += al(sizeof(float) * 4 * (size_t)g.nbox);
  b.near = (unsigned char*)c;
  c += al((size_t)g.nbox);
  b.partials = (float*)c;
  c += partial_bytes(g);
  b.grad = (float*)c;
  c += al(sizeof(float) * kParams);
  b.lpart = (double*)c;
  c += al(sizeof(double) * (blocks_for(n, kBlock) + 1));
  b.yg = (double*)c;
  return b;
}

bool valid_net(const opm_problem* pb, const opm_guess_net* net) {
  return pb && net && pb->n_cells > 0 && valid_grid(net->nx, net->ny, net->nz) &&
         pb->n_cells <= net->nx * net->ny * net->nz && net->cell_box && net->perm_h &&
         net->master && net->wbf16 && pb->cell_conn_ptr &&
         (pb->n_conns == 0 || (pb->cell_conn && pb->conn_kind && pb->conn_phase &&
                               pb->conn_wi && pb->conn_rate && pb->conn_bhp));
}

// near (may be null): the cells near a well
int features(const opm_problem* pb, const opm_guess_net* net, const Grid& g, const double* yn,
             const double* ynm1, unsigned short* a0, unsigned char* near, hipStream_t s) {
  zero_unwritten(g, pb->n_cells, a0, s);
  if (near) {
    const size_t words = al((size_t)g.nbox) / sizeof(uint4);
    hipLaunchKernelGGL(k_zero_bytes, dim3(blocks_for((long)words, kBlock)), dim3(kBlock), 0, s,
                       reinterpret_cast<uint4*>(near), words);
  }
  hipLaunchKernelGGL(k_features, dim3(blocks_for(pb->n_cells, kBlock)), dim3(kBlock), 0, s, g, *pb,
                     net->cell_box, yn, ynm1, net->perm_h, a0, near);
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

void forward(const Grid& g, const opm_guess_net* net, const Bufs& b, hipStream_t s) {
  const unsigned short* wf = (const unsigned short*)net->wbf16;
  const float* m = net->master;
  conv_launch<kOutRelu>(g, b.a0, wf, m + kLayerW, nullptr, b.a1, nullptr, s);
  conv_launch<kOutRelu>(g, b.a1, wf + kLayerW, m + kLayerParams + kLayerW, nullptr, b.a2, nullptr,
                        s);
  conv_launch<kOutThree>(g, b.a2, wf + 2 * kLayerW, m + 2 * kLayerParams + kLayerW, nullptr,
                         nullptr, b.out, s);
}

}  // namespace

size_t guess_work_bytes(const opm_problem* pb, const opm_guess_net* net) {
  Grid g{net->nx, net->ny, net->nz, net->nx * net->ny * net->nz};
  return bufs_bytes(g, pb->n_cells);
}

int guess_infer(const opm_problem* pb, const opm_guess_net* net, const double* y_n,
                const double* y_nm1, double* y_guess, void* work, hipStream_t s,
                const double** y_extrap) {
  Grid g{net->nx, net->ny, net->nz, net->nx * net->ny * net->nz};
  Bufs b = carve(g, pb->n_cells, work);
  OPM_TRY(features(pb, net, g, y_n, y_nm1, b.a0, b.near, s));
  forward(g, net, b, s);
  const int blocks = blocks_for(pb->n_cells, kBlock);
  hipLaunchKernelGGL(k_guess_apply, dim3(blocks), dim3(kBlock), 0, s, pb->n_cells,
                     net->cell_box, b.near, y_n, y_nm1, b.out, y_guess);
  if (y_extrap) {   // the skip path alone, into the workspace
    hipLaunchKernelGGL(k_guess_apply, dim3(blocks), dim3(kBlock), 0, s, pb->n_cells,
                       net->cell_box, b.near, y_n, y_nm1, (const float*)nullptr, b.yg);
    *y_extrap = b.yg;
  }
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

}  // namespace opm

using namespace opm;

extern "C" {

size_t opm_guess_conv_backward_bytes(int32_t nx, int32_t ny, int32_t nz) {
  if (!valid_grid(nx, ny, nz)) return 0;
  return partial_bytes(Grid{nx, ny, nz, nx * ny * nz});
}

int opm_guess_pack_weights(const float* master, void* wbf16, void* stream) {
  if (!master || !wbf16) return OPM_EINVAL;
  unsigned short* wf = (unsigned short*)wbf16;
  hipLaunchKernelGGL(k_pack_weights, dim3((3 * kLayerW + 255) / 256), dim3(256), 0,
                     as_stream(stream), master, wf, wf + 3 * kLayerW);
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

int opm_guess_conv(int32_t nx, int32_t ny, int32_t nz, const void* in, const void* w_fwd,
                   const float* bias, int32_t relu, void* out_bf16, float* out_f32,
                   void* stream) {
  if (!valid_grid(nx, ny, nz) || !in || !w_fwd || !bias || (relu ? !out_bf16 : !out_f32))
    return OPM_EINVAL;
  Grid g{nx, ny, nz, nx * ny * nz};
  if (relu)
    conv_launch<kOutRelu>(g, (const unsigned short*)in, (const unsigned short*)w_fwd, bias,
                          nullptr, (unsigned short*)out_bf16, nullptr, as_stream(stream));
  else
    conv_launch<kOutAll>(g, (const unsigned short*)in, (const unsigned short*)w_fwd, bias, nullptr,
                         nullptr, out_f32, as_stream(stream));
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

int opm_guess_conv_backward(int32_t nx, int32_t ny, int32_t nz, const void* in, const void* dout,
                            const void* w_bwd, const void* act_in, void* din, float* grad,
                            void* work, size_t work_bytes, void* stream) {
  if (!valid_grid(nx, ny, nz) || !in || !dout || !grad || !work) return OPM_EINVAL;
  if (din && (!w_bwd || !act_in)) return OPM_EINVAL;
  Grid g{nx, ny, nz, nx * ny * nz};
  if (work_bytes < partial_bytes(g)) return OPM_EINVAL;
  backward_launch(g, (const unsigned short*)in, (const unsigned short*)dout,
                  (const unsigned short*)w_bwd, (const unsigned short*)act_in,
                  (unsigned short*)din, grad, (float*)work, as_stream(stream));
  OPM_TRY_HIP(hipGetLastError());
  return OPM_OK;
}

size_t opm_guess_work_bytes(const opm_problem* pb, const opm_guess_net* net) {
  if (!valid_net(pb, net)) return 0;
  return guess_work_bytes(pb, net);
}

int opm_guess_features(const opm_problem* pb, const opm_guess_net* net, const double* y_n,
                       const double* y_nm1, void* feats, void* stream) {
  if (!valid_net(pb, net) || !y_n || !y_nm1 || !feats) return OPM_EINVAL;
  Grid g{net->nx, net->ny, net->nz, net->nx * net->ny * net->nz};
  return features(pb, net, g, y_n, y_nm1, (unsigned short*)feats, nullptr, as_stream(stream));
}

int opm_guess_infer(const opm_problem* pb, const opm_guess_net* net, const double* y_n,
                    const double* y_nm1, double* y_guess, void* work, void* stream) {
  if (!valid_net(pb, net) || !y_n || !y_nm1 || !y_guess || !work) return OPM_EINVAL;
  return guess_infer(pb, net, y_n, y_nm1, y_guess, work, as_stream(stream));
}

int opm_guess_train_step(const opm_problem* pb, const opm_guess_net* net, const double* y_n,
                         const double* y_nm1, const double* y_next, float* adam_m, float* adam_v,
                         int32_t step, float lr, double* loss, void* work, void* stream) {
  if (!valid_net(pb, net) || !y_n || !y_nm1 || !y_next || !adam_m || !adam_v || step < 1 ||
      !(lr > 0.f) || !loss || !work)
    return OPM_EINVAL;
  hipStream_t s = as_stream(stream);
  Grid g{net->nx, net->ny, net->nz, net->nx * net->ny * net->nz};
  Bufs b = carve(g, pb->n_cells, work);
  const unsigned short* wb = (const unsigned short*)net->wbf16 + 3 * kLayerW;
  OPM_TRY(features(pb, net, g, y_n, y_nm1, b.a0, b.near, s));
  forward(g, net, b, s);
  zero_unwritten(g, pb->n_cells, b.d3, s);
  const int nblk = blocks_for(pb->n_cells, kBlock);
  hipLaunchKernelGGL(k_loss, dim3(nblk), dim3(kBlock), 0, s, pb->n_cells, net->cell_box, b.near,
                     b.out, y_n, y_nm1, y_next, b.d3, b.lpart);
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(kBlock), 0, s, b.lpart, nblk, pb->n_cells, loss);
  const unsigned short* layer_in[3] = {b.a0, b.a1, b.a2};
  unsigned short* layer_d[3] = {b.d1, b.d2, b.d3};
  for (int l = 2; l >= 0; --l)
    backward_launch(g, layer_in[l], layer_d[l], wb + (size_t)l * kLayerW, layer_in[l],
                    l > 0 ? layer_d[l - 1] : nullptr, b.grad + (size_t)l * kLayerParams,
                    b.partials, s);
  hipLaunchKernelGGL(k_adam, dim3((kParams + 255) / 256), dim3(256), 0, s, net->master, b.grad,
                     adam_m, adam_v, kParams, lr, 0.9f, 0.999f, 1e-8f, step);
  OPM_TRY_HIP(hipGetLastError());
  return opm_guess_pack_weights(net->master, net->wbf16, stream);
}

}  // extern "C"
