// Block-CSR products y = P0 x for many channels (nch > 4, packed blocks) on the matrix cores.
//
// A packed block holds, for every block column u (a position of the packed channel order), the rows
// [lo_u, hi_u) at off_u - lo_u + r (PackDesc; pkt[0, NC) = position -> channel, then lo, hi, off).
// x and y are [cell][channel][column] complex, seen here as [cell][channel][2 B] reals.
//
// The product is bound by the P0 stream (few columns) or by the x gathers (many): the kernels are
// laid out so that a block costs few instructions and no LDS, which leaves the registers to hold
// loads in flight. Small matrix tiles of 4 rows fit 10, 14 and 18 channels without the padding of a
// 16-row tile, and their operands are what the loads deliver: lane = (4-row tile, row) for P0,
// lane = real column for x.
//
// Measured at 18 channels, M = N = 100 (250 k blocks), 32 columns: FP32 283 us (1.4 GB of P0 and
// gathered x, 5 TB/s) and FP32 blocks on FP64 vectors 384 us; lanes over the columns with every block
// staged in LDS took 2276 and 2428 us (half the lanes idle at 32 columns, one block in flight). At 14
// channels, 6 columns, FP64: 120 us, against 275 us for two passes of 4 columns.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "wpcd_internal.h"

namespace wpcd {
namespace spmm {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kCUs = 256;   // MI355X compute units: the persistent grids

template <int R> struct RowsOf { using T = float; };
template <> struct RowsOf<2> { using T = float2; };
__device__ __forceinline__ float part(const float& v, int) { return v; }
__device__ __forceinline__ float part(const float2& v, int k) { return k ? v.y : v.x; }

// rows per load: the packed intervals are pairs of rows when NC is even (PackDesc)
constexpr int rows_per_load(int nc) { return nc % 2 == 0 ? 2 : 1; }
// units of 4 loads that hold the NC rows of a block column
constexpr int row_units(int nc) { return (nc / rows_per_load(nc) + 3) / 4; }
// wavefronts per SIMD that the registers of a kernel leave room for (`regs`: what its arrays take)
constexpr int waves_for(int regs) { return regs <= 72 ? 6 : regs <= 96 ? 5 : regs <= 120 ? 4 : regs <= 160 ? 3 : 2; }

// Row sequence of worker w of W (row s of its sequence, -1 past the end): with the longest rows
// first, stripe s is walked forwards when s is even and backwards when it is odd, so that every
// worker gets about the same number of blocks.
__device__ __forceinline__ int64_t stripe_row(int64_t rows, int64_t W, int64_t w, int64_t s,
                                              const int32_t* __restrict__ order) {
  const int64_t k = s * W + ((s & 1) ? W - 1 - w : w);
  if (k >= rows) return -1;
  return order ? order[k] : k;
}
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(v & 0xffffffffu));
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// FP32 blocks and vectors on v_mfma_f32_4x4x1 (16 products of 4 rows x 4 columns, one k): with A
// broadcast over the 16 products (cbsz = 4), one instruction adds P0[4 rows][u] x[u][64 real columns]. A
// wavefront takes a window of 32 complex columns of a block row, its blocks in order (PackView.one_order);
// lane = real column. Register n of a block holds, in slot s of a quad of lanes, the 4 RPL-row units q of block
// column u with u NQ + q = 16 n + s. The x values of the next block are loaded before the row sums of the
// current one are finished. (Four wavefronts sharing a block row took 232 us where this takes 283 at 18
// channels, M = N = 100, 32 columns, but sum in another order.)
template <int NC>
constexpr int regs_f32() {
  constexpr int r = rows_per_load(NC), q = row_units(NC), n = (NC * q + 15) / 16;
  return n * r + n + NC + 8 * q * r;
}
template <int NC>
__global__ void __launch_bounds__(256, waves_for(regs_f32<NC>())) k_spmm_f32(int64_t rows, int B, int cb0, int cb1,
                                                     const int64_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ col, const float* __restrict__ val,
                                                     int npk, const int* __restrict__ pkt, const float* __restrict__ x,
                                                     float* __restrict__ y, const int32_t* __restrict__ order) {
  constexpr int RPL = rows_per_load(NC), NQ = row_units(NC), T = NC * NQ, S = 16, NL = (T + S - 1) / S;
  using VR = typename RowsOf<RPL>::T;
  const int lane = threadIdx.x & 63, i4 = lane & 3;
  const int64_t W = (int64_t)gridDim.x * 4, w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = cb0 + blockIdx.y * 32;
  const int cr = 2 * c0 + lane;                  // real column of the lane
  const bool live = cr < 2 * cb1;
  const int crc = live ? cr : 2 * cb1 - 1;       // columns past the end are computed and not stored
  // packed position of the lane's rows in every register of a block; rows that are not stored read
  // position 0 and count as zero
  int moff[NL];
  bool mok[NL];
#pragma unroll
  for (int n = 0; n < NL; ++n) {
    const int t = n * S + (lane >> 2);
    const int u = t < T ? t / NQ : 0, r = RPL * (4 * (t - u * NQ) + i4);
    mok[n] = t < T && r >= pkt[NC + u] && r < pkt[2 * NC + u];
    moff[n] = mok[n] ? pkt[3 * NC + u] - pkt[NC + u] + r : 0;
  }
  const int64_t xst = 2 * (int64_t)B;
  float xv[NC];
  auto load_x = [&](int32_t c) {
    const float* xc = x + (int64_t)c * NC * xst + crc;
#pragma unroll
    for (int u = 0; u < NC; ++u) xv[u] = xc[pkt[u] * xst];
  };
  int64_t s = 0;
  int64_t row = uniform(stripe_row(rows, W, w, s, order));
  if (row < 0) return;
  int64_t b0 = rowptr[row], b1 = rowptr[row + 1];
  if (b0 < b1) load_x(col[b0]);
  while (true) {
    const int64_t nrow = uniform(stripe_row(rows, W, w, ++s, order));
    const int64_t n0 = nrow >= 0 ? rowptr[nrow] : 0, n1 = nrow >= 0 ? rowptr[nrow + 1] : 0;
    f32x4 acc[NQ * RPL];
#pragma unroll
    for (int a = 0; a < NQ * RPL; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* vp = val + b0 * npk;
    if (b0 >= b1 && n0 < n1) load_x(col[n0]);
    for (int64_t cb = b0; cb < b1; ++cb) {
      const unsigned eo = (unsigned)(cb - b0) * (unsigned)npk;
      // the next block (of this row or of the next one)
      const bool more = cb + 1 < b1;
      const int64_t f0 = more ? cb + 1 : n0, f1 = more ? b1 : n1;
      VR a[NL];
#pragma unroll
      for (int n = 0; n < NL; ++n) a[n] = *reinterpret_cast<const VR*>(vp + (eo + (unsigned)moff[n]));
      const int32_t cn = f0 < f1 ? col[f0] : 0;
#pragma unroll
      for (int n = 0; n < NL; ++n) {
        float av[RPL];
#pragma unroll
        for (int j = 0; j < RPL; ++j) av[j] = mok[n] ? part(a[n], j) : 0.f;
        // the slots of the register: the broadcast index has to be a literal
#define WP_SLOT(sl)                                                                                          \
  {                                                                                                          \
    const int t = n * S + sl;                                                                                \
    if (t < T) {                                                                                             \
      const int u = t / NQ, q = t - u * NQ;                                                                  \
      _Pragma("unroll") for (int j = 0; j < RPL; ++j)                                                        \
        acc[q * RPL + j] = __builtin_amdgcn_mfma_f32_4x4x1f32(av[j], xv[u], acc[q * RPL + j], 4, sl, 0);     \
    }                                                                                                        \
  }
        WP_SLOT(0) WP_SLOT(1) WP_SLOT(2) WP_SLOT(3) WP_SLOT(4) WP_SLOT(5) WP_SLOT(6) WP_SLOT(7)
        WP_SLOT(8) WP_SLOT(9) WP_SLOT(10) WP_SLOT(11) WP_SLOT(12) WP_SLOT(13) WP_SLOT(14) WP_SLOT(15)
#undef WP_SLOT
      }
      if (f0 < f1) load_x(cn);
    }
    // value k of the lane: row RPL (4 q + k mod 4) + j of the block row, in accumulator q RPL + j
#pragma unroll
    for (int k = 0; k < 4 * NQ * RPL; ++k) {
      const int ac = k >> 2, q = ac / RPL, r = RPL * (4 * q + (k & 3)) + ac - q * RPL;
      if (r < NC && live) y[((int64_t)row * NC + pkt[r]) * xst + cr] = acc[ac][k & 3];
    }
    if (nrow < 0) break;
    row = nrow;
    b0 = n0;
    b1 = n1;
  }
}

// FP64 vectors (blocks FP64 or FP32) on v_mfma_f64_4x4x4 (4 products of 4 rows x 4 columns, k = 4):
// lane = k 16 + product 4 + (row of A | column of B); D has lane = row 16 + product 4 + column. GB = 4:
// the four products are four P0 blocks of the row, each with 4 H complex columns; GB = 1: one block
// with 16 H complex columns. h = 0 .. H - 1 takes complex columns (4 or 16) h + lane column, real and
// imaginary part as two B operands. WR wavefronts share a block row (4 where its one or two blocks per pass would
// leave the longest rows, several times the median, at the end of the launch); their sums are added in LDS.
template <int CTRL>
__device__ __forceinline__ double row_rotated(double v) {   // within rows of 16 lanes
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

template <int NC, int GB, int H, int WR, typename VT>
__global__ void __launch_bounds__(256, 2)
    k_spmm_f64(int64_t rows, int B, int cb0, int cb1, const int64_t* __restrict__ rowptr,
               const int32_t* __restrict__ col, const VT* __restrict__ val, int npk, const int* __restrict__ pkt,
               const double2* __restrict__ x, double2* __restrict__ y, const int32_t* __restrict__ order) {
  constexpr int NR = (NC + 3) / 4, KS = (NC + 3) / 4, CL = GB == 4 ? 4 : 16, CW = CL * H;
  const int lane = threadIdx.x & 63;
  const int k4 = lane >> 4, i4 = lane & 3, blk = GB == 4 ? (lane >> 2) & 3 : 0, cl = lane & (CL - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = WR == 4 ? wv : 0;
  const int64_t W = (int64_t)gridDim.x * (4 / WR), w = WR == 4 ? blockIdx.x : (int64_t)blockIdx.x * 4 + wv;
  const int c0 = cb0 + blockIdx.y * CW;
  __shared__ double2 red[WR == 4 ? 4 : 1][WR == 4 ? NR * H : 1][64];
  // packed position of the lane's row 0 in the block columns of every k step, which of its rows are
  // stored there (the others read position 0 and count as zero), and the lane's channel of x
  int moff[KS], xo[KS];
  bool mok[KS][NR];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int u = min(4 * ks + k4, NC - 1);
    moff[ks] = pkt[3 * NC + u] - pkt[NC + u] + i4;
    xo[ks] = pkt[u] * B;
#pragma unroll
    for (int rt = 0; rt < NR; ++rt) {
      const int r = 4 * rt + i4;
      mok[ks][rt] = 4 * ks + k4 < NC && r >= pkt[NC + u] && r < pkt[2 * NC + u];
    }
  }
  int och[NR];   // channel of the lane's output rows (D: row = lane / 16)
#pragma unroll
  for (int rt = 0; rt < NR; ++rt) och[rt] = 4 * rt + k4 < NC ? pkt[4 * rt + k4] : -1;
  int cc[H];
#pragma unroll
  for (int h = 0; h < H; ++h) cc[h] = min(c0 + h * CL + cl, cb1 - 1);
  double2 xv[KS][H];
  auto load_x = [&](int32_t c) {
    const double2* xc = x + (int64_t)c * NC * B;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int h = 0; h < H; ++h) xv[ks][h] = xc[xo[ks] + cc[h]];
  };
  int64_t s = 0;
  int64_t row = uniform(stripe_row(rows, W, w, s, order));
  if (row < 0) return;
  int64_t b0 = rowptr[row], b1 = rowptr[row + 1];
  if (b0 + wr * GB < b1) load_x(col[min(b0 + wr * GB + blk, b1 - 1)]);
  while (true) {
    const int64_t nrow = uniform(stripe_row(rows, W, w, ++s, order));
    const int64_t n0 = nrow >= 0 ? rowptr[nrow] : 0, n1 = nrow >= 0 ? rowptr[nrow + 1] : 0;
    double acc[NR][H][2];
#pragma unroll
    for (int rt = 0; rt < NR; ++rt)
#pragma unroll
      for (int h = 0; h < H; ++h) acc[rt][h][0] = acc[rt][h][1] = 0.0;
    const VT* vp = val + b0 * npk;
    if (b0 + wr * GB >= b1 && n0 + wr * GB < n1) load_x(col[min(n0 + wr * GB + blk, n1 - 1)]);
    for (int64_t cb = b0 + wr * GB; cb < b1; cb += WR * GB) {
      const bool ok = cb + blk < b1;
      const unsigned eo = ok ? (unsigned)(cb - b0 + blk) * (unsigned)npk : 0u;
      const bool more = cb + WR * GB < b1;
      const int64_t f0 = more ? cb + WR * GB : n0 + wr * GB, f1 = more ? b1 : n1;
      VT a[KS][NR];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int rt = 0; rt < NR; ++rt) a[ks][rt] = vp[mok[ks][rt] ? eo + (unsigned)(moff[ks] + 4 * rt) : 0u];
      const int32_t cn = f0 < f1 ? col[min(f0 + blk, f1 - 1)] : 0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int rt = 0; rt < NR; ++rt) {
          const double av = (ok && mok[ks][rt]) ? (double)a[ks][rt] : 0.0;
#pragma unroll
          for (int h = 0; h < H; ++h) {
            acc[rt][h][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, xv[ks][h].x, acc[rt][h][0], 0, 0, 0);
            acc[rt][h][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, xv[ks][h].y, acc[rt][h][1], 0, 0, 0);
          }
        }
      if (f0 < f1) load_x(cn);
    }
    if constexpr (WR == 4) {
#pragma unroll
      for (int rt = 0; rt < NR; ++rt)
#pragma unroll
        for (int h = 0; h < H; ++h) red[wv][rt * H + h][lane] = make_double2(acc[rt][h][0], acc[rt][h][1]);
      __syncthreads();
    }
#pragma unroll
    for (int rt = 0; rt < NR; ++rt)
#pragma unroll
      for (int h = 0; h < H; ++h) {
        double re = acc[rt][h][0], im = acc[rt][h][1];
        if (WR == 4) {   // value k is finished by wavefront k mod 4
          const int k = rt * H + h;
          if ((k & 3) != wv) continue;
          const double2 r0 = red[0][k][lane], r1 = red[1][k][lane], r2 = red[2][k][lane], r3 = red[3][k][lane];
          re = (r0.x + r1.x) + (r2.x + r3.x);
          im = (r0.y + r1.y) + (r2.y + r3.y);
        }
        if (GB == 4) {   // sum over the products (lane bits 2 and 3), the same in every lane
          re += row_rotated<0x128>(re);
          im += row_rotated<0x128>(im);
          re += row_rotated<0x124>(re);
          im += row_rotated<0x124>(im);
        }
        const int c = c0 + h * CL + cl;
        if (och[rt] >= 0 && c < cb1 && blk == 0) y[((int64_t)row * NC + och[rt]) * B + c] = make_double2(re, im);
      }
    if constexpr (WR == 4) __syncthreads();
    if (nrow < 0) break;
    row = nrow;
    b0 = n0;
    b1 = n1;
  }
}

// Persistent grid: as many workgroups as the device holds at once, at most one per row (WR = 4) or per four rows.
template <typename K>
int resident(K kernel) {   // workgroups per compute unit
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel), 256, 0) != hipSuccess)
    n = 0;
  return std::max(1, n);
}
inline dim3 spmm_grid(int64_t rows, int per_cu, int wr, int cols, int window) {
  const int64_t wg = std::min<int64_t>(wr == 4 ? rows : (rows + 3) / 4, (int64_t)per_cu * kCUs);
  return dim3((unsigned)std::max<int64_t>(1, wg), (unsigned)((cols + window - 1) / window));
}

// Columns a wavefront takes: the narrowest window that holds a call of B columns, at most 32 (an
// explicit spmm_cols asks for the widest from that count on).
inline int spmm_window(int B, int spmm_min) {
  if (spmm_min > 0 && B >= spmm_min) return 32;
  return B <= 4 ? 4 : B <= 8 ? 8 : B <= 16 ? 16 : 32;
}
// The narrow windows share a block row among four wavefronts until the rows alone fill the device:
// 10 channels, M = N = 40, 4 columns, FP64: 12 us shared, 22 us not; 18 channels, M = N = 150, 8
// columns: 441 us shared, 406 us not.
inline bool shared_rows(int64_t rows) { return rows < 16384; }

template <int NC>
void launch_nc(int64_t rows, int B, int cb0, int cb1, const int64_t* rowptr, const int32_t* col, const float* val, int npk,
               const int* pkt, const float2* x, float2* y, const int32_t* order, int, bool, hipStream_t s) {
  static const int per_cu = resident(k_spmm_f32<NC>);
  hipLaunchKernelGGL(k_spmm_f32<NC>, spmm_grid(rows, per_cu, 1, cb1 - cb0, 32), dim3(256), 0, s, rows, B, cb0, cb1,
                     rowptr, col, val, npk, pkt, reinterpret_cast<const float*>(x), reinterpret_cast<float*>(y), order);
}

template <int NC, typename VT>
void launch_nc(int64_t rows, int B, int cb0, int cb1, const int64_t* rowptr, const int32_t* col, const VT* val, int npk,
               const int* pkt, const double2* x, double2* y, const int32_t* order, int window, bool one_order, hipStream_t s) {
#define WP_W(gb, h, wr)                                                                                       \
  {                                                                                                           \
    static const int per_cu = resident(k_spmm_f64<NC, gb, h, wr, VT>);                                        \
    hipLaunchKernelGGL((k_spmm_f64<NC, gb, h, wr, VT>),                                                       \
                       spmm_grid(rows, per_cu, wr, cb1 - cb0, (gb == 4 ? 4 : 16) * h), dim3(256), 0, s, rows, \
                       B, cb0, cb1, rowptr, col, val, npk, pkt, x, y, order);                                 \
  }
  const bool sh = shared_rows(rows);
  if (window <= 4 && sh) WP_W(4, 1, 4)
  else if (window <= 4) WP_W(4, 1, 1)
  else if (window <= 8 && sh) WP_W(4, 2, 4)
  else if (window <= 8) WP_W(4, 2, 1)
  else if (one_order) WP_W(1, 2, 1)
  else if (window <= 16) WP_W(1, 1, 4)
  else WP_W(1, 2, 4)
#undef WP_W
}

template <typename VT, typename XT>
hipError_t launch(int64_t rows, int nch, int B, const int64_t* rowptr, const int32_t* col, const VT* val, const XT* x,
                  XT* y, hipStream_t s, int cb0, int cb1, const int32_t* order, const PackView& pk) {
  if (cb1 < 0) cb1 = B;
  if (cb0 < 0 || cb1 > B || cb0 >= cb1 || rows < 1 || nch < 5 || nch > PK_MAX || !pk.pkt || pk.npk < 1 ||
      pk.npk > nch * nch)
    return hipErrorInvalidValue;
  // the choice depends on B and the options only, so every launch on a given batch width sums in one order
  const int window = pk.one_order ? 32 : spmm_window(B, pk.spmm_min);
  switch (nch) {
#define WP_NC(n) \
  case n: launch_nc<n>(rows, B, cb0, cb1, rowptr, col, val, pk.npk, pk.pkt, x, y, order, window, pk.one_order, s); break;
    WP_NC(5) WP_NC(6) WP_NC(7) WP_NC(8) WP_NC(9) WP_NC(10) WP_NC(11) WP_NC(12) WP_NC(13) WP_NC(14)
    WP_NC(15) WP_NC(16) WP_NC(17) WP_NC(18) WP_NC(19) WP_NC(20) WP_NC(21) WP_NC(22) WP_NC(23) WP_NC(24)
    WP_NC(25) WP_NC(26) WP_NC(27) WP_NC(28) WP_NC(29) WP_NC(30) WP_NC(31) WP_NC(32)
#undef WP_NC
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace spmm
}  // namespace wpcd
