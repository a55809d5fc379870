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
// gathered x, 5 TB/s), FP32 blocks on FP64 vectors 450 us and FP64 554 us; lanes over the columns with every
// block staged in LDS took 2276, 2428 and 2226 us (half the lanes idle at 32 columns, one block in flight). At
// 14 channels, 6 columns, FP64: 128 us, against 299 us for two passes of 4 columns; at 30 channels, M = N = 40,
// 6 and 48 columns 109 and 336 us against 271 and 1572 us.
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

// units of 4 loads that hold the NC rows of a block column
constexpr int row_units(int nc) { return (nc / pk_rows(nc) + 3) / 4; }
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
// wavefront takes a window of 32 complex columns of a block row, its blocks in order;
// lane = real column. Register n of a block holds, in slot s of a quad of lanes, the 4 RPL-row units q of block
// column u with u NQ + q = 16 n + s. The x values of the next block are loaded before the row sums of the
// current one are finished. (Four wavefronts sharing a block row took 232 us where this takes 283 at 18
// channels, M = N = 100, 32 columns, but sum in another order.)
template <int NC>
constexpr int regs_f32() {
  constexpr int r = pk_rows(NC), q = row_units(NC), n = (NC * q + 15) / 16;
  return n * r + n + NC + 8 * q * r;
}
template <int NC>
__global__ void __launch_bounds__(256, waves_for(regs_f32<NC>())) k_spmm_f32(int64_t rows, int B, int cb0, int cb1,
                                                     const int64_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ col, const float* __restrict__ val,
                                                     int npk, const int* __restrict__ pkt, const float* __restrict__ x,
                                                     float* __restrict__ y, const int32_t* __restrict__ order) {
  constexpr int RPL = pk_rows(NC), NQ = row_units(NC), T = NC * NQ, S = 16, NL = (T + S - 1) / S;
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

// FP64 vectors (blocks FP64 or FP32) on v_mfma_f64_4x4x4 (4 products of 4 rows x 4 columns, k = 4, added one
// after another): lane = k 16 + product 4 + (row of A | column of B); D has lane = row 16 + product 4 + column.
// h = 0 .. H - 1 takes complex columns (4 or 16) h + lane column, real and imaginary part as two B operands.
// The Pade sums of a divergent series carry the last bits of a product into the amplitude and into whether it
// is accepted, so the sums are those of the kernels with one lane per row or column, bit for bit, in one of
// two orders (which one: launch_spmv_gen):
//   SP = 0: block after block; the four products are 16 H columns of one block, a wavefront takes a row.
//   SP > 0: pk_slots(NC) partial sums, block e of a row in slot e mod pk_slots(NC), then slot after slot, as
//           k_spmv_pk; the products are up to SP <= 4 slots with 4 H columns each, the wavefronts of a
//           workgroup share a row, that many slots each, and the sums are finished from LDS.
// The sharing also keeps the longest rows, several times the median, off the end of the launch: one wavefront
// per row and all its slots took 384 us at 18 channels, M = N = 150, 4 columns, where this takes 347, and 102
// against 84 at 10 channels, M = N = 130, 2 columns.
constexpr int f64_waves(int nc, int sp) { return sp == 0 ? 1 : (pk_slots(nc) + sp - 1) / sp; }   // of a row

template <int NC, int SP, int H, typename VT>
__global__ void __launch_bounds__(SP ? 64 * f64_waves(NC, SP) : 256, 2)
    k_spmm_f64(int64_t rows, int B, int cb0, int cb1, const int64_t* __restrict__ rowptr,
               const int32_t* __restrict__ col, const VT* __restrict__ val, int npk, const int* __restrict__ pkt,
               const double2* __restrict__ x, double2* __restrict__ y, const int32_t* __restrict__ order) {
  constexpr bool SLOTS = SP > 0;
  constexpr int SL = SLOTS ? pk_slots(NC) : 1, P = SLOTS ? SP : 1, WR = f64_waves(NC, SP);
  constexpr int NR = (NC + 3) / 4, KS = (NC + 3) / 4, CL = SLOTS ? 4 : 16, CW = CL * H;
  // k steps whose values are loaded together: half of them where the registers would spill (more than 24
  // channels; at 29 to 32 with 8 columns 10 to 15 registers still do) or one wavefront fewer per SIMD would fit (13 to
  // 16 channels, 8 columns: 154 -> 128 us at 14 channels, M = N = 100, 6 columns)
  constexpr int KC = (sizeof(VT) == 8 && KS > 6) || (SLOTS && H == 2 && KS == 4) ? (KS + 1) / 2 : KS;
  const int lane = threadIdx.x & 63;
  const int k4 = lane >> 4, i4 = lane & 3, blk = SLOTS ? (lane >> 2) & 3 : 0, cl = lane & (CL - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t W = (int64_t)gridDim.x * (SLOTS ? 1 : 4), w = SLOTS ? blockIdx.x : (int64_t)blockIdx.x * 4 + wv;
  // the wavefront's first slot, the lane's slot relative to it, and whether there is such a slot
  const int c0 = cb0 + blockIdx.y * CW, s0 = SLOTS ? wv * P : 0, sl = min(blk, P - 1);
  const bool has = blk < P && s0 + blk < SL;
  __shared__ double2 red[WR][SLOTS ? NR * H : 1][64];
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
  // channel of the rows a lane writes: of D (row = lane / 16), or of the thread's share of the values
  // (rt H + h, row, column) finished from LDS
  constexpr int OUT = SLOTS ? (NR * H * 16 + 64 * WR - 1) / (64 * WR) : NR;
  int och[OUT];
#pragma unroll
  for (int o = 0; o < OUT; ++o) {
    const int t = o * 64 * WR + threadIdx.x;
    const int r = SLOTS ? 4 * (t / (16 * H)) + ((t >> 2) & 3) : 4 * o + k4;
    och[o] = r < NC ? pkt[r] : -1;
  }
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
  if (b0 + s0 < b1) load_x(col[min(b0 + s0 + sl, b1 - 1)]);
  while (true) {
    const int64_t nrow = uniform(stripe_row(rows, W, w, ++s, order));
    const int64_t n0 = nrow >= 0 ? rowptr[nrow] : 0, n1 = nrow >= 0 ? rowptr[nrow + 1] : 0;
    double re[NR][H], im[NR][H];
#pragma unroll
    for (int rt = 0; rt < NR; ++rt)
#pragma unroll
      for (int h = 0; h < H; ++h) re[rt][h] = im[rt][h] = 0.0;
    const VT* vp = val + b0 * npk;
    if (b0 + s0 >= b1 && n0 + s0 < n1) load_x(col[min(n0 + s0 + sl, n1 - 1)]);
    for (int64_t cb = b0 + s0; cb < b1; cb += SL) {
      const bool ok = has && cb + blk < b1;
      const unsigned eo = ok ? (unsigned)(cb - b0 + blk) * (unsigned)npk : 0u;
      const bool more = cb + SL < b1;
      const int64_t f0 = more ? cb + SL : n0 + s0, f1 = more ? b1 : n1;
      int32_t cn = 0;
#pragma unroll
      for (int kc = 0; kc < KS; kc += KC) {
        VT a[KC][NR];
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
          for (int rt = 0; rt < NR; ++rt)
            if (kc + ks < KS) a[ks][rt] = vp[mok[kc + ks][rt] ? eo + (unsigned)(moff[kc + ks] + 4 * rt) : 0u];
        if (kc == 0) cn = f0 < f1 ? col[min(f0 + sl, f1 - 1)] : 0;
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
          for (int rt = 0; rt < NR; ++rt)
            if (kc + ks < KS) {
              const double av = (ok && mok[kc + ks][rt]) ? (double)a[ks][rt] : 0.0;
#pragma unroll
              for (int h = 0; h < H; ++h) {
                re[rt][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, xv[kc + ks][h].x, re[rt][h], 0, 0, 0);
                im[rt][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, xv[kc + ks][h].y, im[rt][h], 0, 0, 0);
              }
            }
      }
      if (f0 < f1) load_x(cn);
    }
    if constexpr (SLOTS) {
#pragma unroll
      for (int rt = 0; rt < NR; ++rt)
#pragma unroll
        for (int h = 0; h < H; ++h) red[wv][rt * H + h][lane] = make_double2(re[rt][h], im[rt][h]);
      __syncthreads();
#pragma unroll
      for (int o = 0; o < OUT; ++o) {
        const int t = o * 64 * WR + threadIdx.x, k = t / 16, l = ((t >> 2) & 3) * 16 + (t & 3);
        const int c = c0 + (k % H) * CL + (t & 3);
        if (och[o] < 0 || c >= cb1) continue;
        double2 v = red[0][k][l];
#pragma unroll
        for (int q = 1; q < SL; ++q) {
          const double2 p = red[q / P][k][l + 4 * (q % P)];
          v.x += p.x;
          v.y += p.y;
        }
        y[((int64_t)row * NC + och[o]) * B + c] = v;
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int rt = 0; rt < NR; ++rt)
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int c = c0 + h * CL + cl;
          if (och[rt] >= 0 && c < cb1) y[((int64_t)row * NC + och[rt]) * B + c] = make_double2(re[rt][h], im[rt][h]);
        }
    }
    if (nrow < 0) break;
    row = nrow;
    b0 = n0;
    b1 = n1;
  }
}

// Persistent grid: as many workgroups as the device holds at once, at most one per row (shared by its wavefronts) or
// per four rows.
template <typename K>
int resident(K kernel, int threads) {   // workgroups per compute unit
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel), threads, 0) != hipSuccess)
    n = 0;
  return std::max(1, n);
}
inline dim3 spmm_grid(int64_t rows, int per_cu, bool shared, int cols, int window) {
  const int64_t wg = std::min<int64_t>(shared ? rows : (rows + 3) / 4, (int64_t)per_cu * kCUs);
  return dim3((unsigned)std::max<int64_t>(1, wg), (unsigned)((cols + window - 1) / window));
}

// Slots per wavefront, the same in all of them if possible: 4 of 12 (10 channels), 3 of 9 (14), 4 and 3 of 7 (18),
// 4 of 4 (30). Fewer read P0 in more, emptier loads: 2 of 7 took 227 us where 4 take 147 (M = N = 100, 2 columns).
constexpr int f64_slots(int nc) {
  const int waves = (pk_slots(nc) + 3) / 4;
  return (pk_slots(nc) + waves - 1) / waves;
}

// FP32 vectors: 24 channels at most (launch)
template <int NC>
void launch_nc(int64_t rows, int B, int cb0, int cb1, const int64_t* rowptr, const int32_t* col, const float* val, int npk,
               const int* pkt, const float2* x, float2* y, const int32_t* order, bool, hipStream_t s) {
  if constexpr (NC <= 24) {
    static const int per_cu = resident(k_spmm_f32<NC>, 256);
    hipLaunchKernelGGL(k_spmm_f32<NC>, spmm_grid(rows, per_cu, false, cb1 - cb0, 32), dim3(256), 0, s, rows, B, cb0, cb1,
                       rowptr, col, val, npk, pkt, reinterpret_cast<const float*>(x), reinterpret_cast<float*>(y), order);
  }
}

template <int NC, typename VT>
void launch_nc(int64_t rows, int B, int cb0, int cb1, const int64_t* rowptr, const int32_t* col, const VT* val, int npk,
               const int* pkt, const double2* x, double2* y, const int32_t* order, bool blockwise, hipStream_t s) {
#define WP_W(SP, H)                                                                                                \
  {                                                                                                                \
    constexpr int threads = SP ? 64 * f64_waves(NC, SP) : 256;                                                     \
    static const int per_cu = resident(k_spmm_f64<NC, SP, H, VT>, threads);                                        \
    hipLaunchKernelGGL((k_spmm_f64<NC, SP, H, VT>), spmm_grid(rows, per_cu, SP != 0, cb1 - cb0, (SP ? 4 : 16) * H), \
                       dim3(threads), 0, s, rows, B, cb0, cb1, rowptr, col, val, npk, pkt, x, y, order);           \
  }
  // the narrowest window that holds the call's columns, at most 8 by slots and 32 block after block
  if (!blockwise) {
    if (B <= 4) WP_W(f64_slots(NC), 1)
    else WP_W(f64_slots(NC), 2)
  } else if constexpr (NC <= 24) {
    if (B <= 16) WP_W(0, 1)
    else WP_W(0, 2)
  }
#undef WP_W
}

// blockwise: block after block (at most 24 channels), else by slots (FP64 vectors only)
template <typename VT, typename XT>
hipError_t launch(int64_t rows, int nch, int B, const int64_t* rowptr, const int32_t* col, const VT* val, const XT* x,
                  XT* y, hipStream_t s, int cb0, int cb1, const int32_t* order, const PackView& pk, bool blockwise) {
  if (cb1 < 0) cb1 = B;
  if (cb0 < 0 || cb1 > B || cb0 >= cb1 || rows < 1 || nch < 5 || nch > PK_MAX || !pk.pkt || pk.npk < 1 ||
      pk.npk > nch * nch || (blockwise ? nch > 24 : sizeof(XT) == 8))
    return hipErrorInvalidValue;
  switch (nch) {
#define WP_NC(n) \
  case n: launch_nc<n>(rows, B, cb0, cb1, rowptr, col, val, pk.npk, pk.pkt, x, y, order, blockwise, s); break;
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
