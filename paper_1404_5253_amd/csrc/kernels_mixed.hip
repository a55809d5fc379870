// Mixed-precision kernels of the iteration (FP32 vectors, BF16 blocks on MFMA with FP32
// accumulation) and the FP64 helpers of the residual refinement.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "spmm_rows.h"
#include "wpcd_internal.h"

namespace wpcd {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// hi + lo split of a value: hi = bf16(x), lo = bf16(x - hi), each rounded to nearest even
__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
#pragma clang fp contract(off)   // x is a rounded product: a fused x - hi would be of the exact one
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

// One channel g (pair wave w) and 8*CT complex columns (16*CT real columns: re/im of each):
//   t = O y on MFMA 16x16x16 bf16, t *= G1 (FP32), s = (v O^T) t on MFMA, s written in FP32.
// SPLIT = false: y, t, O and v O^T rounded to bf16 once (one product per tile);
// SPLIT = true: every operand x is carried as hi + lo with hi = bf16(x), lo = bf16(x - hi), and
//   a tile product is A_hi B_hi + A_hi B_lo + A_lo B_hi (16 significant bits per operand).
// Accumulation is FP32 throughout.
// MFMA operands: lane l holds row l%16 of A and column l%16 of B at the 8 k of its quarter q = l/16; within
// a block of 32 these are 4q .. 4q+3 and 16+4q .. 16+4q+3, the order in which the fragment tables and the
// LDS tile hold them, so that one 16-byte read serves two 16x16x16 products in ascending k (one 16x16x32
// instruction would be 1 to 3 us faster at the sizes below, but sums in another order: a refinement's columns
// then stop elsewhere). The result is D[4(l/16)+r][l%16], r = 0..3.
// The products are a small part of the time (18 channels, M = N = 150, 4 columns: 6.6 GFLOP); what counts
// is how many loads are under way. O and v O^T come as fragment tables (launch_pack_bf16): for row tile
// kt and k step s of 32, the hi then the lo operands of the 64 lanes, 16 bytes each, read D steps ahead
// and first before y is staged. The wavefronts share the row tiles, TPW each, with all accumulators in
// registers, so one LDS tile [real column][k] serves as Y and then as T; a thread stages four
// neighbouring k of one column. Rows of the LDS tile are Kp + 8 entries long: 16 lanes reading 16
// bytes of 16 columns then fall on all banks. Measured (split; with events around each launch) against two
// LDS tiles and row-major tables: 47 -> 30 us at the sizes above, 27 -> 21 us at 2 channels, M = N = 100, 64
// columns and 17 -> 8 us at one, 121 -> 22 us at 1 channel, M = 400, N = 300, 4 columns.
// one half (q) of a 32-wide k step
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, int q, f32x4 c) {
  const s16x8 x = __builtin_bit_cast(s16x8, a), z = __builtin_bit_cast(s16x8, b);
  return q == 0 ? __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(x, x, 0, 1, 2, 3),
                                                            __builtin_shufflevector(z, z, 0, 1, 2, 3), c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_shufflevector(x, x, 4, 5, 6, 7),
                                                            __builtin_shufflevector(z, z, 4, 5, 6, 7), c, 0, 0, 0);
}

template <bool SPLIT, int CT, int TPW, int D>
__global__ void __launch_bounds__(1024) k_step_bf16(RotArgsMixed r, const float2* __restrict__ y,
                                                    float2* __restrict__ s_out, int nt, int ns) {
  extern __shared__ __align__(16) unsigned char shb[];
  constexpr int NP = SPLIT ? 2 : 1;
  constexpr int RC = 16 * CT;     // real columns per block
  constexpr int CC = 8 * CT;      // complex columns per block
  const int M = r.M, B = r.B, nch = r.nch, ncol = r.N * B;
  const int Kp = 32 * ns, KS = Kp + 8;
  __bf16* T = reinterpret_cast<__bf16*>(shb);   // [NP][RC][KS], real column rc = 2 cc + part
  // Workgroups are dispatched round robin to the 8 XCDs by linear id. Each XCD is given a contiguous
  // range of the sequence (channel group, tile, channel of the group), so that it reads the tables of
  // a few channels (which then stay in its L2); a group holds the channels whose entries of one cell
  // share a 128-byte line of y, G1 and s. The map is a bijection over the grid.
  const int ntx = gridDim.x, W = ntx * gridDim.y;
  const int lin = blockIdx.x + ntx * blockIdx.y;
  const int xcd = lin & 7, per = W >> 3, extra = W & 7;
  const int idx = xcd * per + min(xcd, extra) + (lin >> 3);
  const int cg = max(1, min(nch, 16 / B)), gp = idx / (ntx * cg), rem = idx - gp * ntx * cg;
  const int gn = min(cg, nch - gp * cg);
  const int tile = rem / gn, g = gp * cg + rem - tile * gn;
  const int col0 = tile * CC;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nthr = blockDim.x, nw = nthr >> 6;
  const int rc = lane & 15, quad = lane >> 4, part = rc & 1;
  const size_t woff = (size_t)r.wave[g] * nt * ns * 128 + lane;

  const bf16x8* p[TPW];
  bf16x8 buf[D][TPW][NP];
  auto fetch = [&](int u, int s) {
#pragma unroll
    for (int h = 0; h < TPW; ++h)
#pragma unroll
      for (int q = 0; q < NP; ++q) buf[u][h][q] = p[h][(size_t)min(s, ns - 1) * 128 + q * 64];
  };
  auto start = [&](const bf16x8* table) {
#pragma unroll
    for (int h = 0; h < TPW; ++h) p[h] = table + woff + (size_t)min(wv + h * nw, nt - 1) * ns * 128;
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(u, u);
  };
  f32x4 acc[TPW][CT];
  auto mult = [&](int s, const bf16x8 (&a)[TPW][NP]) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const __bf16* bp = T + (ct * 16 + rc) * KS + 32 * s + 8 * quad;
      const bf16x8 bh = *reinterpret_cast<const bf16x8*>(bp);
      bf16x8 bl;
      if (SPLIT) bl = *reinterpret_cast<const bf16x8*>(bp + RC * KS);
#pragma unroll
      for (int h = 0; h < TPW; ++h) {
        // k in ascending order, high x high, high x low and low x high parts per 16 of it
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          acc[h][ct] = mfma16(a[h][0], bh, q, acc[h][ct]);
          if (SPLIT) {
            acc[h][ct] = mfma16(a[h][0], bl, q, acc[h][ct]);
            acc[h][ct] = mfma16(a[h][NP - 1], bh, q, acc[h][ct]);
          }
        }
      }
    }
  };
  auto product = [&]() {
#pragma unroll
    for (int h = 0; h < TPW; ++h)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[h][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    int s0 = 0;
    for (; s0 + D <= ns; s0 += D)
#pragma unroll
      for (int u = 0; u < D; ++u) {
        mult(s0 + u, buf[u]);
        fetch(u, s0 + u + D);
      }
#pragma unroll
    for (int u = 0; u < D - 1; ++u)
      if (s0 + u < ns) mult(s0 + u, buf[u]);
  };

  start(reinterpret_cast<const bf16x8*>(r.Of));
  {   // y: column cc of the thread is fixed (the workgroup is a multiple of CC threads)
    const int cc = tid % CC, col = col0 + cc;
    const bool live = col < ncol;
    const int jj = live ? col / B : 0, cb = live ? col - jj * B : 0;
    const float sc = r.yscale ? (float)r.yscale[cb] : 1.f;
    const float2* yc = y + ((size_t)jj * M * nch + g) * B + cb;
    const size_t ist = (size_t)nch * B;
    for (int ib = tid / CC; ib < Kp / 4; ib += nthr / CC) {
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = live && 4 * ib + t < M ? yc[(4 * ib + t) * ist] : make_float2(0.f, 0.f);
      bf16x4 h[2], l[2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        __bf16 hx, lx, hy, ly;
        split_bf16(v[t].x * sc, hx, lx);
        split_bf16(v[t].y * sc, hy, ly);
        h[0][t] = hx;
        h[1][t] = hy;
        l[0][t] = lx;
        l[1][t] = ly;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        __bf16* d = T + (2 * cc + q) * KS + 32 * (ib >> 3) + 8 * (ib & 3) + (ib & 4);
        *reinterpret_cast<bf16x4*>(d) = h[q];
        if (SPLIT) *reinterpret_cast<bf16x4*>(d + RC * KS) = l[q];
      }
    }
  }
  bool live[CT];
  int jj[CT], cb[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int col = col0 + ct * 8 + (rc >> 1);
    live[ct] = col < ncol;
    jj[ct] = live[ct] ? col / B : 0;
    cb[ct] = live[ct] ? col - jj[ct] * B : 0;
  }
  // G1 of the wavefront's rows, in flight during the product where the registers allow it
  constexpr bool AHEAD = TPW * CT <= 2;
  float2 gv[AHEAD ? TPW : 1][AHEAD ? CT : 1][4];
  auto load_g = [&](int h, int ct, float2 (&v)[4]) {
    const int k0 = (wv + h * nw) * 16 + 4 * quad;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = r.G[(((size_t)jj[ct] * M + (k0 + q < M ? k0 + q : 0)) * nch + g) * B + cb[ct]];
  };
  if constexpr (AHEAD) {
#pragma unroll
    for (int h = 0; h < TPW; ++h)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) load_g(h, ct, gv[h][ct]);
  }
  __syncthreads();
  product();
  start(reinterpret_cast<const bf16x8*>(r.Wf));
#pragma unroll
  for (int h = 0; h < TPW; ++h)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      if constexpr (!AHEAD) load_g(h, ct, gv[0][0]);
      const float2(&gq)[4] = gv[AHEAD ? h : 0][AHEAD ? ct : 0];
      const int k0 = (wv + h * nw) * 16 + 4 * quad;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float val = acc[h][ct][q];
        const float other = __shfl_xor(val, 1, 64);
        const float re = part ? other : val, im = part ? val : other;
        // one rounded product, then one fused step, spelled out: with single BF16 operands a different
        // last bit of t here and there already makes another refinement path
        const float pi = re * gq[q].y, pr = im * gq[q].y;
        const float out = part ? fmaf(im, gq[q].x, pi) : fmaf(re, gq[q].x, -pr);
        acc[h][ct][q] = live[ct] && k0 + q < M ? out : 0.f;
      }
      if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
    }
  __syncthreads();   // every wavefront has read Y (entries past the last row tile stay zero)
#pragma unroll
  for (int h = 0; h < TPW; ++h)
    if (wv + h * nw < nt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        bf16x4 hi, lo;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          __bf16 a, b;
          split_bf16(acc[h][ct][q], a, b);
          hi[q] = a;
          lo[q] = b;
        }
        const int tl = wv + h * nw;
        __bf16* d = T + (ct * 16 + rc) * KS + 32 * (tl >> 1) + 8 * quad + 4 * (tl & 1);
        *reinterpret_cast<bf16x4*>(d) = hi;
        if (SPLIT) *reinterpret_cast<bf16x4*>(d + RC * KS) = lo;
      }
  __syncthreads();
  product();
  float* so = reinterpret_cast<float*>(s_out);
#pragma unroll
  for (int h = 0; h < TPW; ++h)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = (wv + h * nw) * 16 + 4 * quad + q;
        if (live[ct] && i < M) so[2 * ((((size_t)jj[ct] * M + i) * nch + g) * B + cb[ct]) + part] = acc[h][ct][q];
      }
}

// fragment tables of nw M x M FP64 matrices: per (w, row tile, k step of 32) the 64 lanes' hi operands,
// then their lo operands, zero past M
__global__ void k_pack_bf16(int M, int nt, int ns, int nw, const double* __restrict__ A, bf16x8* __restrict__ F) {
  const int64_t n = (int64_t)nw * nt * ns * 64;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int l = (int)(t & 63);
  int64_t q = t >> 6;
  const int64_t base = q * 128 + l;
  const int s = (int)(q % ns);
  q /= ns;
  const int row = (int)(q % nt) * 16 + (l & 15), w = (int)(q / nt), k0 = 32 * s + 4 * (l >> 4);
  bf16x8 hi, lo;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int k = k0 + (u & 3) + 4 * (u & 4);
    const float v = row < M && k < M ? (float)A[((size_t)w * M + row) * M + k] : 0.f;
    __bf16 h, r;
    split_bf16(v, h, r);
    hi[u] = h;
    lo[u] = r;
  }
  F[base] = hi;
  F[base + 64] = lo;
}

hipError_t launch_pack_bf16(int M, int nw, const double* A, uint4* F, hipStream_t s) {
  if (M < 1 || nw < 1) return hipErrorInvalidValue;
  const int nt = (M + 15) / 16, ns = (M + 31) / 32;
  const int64_t n = (int64_t)nw * nt * ns * 64;
  hipLaunchKernelGGL(k_pack_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, M, nt, ns, nw, A,
                     reinterpret_cast<bf16x8*>(F));
  return hipGetLastError();
}

template <bool SPLIT, int CT, int TPW, int D>
static hipError_t launch_step_bf16_k(const RotArgsMixed& r, const float2* y, float2* s_out, int nt, int ns,
                                     hipStream_t s) {
  auto kern = k_step_bf16<SPLIT, CT, TPW, D>;
  const size_t lds = (size_t)(SPLIT ? 2 : 1) * 16 * CT * (32 * ns + 8) * 2;
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
          hipSuccess)
    return hipErrorInvalidValue;
  const dim3 grid((r.N * r.B + 8 * CT - 1) / (8 * CT), r.nch);
  hipLaunchKernelGGL(kern, grid, dim3(64 * ((nt + TPW - 1) / TPW)), lds, s, r, y, s_out, nt, ns);
  return hipGetLastError();
}

// Row tiles per wavefront: the fewest that leave at most 16 wavefronts.
template <bool SPLIT, int CT>
static hipError_t launch_step_bf16_ct(const RotArgsMixed& r, const float2* y, float2* s_out, hipStream_t s) {
  const int nt = (r.M + 15) / 16, ns = (r.M + 31) / 32;
  if (nt <= 16) return launch_step_bf16_k<SPLIT, CT, 1, 4>(r, y, s_out, nt, ns, s);
  if (nt <= 32) return launch_step_bf16_k<SPLIT, CT, 2, 2>(r, y, s_out, nt, ns, s);
  if constexpr (SPLIT) return hipErrorInvalidValue;   // more than 512 rows
  else return launch_step_bf16_k<false, 1, 4, 2>(r, y, s_out, nt, ns, s);
}

hipError_t launch_step_bf16(const RotArgsMixed& r, const float2* y, float2* s_out, hipStream_t s) {
  // split operands up to 512 rows, single ones up to 1024
  if (r.M < 1 || r.M > (r.split ? 512 : 1024) || r.N < 1 || r.B < 1 || r.nch < 1 || !r.G || !r.Of || !r.Wf)
    return hipErrorInvalidValue;
  // 16 columns per workgroup read the tables half as often as 8, which wins once the row tiles of all
  // workgroups fill the device (us, 8 / 16 columns, split): 2 channels, M = N = 100, 8 columns 8.7 / 10.1,
  // 16 columns (1400 row tiles) 10.9 / 10.5, 32 columns (2800) 16.0 / 12.8, 64 columns 24.6 / 20.2; 18 channels,
  // M = N = 150, 4 columns 37 / 30; 1 channel, M = 400, N = 300, 4 columns (1875) 22 / 29, 8 columns 38 / 30
  const bool wide = (int64_t)((r.N * r.B + 15) / 16) * r.nch * ((r.M + 15) / 16) >= 2400;
  if (r.split) return wide ? launch_step_bf16_ct<true, 2>(r, y, s_out, s) : launch_step_bf16_ct<true, 1>(r, y, s_out, s);
  return wide ? launch_step_bf16_ct<false, 2>(r, y, s_out, s) : launch_step_bf16_ct<false, 1>(r, y, s_out, s);
}

// ------------------------------------------------------------------ refinement helpers (FP64)

__global__ void k_cvt_d2f(int64_t n, const double2* __restrict__ in, float2* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

__global__ void k_cvt_scalar(int64_t n, const double* __restrict__ in, float* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (float)in[i];
}

hipError_t launch_cvt_scalar(int64_t n, const double* in, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_cvt_scalar, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, in, out);
  return hipGetLastError();
}

// the columns [c0, c1) of a [rows][B] array
__global__ void k_cvt_d2f_cols(int64_t rows, int B, int c0, int c1, const double2* __restrict__ in,
                               float2* __restrict__ out) {
  const int w = c1 - c0;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= rows * w) return;
  const int64_t d = t / w;
  const size_t i = (size_t)d * B + c0 + (int)(t - d * w);
  out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

hipError_t launch_cvt_d2f_cols(int64_t rows, int B, int c0, int c1, const double2* in, float2* out, hipStream_t s) {
  if (c0 < 0 || c1 > B || c0 >= c1) return hipErrorInvalidValue;
  const int64_t n = rows * (c1 - c0);
  hipLaunchKernelGGL(k_cvt_d2f_cols, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rows, B, c0, c1, in, out);
  return hipGetLastError();
}

hipError_t launch_cvt_d2f(int64_t n, const double2* in, float2* out, hipStream_t s) {
  hipLaunchKernelGGL(k_cvt_d2f, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, in, out);
  return hipGetLastError();
}

// r = b - y + Ky
__global__ void k_residual(int64_t n, const double2* __restrict__ b, const double2* __restrict__ y,
                           const double2* __restrict__ Ky, double2* __restrict__ r) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = make_double2(b[i].x - y[i].x + Ky[i].x, b[i].y - y[i].y + Ky[i].y);
}

hipError_t launch_residual(int64_t n, const double2* b, const double2* y, const double2* Ky, double2* r, hipStream_t s) {
  hipLaunchKernelGGL(k_residual, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, b, y, Ky, r);
  return hipGetLastError();
}

// out[d][c] += sum_m coef[m][c] * vecs[m][d][c] (complex coefficients, FP64 accumulation)
__global__ void k_lincomb(int64_t rows, int B, int nv, const float2* __restrict__ vecs, int64_t vstride,
                          const double2* __restrict__ coef, double2* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * B) return;
  const int c = (int)(i % B);
  double sr = 0.0, si = 0.0;
  for (int m = 0; m < nv; ++m) {
    const double2 w = coef[(size_t)m * B + c];
    if (w.x == 0.0 && w.y == 0.0) continue;
    const float2 v = vecs[(size_t)m * vstride + i];
    sr += w.x * v.x - w.y * v.y;
    si += w.x * v.y + w.y * v.x;
  }
  out[i] = make_double2(out[i].x + sr, out[i].y + si);
}

hipError_t launch_lincomb(int64_t rows, int B, int nv, const float2* vecs, int64_t vstride, const double2* coef,
                          double2* out, hipStream_t s) {
  if (vstride < rows * B) return hipErrorInvalidValue;
  const int64_t n = rows * B;
  hipLaunchKernelGGL(k_lincomb, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rows, B, nv, vecs, vstride, coef,
                     out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ Arnoldi (per column c)
// Vectors are [rows][B] float2 (rows = D lattice entries, row d = cell * nch + g); a basis is
// kept unnormalised, V_i = scl[i][c] * Vt_i, with the basis slots vstride apart. Every kernel
// below has lanes over 64 columns (blockIdx.y picks the column block) and waves striding over
// rows; FP64 partial sums per block are reduced in LDS and written to part[blk][i][c], which a
// wavefront-per-output pass sums in a fixed order (results do not depend on scheduling).

// Lane layout of the column kernels: with Bp = min(64, B rounded up to a power of two), lane l
// takes column blockIdx.y * 64 + l % Bp and row offset l / Bp, so a wavefront covers 64 / Bp rows
// per pass and no lane idles for small B.
struct ArnLanes {
  int Bp, R, cw, rsub, c;
  bool live;
};
__device__ __forceinline__ ArnLanes arn_lanes(int B) {
  ArnLanes a;
  const int lane = threadIdx.x & 63;
  const int bb = B - (int)blockIdx.y * 64;
  a.Bp = 64;
  if (bb < 64) {
    a.Bp = 1;
    while (a.Bp < bb) a.Bp <<= 1;
  }
  a.R = 64 / a.Bp;
  a.cw = lane % a.Bp;
  a.rsub = lane / a.Bp;
  a.c = (int)blockIdx.y * 64 + a.cw;
  a.live = a.c < B;
  return a;
}

// Sums the per-lane partials (hr, hi)[0 .. nv) of equal column over the lanes and waves of the
// block (fixed order: wave, then row offset) into part[blk][i][c].
template <int NV>
__device__ __forceinline__ void arn_block_reduce(const double (&hr)[NV], const double (&hi)[NV], int nv,
                                                 const ArnLanes& ln, int B, double2* __restrict__ part) {
  __shared__ double2 red[4][4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  static_assert(NV % 4 == 0, "partials are reduced four at a time");
#pragma unroll
  for (int i0 = 0; i0 < NV; i0 += 4) {
    if (i0 < nv) {   // uniform over the block
#pragma unroll
      for (int q = 0; q < 4; ++q) red[wv][q][lane] = make_double2(hr[i0 + q], hi[i0 + q]);
      __syncthreads();
      const int q = wv, i = i0 + wv, l = lane;
      const int c = (int)blockIdx.y * 64 + l;
      if (l < ln.Bp && i < nv && c < B) {
        double2 t = make_double2(0.0, 0.0);
        for (int w4 = 0; w4 < 4; ++w4)
          for (int r = 0; r < ln.R; ++r) {
            t.x += red[w4][q][r * ln.Bp + l].x;
            t.y += red[w4][q][r * ln.Bp + l].y;
          }
        part[((size_t)blockIdx.x * nv + i) * B + c] = t;
      }
      __syncthreads();
    }
  }
}

template <int NV>
__device__ __forceinline__ void arn_dot_row(const float2* __restrict__ V, int64_t vstride, int nv, size_t idx,
                                            float wr, float wi, double (&hr)[NV], double (&hi)[NV]) {
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    if (q < nv) {
      const float2 v = V[(size_t)q * vstride + idx];
      hr[q] += (double)v.x * wr + (double)v.y * wi;
      hi[q] += (double)v.x * wi - (double)v.y * wr;
    }
  }
}

// Fused Arnoldi product for B >= 16, nch <= 4: w = V_j - P0 t (block-CSR, lanes over columns,
// the nonzero blocks of a row taken four at a time so their gathers overlap), w stored in basis
// slot j + 1, and the partial sums of conj(Vt_i) w for i <= j.
template <int NC>
__global__ void __launch_bounds__(256) k_spmm_arn(int64_t cells, int B, const int64_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ col, const float* __restrict__ val,
                                                  const int32_t* __restrict__ order,
                                                  const float2* __restrict__ t, float2* __restrict__ V,
                                                  int64_t vstride, int j, const double* __restrict__ scl,
                                                  double2* __restrict__ part) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  ArnLanes ln;
  ln.Bp = 64;
  ln.R = 1;
  ln.cw = lane;
  ln.rsub = 0;
  ln.c = blockIdx.y * 64 + lane;
  ln.live = ln.c < B;
  const int c = ln.c;
  const bool live = ln.live;
  const int cl = live ? c : B - 1;
  const float2* Vj = V + (size_t)j * vstride;
  float2* Wo = V + (size_t)(j + 1) * vstride;
  const float sj = (float)scl[(size_t)j * B + cl];
  const int nv = j + 1;
  double hr[ARN_NV], hi[ARN_NV];
#pragma unroll
  for (int q = 0; q < ARN_NV; ++q) hr[q] = hi[q] = 0.0;
  for (int64_t rw = (int64_t)blockIdx.x * 4 + wv; rw < cells; rw += (int64_t)gridDim.x * 4) {
    const int64_t row = order ? order[rw] : rw;
    float ar[NC], ai[NC];
#pragma unroll
    for (int g = 0; g < NC; ++g) ar[g] = ai[g] = 0.f;
    const int64_t b0 = rowptr[row], b1 = rowptr[row + 1];
    int64_t e = b0;
    for (; e + 8 <= b1; e += 8) {   // eight blocks' gathers in flight; sums in block order
      int cc[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) cc[u] = col[e + u];
      float2 xv[8][NC];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int gp = 0; gp < NC; ++gp) xv[u][gp] = t[((size_t)cc[u] * NC + gp) * B + cl];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* v = val + (e + u) * NC * NC;
#pragma unroll
        for (int gp = 0; gp < NC; ++gp)
#pragma unroll
          for (int g = 0; g < NC; ++g) {
            const float a = v[gp * NC + g];
            ar[g] = fmaf(a, xv[u][gp].x, ar[g]);
            ai[g] = fmaf(a, xv[u][gp].y, ai[g]);
          }
      }
    }
    for (; e < b1; ++e) {
      const int cc = col[e];
      const float* v = val + e * NC * NC;
#pragma unroll
      for (int gp = 0; gp < NC; ++gp) {
        const float2 xv = t[((size_t)cc * NC + gp) * B + cl];
#pragma unroll
        for (int g = 0; g < NC; ++g) {
          const float a = v[gp * NC + g];
          ar[g] = fmaf(a, xv.x, ar[g]);
          ai[g] = fmaf(a, xv.y, ai[g]);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < NC; ++g) {
      const size_t idx = ((size_t)row * NC + g) * B + cl;
      const float2 v = Vj[idx];
      const float wr = sj * v.x - ar[g], wi = sj * v.y - ai[g];
      if (live) Wo[idx] = make_float2(wr, wi);
      arn_dot_row(V, vstride, nv, idx, wr, wi, hr, hi);
    }
  }
  arn_block_reduce(hr, hi, nv, ln, B, part);
}

// The same over 128-byte tiles of 16 columns, tile by tile over all rows, so that one tile of t stays in an
// XCD's L2 (as k_spmm): row_product on 16 lanes per row, rpw rows (a multiple of 16) per workgroup, and its own
// partial sums. With the finishing launch: M = N = 100, 2 channels, 64 columns 65 -> 52 us, 16 columns 62 -> 36;
// M = N = 60 40 -> 28 and 37 -> 19. In the unsplit mode k_spmm_arn keeps the order of its partial sums.
template <int NC, int NV, int U>
__global__ void __launch_bounds__(256) k_spmm_arn_tiles(int64_t cells, int B, int P, int rpw,
                                                        const int64_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col, const float* __restrict__ val,
                                                        const float2* __restrict__ t, float2* __restrict__ V,
                                                        int64_t vstride, int j, const double* __restrict__ scl,
                                                        double2* __restrict__ part) {
  constexpr int LW = 16;
  __shared__ double2 red[4][NV][LW];
  const int unit = xcd_unit(blockIdx.x, gridDim.x), tile = unit / P, p = unit - tile * P;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = tile * LW + (threadIdx.x & (LW - 1));
  const bool live = c < B;
  const int cl = live ? c : B - 1;
  const float2* Vj = V + (size_t)j * vstride;
  float2* Wo = V + (size_t)(j + 1) * vstride;
  const float sj = (float)scl[(size_t)j * B + cl];
  const int nv = j + 1;
  double hr[NV], hi[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) hr[q] = hi[q] = 0.0;
  const int64_t r1 = min(cells, (int64_t)(p + 1) * rpw);
  for (int64_t row = (int64_t)p * rpw + threadIdx.x / LW; row < r1; row += 256 / LW) {
    float2 acc[NC];
    row_product<NC, U, float, float, float2>(rowptr[row], rowptr[row + 1], col, val, t + cl, B, acc);
#pragma unroll
    for (int g = 0; g < NC; ++g) {
      const size_t idx = ((size_t)row * NC + g) * B + cl;
      const float2 v = Vj[idx];
      const float wr = sj * v.x - acc[g].x, wi = sj * v.y - acc[g].y;
      if (live) Wo[idx] = make_float2(wr, wi);
      arn_dot_row(V, vstride, nv, idx, wr, wi, hr, hi);
    }
  }
  // over the row groups of the wavefront, then over the wavefronts
#pragma unroll
  for (int q = 0; q < NV; ++q)
    if (q < nv) {
      for (int o = LW; o < 64; o <<= 1) {
        hr[q] += __shfl_xor(hr[q], o, 64);
        hi[q] += __shfl_xor(hi[q], o, 64);
      }
      if (lane < LW) red[wv][q][lane] = make_double2(hr[q], hi[q]);
    }
  __syncthreads();
  for (int k = threadIdx.x; k < nv * LW; k += 256) {
    const int q = k / LW, l = k - q * LW;
    if (tile * LW + l >= B) continue;
    double2 s = make_double2(0.0, 0.0);
    for (int w = 0; w < 4; ++w) {
      s.x += red[w][q][l].x;
      s.y += red[w][q][l].y;
    }
    part[((size_t)p * nv + q) * B + tile * LW + l] = s;
  }
}

// Unfused variant (any B, any nch): w = V_j - kv with kv = P0 t from the general SpMM.
// NV: basis slots held per lane (8 when the cycle has at most 8 Arnoldi steps, else ARN_NV): fewer
// registers, more waves in flight for these bandwidth-bound passes.
template <int NV>
__global__ void __launch_bounds__(256) k_sub_dots(int64_t rows, int B, const float2* __restrict__ kv,
                                                  float2* __restrict__ V, int64_t vstride, int j,
                                                  const double* __restrict__ scl, double2* __restrict__ part) {
  const int wv = threadIdx.x >> 6;
  const ArnLanes ln = arn_lanes(B);
  const int cl = ln.live ? ln.c : B - 1;
  const float2* Vj = V + (size_t)j * vstride;
  float2* Wo = V + (size_t)(j + 1) * vstride;
  const float sj = (float)scl[(size_t)j * B + cl];
  const int nv = j + 1;
  double hr[NV], hi[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) hr[q] = hi[q] = 0.0;
  const int64_t step = (int64_t)gridDim.x * 4 * ln.R;
  // two rows per pass, all their reads issued before the store (the output slot shares the basis
  // buffer, so the reads of a later row could not move above it); the sums take the rows in the
  // same order as one row per pass
  for (int64_t d = ((int64_t)blockIdx.x * 4 + wv) * ln.R + ln.rsub; d < rows; d += 2 * step) {
    const bool two = d + step < rows;
    const size_t i1 = (size_t)d * B + cl, i2 = (size_t)(two ? d + step : d) * B + cl;
    const float2 v1 = Vj[i1], k1 = kv[i1], v2 = Vj[i2], k2 = kv[i2];
    float2 b1[NV], b2[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q)
      if (q < nv) {
        b1[q] = V[(size_t)q * vstride + i1];
        b2[q] = V[(size_t)q * vstride + i2];
      }
    const float w1r = sj * v1.x - k1.x, w1i = sj * v1.y - k1.y;
    const float w2r = sj * v2.x - k2.x, w2i = sj * v2.y - k2.y;
    if (ln.live) {
      Wo[i1] = make_float2(w1r, w1i);
      if (two) Wo[i2] = make_float2(w2r, w2i);
#pragma unroll
      for (int q = 0; q < NV; ++q)
        if (q < nv) {
          hr[q] += (double)b1[q].x * w1r + (double)b1[q].y * w1i;
          hi[q] += (double)b1[q].x * w1i - (double)b1[q].y * w1r;
        }
      if (two) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
          if (q < nv) {
            hr[q] += (double)b2[q].x * w2r + (double)b2[q].y * w2i;
            hi[q] += (double)b2[q].x * w2i - (double)b2[q].y * w2r;
          }
      }
    }
  }
  arn_block_reduce(hr, hi, nv, ln, B, part);
}

// w -= sum_{i <= j} h_i V_i (FP64 arithmetic, FP32 storage) in basis slot j + 1, with the partial
// sums of |w|^2 of the stored values.
template <int NV>
__global__ void __launch_bounds__(256) k_orth_norm(int64_t rows, int B, float2* __restrict__ V, int64_t vstride, int j,
                                                   const double2* __restrict__ h, const double* __restrict__ scl,
                                                   double2* __restrict__ part) {
  const int wv = threadIdx.x >> 6;
  const ArnLanes ln = arn_lanes(B);
  const int cl = ln.live ? ln.c : B - 1;
  const int nv = j + 1;
  double cr[NV], ci[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    cr[q] = ci[q] = 0.0;
    if (q < nv) {
      const double sc = scl[(size_t)q * B + cl];
      cr[q] = h[(size_t)q * B + cl].x * sc;
      ci[q] = h[(size_t)q * B + cl].y * sc;
    }
  }
  float2* Wo = V + (size_t)(j + 1) * vstride;
  double acc[4], dummy[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = dummy[q] = 0.0;
  const int64_t step = (int64_t)gridDim.x * 4 * ln.R;
  // two rows per pass, their reads before the stores, sums in row order (as in k_sub_dots)
  for (int64_t d = ((int64_t)blockIdx.x * 4 + wv) * ln.R + ln.rsub; d < rows; d += 2 * step) {
    if (!ln.live) continue;
    const bool two = d + step < rows;
    const size_t i1 = (size_t)d * B + cl, i2 = (size_t)(two ? d + step : d) * B + cl;
    const float2 w1 = Wo[i1], w2 = Wo[i2];
    float2 b1[NV], b2[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q)
      if (q < nv) {
        b1[q] = V[(size_t)q * vstride + i1];
        b2[q] = V[(size_t)q * vstride + i2];
      }
    double x1r = w1.x, x1i = w1.y, x2r = w2.x, x2i = w2.y;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      if (q < nv) {
        x1r -= cr[q] * b1[q].x - ci[q] * b1[q].y;
        x1i -= cr[q] * b1[q].y + ci[q] * b1[q].x;
        x2r -= cr[q] * b2[q].x - ci[q] * b2[q].y;
        x2i -= cr[q] * b2[q].y + ci[q] * b2[q].x;
      }
    }
    const float2 o1 = make_float2((float)x1r, (float)x1i), o2 = make_float2((float)x2r, (float)x2i);
    Wo[i1] = o1;
    acc[0] += (double)o1.x * o1.x + (double)o1.y * o1.y;
    if (two) {
      Wo[i2] = o2;
      acc[0] += (double)o2.x * o2.x + (double)o2.y * o2.y;
    }
  }
  arn_block_reduce(acc, dummy, 1, ln, B, part);
}

__device__ __forceinline__ double wsum64(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wavefront per output (i, c), lanes over the blocks in a fixed order; a lane's partials (at most
// ARN_MAXBLK / 64) are all read before they are added (one after another they cost 16 memory latencies,
// 7 us a launch; 3 us now).
// mode 0: out[i][c] = scl[i][c] * sum_blk part[blk][i][c]       (Hessenberg column, i < nv)
// mode 1: n = sqrt(sum_blk part[blk][0][c].x); out[0][c] = n;    (subdiagonal entry)
//         scl_next[c] = 1 / n (0 for a zero vector)
#define ARN_MAXBLK 1024
template <int PL>
__global__ void __launch_bounds__(256) k_arn_finish(int nblk, int B, int nv, const double2* __restrict__ part,
                                                    const double* __restrict__ scl, double2* __restrict__ out,
                                                    double* __restrict__ scl_next, int mode) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= nv * B) return;
  const int i = t / B, c = t - i * B;
  double2 v[PL];
#pragma unroll
  for (int u = 0; u < PL; ++u) {
    const int b = lane + 64 * u;
    v[u] = b < nblk ? part[((size_t)b * nv + i) * B + c] : make_double2(0.0, 0.0);
  }
  double sr = 0.0, si = 0.0;
#pragma unroll
  for (int u = 0; u < PL; ++u) {
    sr += v[u].x;
    si += v[u].y;
  }
  sr = wsum64(sr);
  si = wsum64(si);
  if (lane == 0) {
    if (mode == 0) {
      const double sc = scl ? scl[(size_t)i * B + c] : 1.0;
      out[t] = make_double2(sr * sc, si * sc);
    } else {
      const double n = sqrt(fmax(sr, 0.0));
      out[c] = make_double2(n, 0.0);
      scl_next[c] = n > 1e-300 ? 1.0 / n : 0.0;
    }
  }
}

static void arn_finish(int nblk, int B, int nv, const double2* part, const double* scl, double2* out, double* scl_next,
                       int mode, hipStream_t s) {
  const dim3 g((nv * B + 3) / 4), b(256);
  if (nblk <= 64) hipLaunchKernelGGL(k_arn_finish<1>, g, b, 0, s, nblk, B, nv, part, scl, out, scl_next, mode);
  else if (nblk <= 256) hipLaunchKernelGGL(k_arn_finish<4>, g, b, 0, s, nblk, B, nv, part, scl, out, scl_next, mode);
  else hipLaunchKernelGGL(k_arn_finish<16>, g, b, 0, s, nblk, B, nv, part, scl, out, scl_next, mode);
}

// Workgroups of a column reduction over `rows` rows: as many as the rows fill with `per` rows per
// wavefront, at most nblk. The partial sums follow the grid, so the unsplit mode keeps one (per = 1, up to
// 64 times the rows a wavefront holds on few columns: 1024 partials where 112 hold every row).
static dim3 arn_grid(int64_t rows, int B, int nblk, int per) {
  const int64_t need = (rows + 4 * per - 1) / (4 * per);
  return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(std::min(nblk, ARN_MAXBLK), need)), (unsigned)((B + 63) / 64));
}
// rows a wavefront takes per pass of the Gram-Schmidt kernels: two for every group of lanes (arn_lanes)
static int arn_rows(int B) {
  int bp = 1;
  while (bp < B && bp < 64) bp <<= 1;
  return 2 * (64 / bp);
}

template <int NC>
static void spmm_arn_launch(dim3 grid, hipStream_t s, int64_t cells, int B, const int64_t* rowptr, const int32_t* col,
                            const float* val, const int32_t* order, const float2* t, float2* V, int64_t vstride, int j,
                            const double* scl, double2* part) {
  hipLaunchKernelGGL(k_spmm_arn<NC>, grid, dim3(256), 0, s, cells, B, rowptr, col, val, order, t, V, vstride, j, scl,
                     part);
}

hipError_t launch_arnoldi_product(const ArnoldiArgs& a, const float2* t, float2* kv_scratch, hipStream_t s) {
  if (a.j < 0 || a.j + 1 >= ARN_NV + 1 || a.j >= a.m || a.B < 1 || a.nch < 1 || a.vstride < a.cells * a.nch * a.B)
    return hipErrorInvalidValue;
  const int64_t rows = a.cells * a.nch;
  if (a.B >= 16 && a.nch <= 4) {
    ProfScope ps("spmm_arnoldi", s);
    int nb;
    if (!a.split) {
      const dim3 grid = arn_grid(a.cells, a.B, a.nblk, 1);
      switch (a.nch) {
        case 1: spmm_arn_launch<1>(grid, s, a.cells, a.B, a.rowptr, a.col, a.val, a.order, t, a.V, a.vstride, a.j, a.scl, a.part); break;
        case 2: spmm_arn_launch<2>(grid, s, a.cells, a.B, a.rowptr, a.col, a.val, a.order, t, a.V, a.vstride, a.j, a.scl, a.part); break;
        case 3: spmm_arn_launch<3>(grid, s, a.cells, a.B, a.rowptr, a.col, a.val, a.order, t, a.V, a.vstride, a.j, a.scl, a.part); break;
        default: spmm_arn_launch<4>(grid, s, a.cells, a.B, a.rowptr, a.col, a.val, a.order, t, a.V, a.vstride, a.j, a.scl, a.part); break;
      }
      nb = (int)grid.x;
    } else {
      // rows per workgroup: 16 on small lattices (M = N = 60 28 us, 31 with 32), else 32 (M = N = 100 52 and 59
      // with 16), more where that leaves more partial sums than there is room for
      const int most = std::min(a.nblk, ARN_MAXBLK);
      int rpw = a.cells <= 4096 ? 16 : 32;
      while ((a.cells + rpw - 1) / rpw > most) rpw += 16;
      nb = (int)((a.cells + rpw - 1) / rpw);
      const unsigned wgs = (unsigned)nb * ((a.B + 15) / 16);
      // 8 blocks in flight per row while the workgroups fit the registers at once (4 per compute unit with 2
      // channels), else 4 (2 channels, 64 columns 61 -> 52 us; 1 channel, with registers to spare, 30 and 33)
      const bool deep = a.m <= 8 && (a.nch == 1 || wgs <= 1024);
#define WP_TILES(NC, NV, U)                                                                                          \
  hipLaunchKernelGGL((k_spmm_arn_tiles<NC, NV, U>), dim3(wgs), dim3(256), 0, s, a.cells, a.B, nb, rpw, a.rowptr, a.col, \
                     a.val, t, a.V, a.vstride, a.j, a.scl, a.part)
#define WP_TILES_NC(NC)                       \
  if (deep) WP_TILES(NC, 8, 8);               \
  else if (a.m <= 8) WP_TILES(NC, 8, 4);      \
  else WP_TILES(NC, ARN_NV, 4)
      switch (a.nch) {
        case 1: WP_TILES_NC(1); break;
        case 2: WP_TILES_NC(2); break;
        case 3: WP_TILES_NC(3); break;
        default: WP_TILES_NC(4); break;
      }
#undef WP_TILES_NC
#undef WP_TILES
    }
    arn_finish(nb, a.B, a.j + 1, a.part, a.scl, a.H + (size_t)a.j * (a.m + 1) * a.B, nullptr, 0, s);
  } else {
    if (!kv_scratch) return hipErrorInvalidValue;
    {
      ProfScope ps("spmv_f32", s);
      hipError_t e = launch_spmv_f32(a.cells, a.nch, a.B, a.rowptr, a.col, a.val, t, kv_scratch, s, 0, -1, a.order, a.pk);
      if (e != hipSuccess) return e;
    }
    ProfScope ps("arnoldi_dots", s);
    const dim3 grid = arn_grid(rows, a.B, a.nblk, a.split ? arn_rows(a.B) : 1);
    if (a.m <= 8)
      hipLaunchKernelGGL(k_sub_dots<8>, grid, dim3(256), 0, s, rows, a.B, kv_scratch, a.V, a.vstride, a.j, a.scl, a.part);
    else
      hipLaunchKernelGGL(k_sub_dots<ARN_NV>, grid, dim3(256), 0, s, rows, a.B, kv_scratch, a.V, a.vstride, a.j, a.scl,
                         a.part);
    arn_finish((int)grid.x, a.B, a.j + 1, a.part, a.scl, a.H + (size_t)a.j * (a.m + 1) * a.B, nullptr, 0, s);
  }
  return hipGetLastError();
}

hipError_t launch_arnoldi_orth(const ArnoldiArgs& a, hipStream_t s) {
  if (a.j < 0 || a.j + 1 > ARN_NV || a.j + 1 > a.m) return hipErrorInvalidValue;
  const int64_t rows = a.cells * a.nch;
  const dim3 grid = arn_grid(rows, a.B, a.nblk, a.split ? arn_rows(a.B) : 1);
  const double2* hcol = a.H + (size_t)a.j * (a.m + 1) * a.B;
  if (a.m <= 8)
    hipLaunchKernelGGL(k_orth_norm<8>, grid, dim3(256), 0, s, rows, a.B, a.V, a.vstride, a.j, hcol, a.scl, a.part);
  else
    hipLaunchKernelGGL(k_orth_norm<ARN_NV>, grid, dim3(256), 0, s, rows, a.B, a.V, a.vstride, a.j, hcol, a.scl, a.part);
  arn_finish((int)grid.x, a.B, 1, a.part, a.scl, a.H + ((size_t)a.j * (a.m + 1) + a.j + 1) * a.B,
             a.scl + (size_t)(a.j + 1) * a.B, 1, s);
  return hipGetLastError();
}

// U[c][f] = e0^T O y at (g = finals[f], j = j0[c], k = 0): one wavefront per (c, f), lanes over i.
__global__ void __launch_bounds__(256) k_capture64(int M, int nch, int B, int nfin, const double* __restrict__ O,
                                                   const int* __restrict__ wave, const int* __restrict__ j0,
                                                   const int* __restrict__ finals, const double2* __restrict__ y,
                                                   double2* __restrict__ out) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= B * nfin) return;
  const int c = t / nfin, f = t - c * nfin;
  const int g = finals[f];
  const double* o = O + (size_t)wave[g] * M * M;   // row k = 0
  double sr = 0.0, si = 0.0;
  for (int i = lane; i < M; i += 64) {
    const double2 v = y[(((size_t)j0[c] * M + i) * nch + g) * B + c];
    sr += o[i] * v.x;
    si += o[i] * v.y;
  }
  sr = wsum64(sr);
  si = wsum64(si);
  if (lane == 0) out[t] = make_double2(sr, si);
}

// Breakup projections (one wavefront per cell): out[t] = sum_i O[wave(g)][k][i] y[((j M + i) nch + g) B + c]
// for cell t = (c, g, k, j), the pair pseudostate k of channel g at spectator bin j.
__global__ void __launch_bounds__(256) k_project_cells(int M, int nch, int B, const double* __restrict__ O,
                                                       const int* __restrict__ wave, const int4* __restrict__ cells,
                                                       int n, const double2* __restrict__ y,
                                                       double2* __restrict__ out) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= n) return;
  const int4 cl = cells[t];
  const int c = cl.x, g = cl.y, k = cl.z, j = cl.w;
  const double* o = O + ((size_t)wave[g] * M + k) * M;
  double sr = 0.0, si = 0.0;
  for (int i = lane; i < M; i += 64) {
    const double2 v = y[(((size_t)j * M + i) * nch + g) * B + c];
    sr += o[i] * v.x;
    si += o[i] * v.y;
  }
  sr = wsum64(sr);
  si = wsum64(si);
  if (lane == 0) out[t] = make_double2(sr, si);
}

hipError_t launch_project_cells(int M, int nch, int B, const double* O, const int* wave, const int4* cells, int n,
                                const double2* y, double2* out, hipStream_t s) {
  if (M < 1 || B < 1 || n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_project_cells, dim3((n + 3) / 4), dim3(256), 0, s, M, nch, B, O, wave, cells, n, y, out);
  return hipGetLastError();
}

hipError_t launch_capture64(int M, int nch, int B, int nfin, const double* O, const int* wave, const int* j0,
                            const int* finals, const double2* y, double2* out, hipStream_t s) {
  if (M < 1 || B < 1 || nfin < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_capture64, dim3((B * nfin + 3) / 4), dim3(256), 0, s, M, nch, B, nfin, O, wave, j0, finals, y,
                     out);
  return hipGetLastError();
}

// FP64 residual -> squared norms per column (FP64)
__global__ void __launch_bounds__(256) k_norm2_f64(int64_t rows, int B, const double2* __restrict__ x,
                                                   double2* __restrict__ part) {
  const int wv = threadIdx.x >> 6;
  const ArnLanes ln = arn_lanes(B);
  double acc[4], dummy[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = dummy[q] = 0.0;
  const int64_t step = (int64_t)gridDim.x * 4 * ln.R;
  if (ln.live)
    for (int64_t d = ((int64_t)blockIdx.x * 4 + wv) * ln.R + ln.rsub; d < rows; d += step) {
      const double2 v = x[(size_t)d * B + ln.c];
      acc[0] += v.x * v.x + v.y * v.y;
    }
  arn_block_reduce(acc, dummy, 1, ln, B, part);
}

hipError_t launch_norm2_f64(int64_t rows, int B, const double2* x, double2* part, int nblk, bool one_order, double2* out,
                            hipStream_t s) {
  const dim3 grid = arn_grid(rows, B, nblk, one_order ? 1 : arn_rows(B));
  hipLaunchKernelGGL(k_norm2_f64, grid, dim3(256), 0, s, rows, B, x, part);
  arn_finish((int)grid.x, B, 1, part, nullptr, out, nullptr, 0, s);
  return hipGetLastError();
}

__global__ void k_export_cycle(int B, int nH, int nS, const double2* __restrict__ nrm, const double2* __restrict__ H,
                               const double* __restrict__ scl, double2* __restrict__ hn, double2* __restrict__ hH,
                               double* __restrict__ hsc) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < B) hn[t] = nrm[t];
  if (t < nH) hH[t] = H[t];
  if (t < nS) hsc[t] = scl[t];
}
hipError_t launch_export_cycle(int B, int m, const double2* nrm, const double2* H, const double* scl, double2* hn,
                               double2* hH, double* hsc, hipStream_t s) {
  const int nH = m * (m + 1) * B, nS = (m + 1) * B;   // m >= 1: the Hessenberg entries are the most
  hipLaunchKernelGGL(k_export_cycle, dim3((std::max(nH, nS) + 255) / 256), dim3(256), 0, s, B, nH, nS, nrm, H, scl, hn,
                     hH, hsc);
  return hipGetLastError();
}

// out[d][c] = x[d][c] / sqrt(nrm2[c]) with x in FP64, out in FP32
__global__ void k_scale_d2f(int64_t n, int B, const double2* __restrict__ nrm2, const double2* __restrict__ x,
                            float2* __restrict__ out, double* __restrict__ scl0) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int c = (int)(t % B);
  if (scl0 && t < B) scl0[t] = 1.0;
  const double nr = sqrt(fmax(nrm2[c].x, 0.0));
  const double inv = nr > 1e-300 ? 1.0 / nr : 0.0;
  out[t] = make_float2((float)(x[t].x * inv), (float)(x[t].y * inv));
}

hipError_t launch_scale_d2f(int64_t rows, int B, const double2* nrm2, const double2* x, float2* out, double* scl0,
                            hipStream_t s) {
  const int64_t n = rows * B;
  hipLaunchKernelGGL(k_scale_d2f, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, B, nrm2, x, out, scl0);
  return hipGetLastError();
}

}  // namespace wpcd
