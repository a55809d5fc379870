// One block row of P0 times complex vectors, 16 lanes (a DPP row) over a tile of columns.
#pragma once
#include <hip/hip_runtime.h>

namespace wpcd {

// the value of lane N of each row of 16 lanes
template <int N>
__device__ __forceinline__ int row_bcast(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(row_bcast<N>(__float_as_int(v)));
}
template <int N>
__device__ __forceinline__ double row_bcast(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = row_bcast<N>((int)b), hi = row_bcast<N>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <typename AT, typename E> __device__ __forceinline__ void fma_to(AT a, E v, E& s);
template <> __device__ __forceinline__ void fma_to(float a, float2 v, float2& s) {
  s.x = fmaf(a, v.x, s.x);
  s.y = fmaf(a, v.y, s.y);
}
template <> __device__ __forceinline__ void fma_to(double a, double2 v, double2& s) {
  s.x = fma(a, v.x, s.x);
  s.y = fma(a, v.y, s.y);
}

template <int NC, typename VT, typename AT, typename E, int U, int u, bool ALL, int R>
__device__ __forceinline__ void row_block(const VT (&v)[R], const E (&xv)[U][NC], E (&acc)[NC], int left) {
  if constexpr (u < U) {
    if (ALL || u < left) {
#define WP_RB(GP, G)                                                                              \
  if constexpr (GP < NC && G < NC) {                                                              \
    constexpr int n = (u * NC + GP) * NC + G;                                                     \
    fma_to<AT, E>((AT)row_bcast<n % 16>(v[n / 16]), xv[u][GP], acc[G]);                           \
  }
      WP_RB(0, 0) WP_RB(0, 1) WP_RB(0, 2) WP_RB(0, 3) WP_RB(1, 0) WP_RB(1, 1) WP_RB(1, 2) WP_RB(1, 3)
      WP_RB(2, 0) WP_RB(2, 1) WP_RB(2, 2) WP_RB(2, 3) WP_RB(3, 0) WP_RB(3, 1) WP_RB(3, 2) WP_RB(3, 3)
#undef WP_RB
      row_block<NC, VT, AT, E, U, u + 1, ALL>(v, xv, acc, left);
    }
  }
}
__device__ __forceinline__ void keep_loaded(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }
__device__ __forceinline__ void keep_loaded(double2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

template <int NC, typename E, int U, int u>
__device__ __forceinline__ void row_gather(int cols, const E* __restrict__ x, int64_t ld, E (&xv)[U][NC]) {
  if constexpr (u < U) {
    const E* p = x + (int64_t)row_bcast<u>(cols) * NC * ld;
#pragma unroll
    for (int gp = 0; gp < NC; ++gp) xv[u][gp] = p[gp * ld];
    row_gather<NC, E, U, u + 1>(cols, x, ld, xv);
  }
}

// acc[g] = sum over the blocks e in [b0, b1) and g' of val[e][g'][g] x[(col[e] NC + g') ld], x pointing at the
// lane's column, in block order. The 16 lanes read U blocks' columns and values once, one element each, and
// pass them on by row broadcasts: read by every lane, the values cost the address unit as much as the
// gathers. U blocks' gathers are in flight, and the next U columns. b0 and b1 are the same in the 16 lanes,
// all of which are active.
template <int NC, int U, typename VT, typename AT, typename E>
__device__ __forceinline__ void row_product(int64_t b0, int64_t b1, const int32_t* __restrict__ col,
                                            const VT* __restrict__ val, const E* __restrict__ x, int64_t ld,
                                            E (&acc)[NC]) {
  static_assert(U <= 16 && NC <= 4, "columns of a turn: one per lane");
  constexpr int N2 = NC * NC, R = (U * N2 + 15) / 16;
  const int l = threadIdx.x & 15;
#pragma unroll
  for (int g = 0; g < NC; ++g) acc[g] = E{};
  if (b0 >= b1) return;
  int cols = col[min(b0 + l % U, b1 - 1)];
  VT v[R];
  E xv[U][NC];
  int64_t e = b0;
  for (; e + U <= b1; e += U) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = val[min(e * N2 + 16 * r + l, b1 * N2 - 1)];
    row_gather<NC, E, U, 0>(cols, x, ld, xv);
    cols = col[min(e + U + l % U, b1 - 1)];
    row_block<NC, VT, AT, E, U, 0, true, R>(v, xv, acc, U);
  }
  if (e < b1) {   // the last blocks; the gathers past them repeat the last one
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = val[min(e * N2 + 16 * r + l, b1 * N2 - 1)];
    row_gather<NC, E, U, 0>(cols, x, ld, xv);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int gp = 0; gp < NC; ++gp) keep_loaded(xv[u][gp]);   // here, not block by block below
    row_block<NC, VT, AT, E, U, 0, false, R>(v, xv, acc, (int)(b1 - e));
  }
}

}  // namespace wpcd
