// wide2d_kernel.hpp -- one level of a wide 2D box (radius 3 or 4): one wave per
// tile, U rows per step.
//
// Same contract, same tiles and the same per-cell arithmetic as march2d_kernel
// (each output's FMA chain starts from +0 and runs over the points in
// lexicographic order), so the two give identical bits.  One level of 49 or 81
// points is bound by the multiply-adds, and a march of one row per step loses
// a third of their rate at the sizes of a chunk:
//   * the weights do not fit the scalar registers beside the march's own state
//     (81 FP32 weights of 102 registers; 49 FP64 ones take 98), so that every
//     row waits for scalar loads or reads spilled lanes (FP64: more of those
//     than multiply-adds);
//   * every segment runs its first and last 2R rows for outputs that are not its
//     own, 8 of 49 rows where a chunk of 3360 rows fills the chip.
// Here a step takes U input rows and runs over the rows of weights: 2R+1
// weights stay in scalar registers for U VX (2R+1) multiply-adds per lane
// while the next row of weights is loaded, and a row of weights none of whose
// outputs belongs to the segment is skipped as a whole.  2R + U rows of partial
// sums move down by U rows once per step (2R VX moves against U VX (2R+1)^2
// multiply-adds).
// Measured on MI355X, us per level, the march against this (12800 x 3360 and
// 1201 x 1003; 73 TFLOP/s is what FP32 multiply-adds reach at four waves per
// SIMD): FP32 radius 4 148 and 27 against 123 and 12 (57 TFLOP/s; 62 on
// 12800 x 12800), radius 3 90 and 20 against 87 and 8 (reads and writes at
// 4 TB/s of 5.6); FP64 radius 4 276 and 28 against 178 and 13, radius 3 171 and
// 18 against 151 and 11.  U = 2, 3, 4 and 5 lie within 4 % of one another, and
// two cells per lane (four in FP64) within 8 %.
#pragma once
#include <cstddef>

#include "march2d_kernel.hpp"

namespace so2dr {

// The launch's weights in the kernel argument block, for scalar loads that
// stay where they are written: through the pointer the compiler sees, it would
// load all of them ahead of the march and spill.
template <typename A>
using ScalarPtr = const __attribute__((address_space(4))) A *;

template <typename T, int R, int VX, int U, int EDGE>
__device__ __forceinline__ void wide2d_tile(const TbArgs<typename Store<T>::A> &a,
                                            ScalarPtr<typename Store<T>::A> w, int lane, int x_lo, int zo0, int zo1) {
  using A = typename Store<T>::A;
  using G = RowTile<R, 1, VX>;
  constexpr int W = 2 * R + 1, NA = 2 * R + U;
  const int n_axis = (int)a.n_axis;
  const int p_lo = max((int)a.in_lo, 0), p_hi = min((int)a.in_hi, n_axis) - 1;
  const T *__restrict__ in = static_cast<const T *>(a.in);
  T *__restrict__ out = static_cast<T *>(a.out);

  // columns as in march2d_tile
  const int cx0 = lane * VX;
  const int gx0 = x_lo + cx0;
  constexpr int NV = EDGE == kEdgeCells ? VX : 1;
  uint32_t boff[NV];
  bool keep[NV], st[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int gx = gx0 + j;
    keep[j] = !EDGE || (gx >= 0 && gx < a.nx) || a.per_x;
    boff[j] = (uint32_t)(EDGE ? row_source(gx, a.nx, VX / NV, a.per_x) : gx) * (uint32_t)sizeof(T);
    st[j] = cx0 >= G::HX && cx0 < G::TX - G::HX && (!EDGE || gx < a.nx);
  }

  auto load_row = [&](int p, A *dst) {
    const int pc = min(max(p, p_lo), p_hi);
    const char *base = reinterpret_cast<const char *>(in + (int64_t)(pc - (int)a.buf_z0) * a.plane);
    if constexpr (EDGE != kEdgeCells) {
      VecIO<T, VX>::load(reinterpret_cast<const T *>(base + boff[0]), dst);
    } else {
#pragma unroll
      for (int j = 0; j < VX; ++j) dst[j] = Store<T>::load(reinterpret_cast<const T *>(base + boff[j]));
    }
  };

  A acc[NA][VX];    // acc[k]: output row i0 - R + k of the step that starts at row i0
  A cur[U][VX];     // the step's rows
#pragma unroll
  for (int k = 0; k < NA; ++k)
#pragma unroll
    for (int j = 0; j < VX; ++j) acc[k][j] = A(0);
#pragma unroll
  for (int u = 0; u < U; ++u) load_row(zo0 - R + u, cur[u]);

  for (int i0 = zo0 - R; i0 < zo1 + R; i0 += U) {
    A row[U][VX + 2 * R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool zg = EDGE != kInside && (i0 + u < 0 || i0 + u >= n_axis);
#pragma unroll
      for (int j = 0; j < VX; ++j) row[u][R + j] = EDGE == kInside || (keep[j % NV] && !zg) ? cur[u][j] : A(0);
    }
    A next[U][VX];
#pragma unroll
    for (int u = 0; u < U; ++u) load_row(i0 + U + u, next[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 1; k <= R; ++k) {
        const int sh = (k + VX - 1) / VX;
        const A lv = row[u][R + VX * sh - k], rv = row[u][R + k - 1 - VX * (sh - 1)];
        row[u][R - k] = sh == 1 ? dpp_f<kDppWaveShr1>(lv) : dpp_f<kDppWaveShr1>(dpp_f<kDppWaveShr1>(lv));
        row[u][R + VX - 1 + k] = sh == 1 ? dpp_f<kDppWaveShl1>(rv) : dpp_f<kDppWaveShl1>(dpp_f<kDppWaveShl1>(rv));
      }
    asm volatile("" : "+s"(w));   // this step's own loads of the weights
    A wc[W], wn[W];
#pragma unroll
    for (int k = 0; k < W; ++k) wc[k] = w[k];
#pragma unroll
    for (int dy = -R; dy <= R; ++dy) {
      if (dy < R) {
#pragma unroll
        for (int k = 0; k < W; ++k) wn[k] = w[(dy + 1 + R) * W + k];
      }
      __builtin_amdgcn_sched_barrier(0);
      if (i0 + U - 1 - dy >= zo0 && i0 - dy < zo1) {   // outputs i0 - dy .. i0 - dy + U - 1
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < VX; ++j) {
            A sum = dy == -R ? A(0) : acc[u - dy + R][j];
#pragma unroll
            for (int k = 0; k < W; ++k) sum = fma_(wc[k], row[u][j + k], sum);
            acc[u - dy + R][j] = sum;
          }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < W; ++k) wc[k] = wn[k];
    }
    // the next rows have arrived by now: waiting for them here, and not behind
    // the stores, leaves those in flight
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < VX; ++j) {
        cur[u][j] = next[u][j];
        asm volatile("" : "+v"(cur[u][j]));
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = i0 - R + u;
      if (!(st[0] && q >= zo0 && q < zo1)) continue;
      A res[VX];
#pragma unroll
      for (int j = 0; j < VX; ++j) res[j] = Store<T>::round(acc[u][j]);
      char *dst = reinterpret_cast<char *>(out + (int64_t)(q - (int)a.out_z0) * a.plane);
      if constexpr (EDGE != kEdgeCells) {
        VecIO<T, VX>::store(reinterpret_cast<T *>(dst + boff[0]), res);
      } else {
#pragma unroll
        for (int j = 0; j < VX; ++j)
          if (st[j]) Store<T>::store(reinterpret_cast<T *>(dst + boff[j]), res[j]);
      }
    }
#pragma unroll
    for (int k = 0; k + U < NA; ++k)
#pragma unroll
      for (int j = 0; j < VX; ++j) acc[k][j] = acc[k + U][j];
  }
}

template <typename T, int R, int VX, int U>
__global__ __launch_bounds__(64 * kRowWaves) void wide2d_kernel(const TbArgs<typename Store<T>::A> a) {
  using A = typename Store<T>::A;
  using G = RowTile<R, 1, VX>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntask = a.ntx * a.nseg;
  const int wg = xcd_tile(blockIdx.x, (ntask + kRowWaves - 1) / kRowWaves);
  if (wg < 0) return;
  const int task = wg * kRowWaves + wave;
  if (task >= ntask) return;
  const int tx_i = task % a.ntx, seg = task / a.ntx;
  const int zo0 = (int)a.out_lo + seg * (int)a.zseg;
  if (zo0 >= (int)a.out_hi) return;
  const int zo1 = min(zo0 + (int)a.zseg, (int)a.out_hi);
  const auto [x_lo, cells] = row_start<G, VX>(tx_i, a.nx);
  ScalarPtr<A> w = (ScalarPtr<A>)((ScalarPtr<char>)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(TbArgs<A>, w));
  const bool edge = x_lo < 0 || x_lo + G::TX > a.nx || zo0 - R < 0 || zo1 + R > (int)a.n_axis;
  if (!edge)
    wide2d_tile<T, R, VX, U, kInside>(a, w, lane, x_lo, zo0, zo1);
  else if (!cells)
    wide2d_tile<T, R, VX, U, kEdge>(a, w, lane, x_lo, zo0, zo1);
  else
    wide2d_tile<T, R, VX, U, kEdgeCells>(a, w, lane, x_lo, zo0, zo1);
}

}  // namespace so2dr
