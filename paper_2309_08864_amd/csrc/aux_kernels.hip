// aux_kernels.hip -- FP64 reductions of the adjoint (loss and weight
// gradients).  Not in the paper: the gradient of L = 1/2 ||u_T - y||^2 with
// respect to the weights is sum_t sum_x lambda_{t+1}(x) u_t(x + o_k), and the
// loss itself; both are accumulated in FP64 on the GPU.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "aux.hpp"
#include "launch.hpp"
#include "tb_kernel.hpp"
#include "../../include/so2dr.h"

namespace so2dr {

constexpr int kRedThreads = 256;

template <typename T>
__device__ __forceinline__ double to_d(T v) { return (double)v; }

__device__ __forceinline__ double block_sum(double v, double *red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = kRedThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// Device-to-device copy on the caller's stream, by a kernel of our own (large
// region-sharing halos, the adjoint's last buffer): 16-byte accesses where both
// ends allow, else 4 or 1.
template <typename W>
__global__ __launch_bounds__(256) void dcopy_kernel(W *__restrict__ dst, const W *__restrict__ src, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

int launch_dcopy(void *dst, const void *src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return 0;
  const uintptr_t a = (uintptr_t)dst | (uintptr_t)src;
  if (a % 16 == 0 && bytes % 16 == 0) {
    hipLaunchKernelGGL(dcopy_kernel<uint4>, dim3(1024), dim3(256), 0, s, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), (int64_t)(bytes / 16));
  } else if (a % 4 == 0 && bytes % 4 == 0) {
    hipLaunchKernelGGL(dcopy_kernel<uint32_t>, dim3(1024), dim3(256), 0, s, static_cast<uint32_t *>(dst),
                       static_cast<const uint32_t *>(src), (int64_t)(bytes / 4));
  } else {
    hipLaunchKernelGGL(dcopy_kernel<uint8_t>, dim3(1024), dim3(256), 0, s, static_cast<uint8_t *>(dst),
                       static_cast<const uint8_t *>(src), (int64_t)bytes);
  }
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

// Region sharing of up to two fields in one launch: halo <- pool, then pool <-
// top, element by element (a lane reads its pool element before it writes it).
// Bound by the launch where its planes fit the last-level cache, by HBM beyond.
// What a lane holds is a plain vector type: an array of HIP's vector class went
// to LDS, 16 us per launch at any size.  Measured on MI355X, us for two or four
// copies, in that array, and now, one field 1 MiB 5.4 16 2.7, 8 MiB 6.1 18 4.5, 32
// MiB 18 27 17, 64 MiB 33 41 32, 128 MiB 72 98 88; two fields 1 MiB 11 16 3.0, 8
// MiB 13 21 10, 32 MiB 36 41 33, 64 MiB 73 101 84: one launch while what it
// reads and writes fits the cache, single copies above.
typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void share_kernel(ShareArgs a, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    Vec4 below[2], above[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      if (a.halo[f]) below[f] = static_cast<const Vec4 *>(a.pool[f])[i];
      if (a.top[f]) above[f] = static_cast<const Vec4 *>(a.top[f])[i];
    }
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      if (a.halo[f]) static_cast<Vec4 *>(a.halo[f])[i] = below[f];
      if (a.top[f]) static_cast<Vec4 *>(a.pool[f])[i] = above[f];
    }
  }
}

int launch_share(const ShareArgs &a, size_t bytes, hipStream_t s) {
  if (bytes == 0) return 0;
  uintptr_t bits = (uintptr_t)bytes;
  bool meet = false;   // a chunk whose halo and top planes overlap
  uint64_t touched = 0;
  for (int f = 0; f < 2; ++f) {
    const char *h = static_cast<const char *>(a.halo[f]), *t = static_cast<const char *>(a.top[f]);
    if (h || t) bits |= (uintptr_t)a.pool[f] | (uintptr_t)h | (uintptr_t)t;
    if (h && t) meet = meet || (h < t + bytes && t < h + bytes);
    if (h || t) touched += bytes * (1 + (h != nullptr) + (t != nullptr));
  }
  if (touched == 0) return 0;
  if (bits % 16 == 0 && !meet && touched <= kLastLevelCache) {
    hipLaunchKernelGGL(share_kernel, dim3(1024), dim3(256), 0, s, a, (int64_t)(bytes / 16));
    return hipGetLastError() == hipSuccess ? 0 : -5;
  }
  int rc = 0;
  for (int f = 0; f < 2; ++f) {
    if (a.halo[f] && !rc) rc = launch_dcopy(a.halo[f], a.pool[f], bytes, s);
    if (a.top[f] && !rc) rc = launch_dcopy(a.pool[f], a.top[f], bytes, s);
  }
  return rc;
}

// Host memory, through its device mapping, to or from HBM.  Bound by the link:
// four 16-byte accesses in flight per lane and a few dozen workgroups carry
// it, while many more (a share of the chip that waits on the link) slow
// whatever else reads memory.  The accesses are aligned to 128 bytes on the
// host's side, where a partial line costs a transaction of its own, and to
// nothing on the other: a chunk's planes begin at any multiple of the element.
// Measured on MI355X, 64 MiB in / out, us: 1188 / 1214 with both sides
// aligned (1240 without the host's side aligned), the DMA engines 1174 / 1184;
// 2 MiB 50 / 50 and 46 / 46.
struct Aligned16 { Vec4 v; };
struct __attribute__((packed)) Anywhere16 { Vec4 v; };

template <typename D, typename S>
__global__ __launch_bounds__(256) void host_copy_kernel(char *__restrict__ dst, const char *__restrict__ src,
                                                        int64_t n, int head) {
  constexpr int U = 4;
  if (blockIdx.x == 0 && (int)threadIdx.x < head) dst[threadIdx.x] = src[threadIdx.x];
  const int64_t units = (n - head) / 16, done = head + units * 16;
  if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < (int)(n - done)) dst[done + threadIdx.x] = src[done + threadIdx.x];
  D *d = reinterpret_cast<D *>(dst + head);
  const S *s = reinterpret_cast<const S *>(src + head);
  const int64_t stride = (int64_t)gridDim.x * 256;
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (; i + (U - 1) * stride < units; i += U * stride) {
    Vec4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = s[i + u * stride].v;
#pragma unroll
    for (int u = 0; u < U; ++u) d[i + u * stride].v = v[u];
  }
  for (; i < units; i += stride) d[i].v = s[i].v;
}

int launch_host_copy(void *dst, const void *src, size_t bytes, bool to_host, int wgs, hipStream_t s) {
  if (bytes == 0) return 0;
  const uintptr_t host = (uintptr_t)(to_host ? dst : src);
  const int head = (int)std::min<size_t>((128 - host % 128) % 128, bytes);
  const int64_t steps = ((int64_t)bytes / 16 + 255) / 256;   // workgroup steps of 4 KiB
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(wgs, steps));
  char *d = static_cast<char *>(dst);
  const char *c = static_cast<const char *>(src);
  if (to_host)
    hipLaunchKernelGGL((host_copy_kernel<Aligned16, Anywhere16>), dim3(grid), dim3(256), 0, s, d, c, (int64_t)bytes, head);
  else
    hipLaunchKernelGGL((host_copy_kernel<Anywhere16, Aligned16>), dim3(grid), dim3(256), 0, s, d, c, (int64_t)bytes, head);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

__global__ __launch_bounds__(64) void empty_kernel() {}

int launch_empty(hipStream_t s) {
  hipLaunchKernelGGL(empty_kernel, dim3(1), dim3(64), 0, s);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <typename T>
__global__ __launch_bounds__(256) void loss_kernel(T *lam_u, const T *y, int64_t n, double *partials) {
  __shared__ double red[kRedThreads];
  double s = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double d = to_d(lam_u[i]) - to_d(y[i]);   // exact for FP32 inputs
    lam_u[i] = (T)d;                                 // one rounding, as u - y in T
    s += 0.5 * d * d;
  }
  const double b = block_sum(s, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = b;
}

// acc[k] += sum_b partials[b * np + k]: one workgroup per k; lane t sums
// b = t, t + 256, ... in order, then a fixed tree -- the same order every run.
__global__ __launch_bounds__(256) void reduce_partials(const double *partials, int nb, int np, double *acc) {
  __shared__ double red[kRedThreads];
  const int k = blockIdx.x;
  double s = 0.0;
  for (int b = threadIdx.x; b < nb; b += kRedThreads) s += partials[(int64_t)b * np + k];
  const double t = block_sum(s, red);
  if (threadIdx.x == 0) acc[k] += t;
}

// Sum over the wave's lanes in a fixed order (rows of 16 lanes by shifts, then
// the rows); lane 63 holds it.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xF, false);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0x111, 0xF>(v);   // row_shr:1, lanes without a source add 0
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
}

// partials[block * NP + k] += sum over the block's cells x of
// lam(x) u(x + o_k).  A lane takes V consecutive cells of a row (V = 4 where
// rows are whole vectors, else 1); vectors are dealt to lanes in flat order
// over the owned planes, and a lane steps from one to its next by carries,
// without divisions.  Per vector it loads lambda, one vector of u per (dz, dy)
// row of the stencil and, where the row has x offsets, the R cells on either
// side, all from clamped in-grid addresses and before any is used; terms whose
// cell is outside the grid are not accumulated.  Sums stay in the block's own
// partials from launch to launch; reduce_partials adds the blocks up once.
//
// Bound by latency at the gradient's usual chunk sizes (16 planes of 320^2: 14
// MB from the caches).  One lane per cell of a row with a tree over the
// workgroup per point and a reduction launch each time took 21 us + 5 us;
// this takes 7.5 us.
template <typename T, int NDIM, bool BOX, int R, int V>
__global__ __launch_bounds__(256) void wgrad_kernel(const T *__restrict__ lam, const T *__restrict__ u,
                                                    int64_t buf_z0, int nx, int ny, int per_x, int per_y,
                                                    int64_t n_axis, int64_t z0, int64_t z1, double *partials) {
  using S = Stencil<NDIM, BOX, R>;
  constexpr int RY = S::RY, NP = S::npts();
  __shared__ double red[4][NP];
  double acc[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) acc[k] = 0.0;
  const int64_t plane = (int64_t)nx * ny;
  const uint32_t nv = (uint32_t)nx / V;   // vectors per row (whole)
  const uint32_t stride = gridDim.x * 256u, q0 = blockIdx.x * 256u + threadIdx.x, nyv = (uint32_t)ny * nv;
  const int sz = (int)(stride / nyv), sy = (int)(stride % nyv / nv), sx = (int)(stride % nv);
  int64_t z = z0 + q0 / nyv;
  int y = (int)(q0 % nyv / nv), xv = (int)(q0 % nv);
  while (z < z1) {
    const int x = xv * V;
    const int64_t at = (z - buf_z0) * plane + (int64_t)y * nx + x;
    T l[V];
    T c[2 * R + 1][2 * RY + 1][V];          // the stencil's rows at the lane's cells
    T e[2 * R + 1][2 * RY + 1][2][R];       // and the R cells left and right of them
    bool ok[2 * R + 1][2 * RY + 1], okx[2][R];
    int xe[2][R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int xl = x - 1 - i, xr = x + V + i;   // e[..][0][i] is x - 1 - i, e[..][1][i] is x + V + i
      okx[0][i] = per_x || xl >= 0;
      okx[1][i] = per_x || xr < nx;
      xe[0][i] = (xl >= 0 ? xl : per_x ? nx - 1 - (-xl - 1) % nx : 0) - x;
      xe[1][i] = (xr < nx ? xr : per_x ? (xr - nx) % nx : 0) - x;
    }
    __builtin_memcpy(l, lam + at, sizeof(l));
#pragma unroll
    for (int a = -R; a <= R; ++a)
#pragma unroll
      for (int b = -RY; b <= RY; ++b) {
        if (!S::row_used(a, b)) continue;
        int yy = y + b;
        bool in = z + a >= 0 && z + a < n_axis;
        if (yy < 0 || yy >= ny) {
          if (per_y) yy = ((yy % ny) + ny) % ny; else in = false;
        }
        ok[a + R][b + RY] = in;
        const T *row = u + at + (in ? a * plane + (int64_t)(yy - y) * nx : 0);
        __builtin_memcpy(c[a + R][b + RY], row, sizeof(l));
        if (S::row_has_x(a, b)) {
#pragma unroll
          for (int side = 0; side < 2; ++side)
#pragma unroll
            for (int i = 0; i < R; ++i) e[a + R][b + RY][side][i] = row[xe[side][i]];
        }
      }
#pragma unroll
    for (int a = -R; a <= R; ++a)
#pragma unroll
      for (int b = -RY; b <= RY; ++b) {
        if (!S::row_used(a, b)) continue;
        if (!ok[a + R][b + RY]) continue;
#pragma unroll
        for (int d = -R; d <= R; ++d) {
          const int k = S::table.idx[a + R][b + RY][d + R];
          if (k < 0) continue;
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const int t = j + d;
            if (t >= 0 && t < V)
              acc[k] += to_d(l[j]) * to_d(c[a + R][b + RY][t]);
            else if (okx[t >= V][t < 0 ? -t - 1 : t - V])
              acc[k] += to_d(l[j]) * to_d(e[a + R][b + RY][t >= V][t < 0 ? -t - 1 : t - V]);
          }
        }
      }
    xv += sx;
    y += sy;
    z += sz;
    if (xv >= (int)nv) {
      xv -= (int)nv;
      ++y;
    }
    if (y >= ny) {
      y -= ny;
      ++z;
    }
  }
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const double w = wave_sum(acc[k]);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6][k] = w;
  }
  __syncthreads();
  if (threadIdx.x < NP)
    partials[(int64_t)blockIdx.x * NP + threadIdx.x] +=
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

template <typename T>
static int loss_t(void *lam_u, const void *y, int64_t n, double *partials, double *acc, hipStream_t s) {
  hipLaunchKernelGGL(loss_kernel<T>, dim3(kRedWgs), dim3(kRedThreads), 0, s, static_cast<T *>(lam_u),
                     static_cast<const T *>(y), n, partials);
  hipLaunchKernelGGL(reduce_partials, dim3(1), dim3(kRedThreads), 0, s, partials, kRedWgs, 1, acc);
  return hipGetLastError() == hipSuccess ? 0 : SO2DR_E_HIP;
}

int launch_loss(int dtype, void *lam_u, const void *y, int64_t n, double *partials, double *acc,
                hipStream_t s) {
  if (n <= 0) return 0;
  switch (dtype) {
    case SO2DR_F32: return loss_t<float>(lam_u, y, n, partials, acc, s);
    case SO2DR_F64: return loss_t<double>(lam_u, y, n, partials, acc, s);
    default: return SO2DR_E_UNSUPPORTED;
  }
}

template <typename T, int NDIM, bool BOX, int R>
static int wgrad_st(const void *lam, const void *u, int64_t buf_z0, int nx, int ny, int per_x, int per_y,
                    int64_t n_axis, int64_t z0, int64_t z1, double *partials, hipStream_t s) {
  // as few passes of kRedWgs workgroups as cover the vectors, evenly filled
  const int v = nx % 4 == 0 ? 4 : 1;
  const int64_t need = ((z1 - z0) * ny * (nx / v) + kRedThreads - 1) / kRedThreads;
  const int64_t passes = (need + kRedWgs - 1) / kRedWgs;
  const int grid = (int)((need + passes - 1) / passes);
  const T *l = static_cast<const T *>(lam), *w = static_cast<const T *>(u);
  if (v == 4)
    hipLaunchKernelGGL((wgrad_kernel<T, NDIM, BOX, R, 4>), dim3(grid), dim3(kRedThreads), 0, s, l, w, buf_z0, nx, ny,
                       per_x, per_y, n_axis, z0, z1, partials);
  else
    hipLaunchKernelGGL((wgrad_kernel<T, NDIM, BOX, R, 1>), dim3(grid), dim3(kRedThreads), 0, s, l, w, buf_z0, nx, ny,
                       per_x, per_y, n_axis, z0, z1, partials);
  return hipGetLastError() == hipSuccess ? 0 : SO2DR_E_HIP;
}

template <typename T>
static int wgrad_t(int stencil, const void *lam, const void *u, int64_t buf_z0, int nx, int ny, int per_x, int per_y,
                   int64_t n_axis, int64_t z0, int64_t z1, double *partials, hipStream_t s) {
#define SO2DR_CASE(ID, NDIM, BOX, R) \
  case ID: return wgrad_st<T, NDIM, BOX, R>(lam, u, buf_z0, nx, ny, per_x, per_y, n_axis, z0, z1, partials, s);
  switch (stencil) {
    SO2DR_CASE(ST_2D_STAR_R1, 2, false, 1)
    SO2DR_CASE(ST_2D_BOX_R1, 2, true, 1)
    SO2DR_CASE(ST_2D_BOX_R2, 2, true, 2)
    SO2DR_CASE(ST_2D_BOX_R3, 2, true, 3)
    SO2DR_CASE(ST_2D_BOX_R4, 2, true, 4)
    SO2DR_CASE(ST_3D_STAR_R1, 3, false, 1)
    SO2DR_CASE(ST_3D_STAR_R2, 3, false, 2)
    SO2DR_CASE(ST_3D_BOX_R1, 3, true, 1)
    default: return SO2DR_E_UNSUPPORTED;
  }
#undef SO2DR_CASE
}

int launch_wgrad(int dtype, int stencil, const void *lam, const void *u, int64_t buf_z0, int nx, int ny, int per_x,
                 int per_y, int64_t n_axis, int64_t z0, int64_t z1, double *partials, hipStream_t s) {
  if (z1 <= z0) return 0;
  switch (dtype) {
    case SO2DR_F32:
      return wgrad_t<float>(stencil, lam, u, buf_z0, nx, ny, per_x, per_y, n_axis, z0, z1, partials, s);
    case SO2DR_F64:
      return wgrad_t<double>(stencil, lam, u, buf_z0, nx, ny, per_x, per_y, n_axis, z0, z1, partials, s);
    default:
      return SO2DR_E_UNSUPPORTED;
  }
}

int launch_wgrad_sum(int npts, const double *partials, double *acc, hipStream_t s) {
  hipLaunchKernelGGL(reduce_partials, dim3(npts), dim3(kRedThreads), 0, s, partials, kRedWgs, npts, acc);
  return hipGetLastError() == hipSuccess ? 0 : SO2DR_E_HIP;
}

}  // namespace so2dr
