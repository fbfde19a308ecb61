// launch_impl.hpp -- shared by the objects of kernels.hip: picks a launch's
// kernel and tile shape, builds its argument block, sizes its grid and launches it.
#pragma once
#include <atomic>
#include <algorithm>
#include <string>

#include "lane_tile.hpp"
#include "launch.hpp"
#include "march2d_kernel.hpp"
#include "march_plan.hpp"
#include "wide2d_kernel.hpp"
#include "march_kernel.hpp"
#include "tb_kernel.hpp"

namespace so2dr {

// Workgroups an LDS-plane launch aims for before it splits the cut axis into
// segments; each re-reads 2*KL*R input planes, so segments stay long.
constexpr int64_t kTargetWgs = 1024;
constexpr int64_t kMinSegPlanes = 16;

// Segmenting of the cut axis for the LDS-plane kernel: kTargetWgs workgroups,
// never segments shorter than kMinSegPlanes.
inline void plan_segments(int64_t span, int64_t tiles, int64_t *zseg, int *nseg) {
  int64_t n = std::max<int64_t>(1, (kTargetWgs + tiles - 1) / tiles);
  n = std::min<int64_t>(n, std::max<int64_t>(1, span / kMinSegPlanes));
  *zseg = (span + n - 1) / n;
  *nseg = (int)((span + *zseg - 1) / *zseg);
}

// Workgroups of `kernel` (block of `threads`) that the current device holds
// at once: resident workgroups per CU times CUs; 0 if the runtime cannot
// tell.  Per-CU residency depends only on the kernel, so it is asked once
// per kernel; the CU count once per device.
inline int64_t resident_wgs(const void *kernel, int threads, std::atomic<int> *per_cu_cache) {
  int per_cu = per_cu_cache->load(std::memory_order_relaxed);
  if (per_cu < 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) per_cu = 0;
    per_cu_cache->store(per_cu, std::memory_order_relaxed);
  }
  static std::atomic<int> cu_count[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int cus = cu_count[dev].load(std::memory_order_relaxed);
  if (cus <= 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    cu_count[dev].store(cus, std::memory_order_relaxed);
  }
  return (int64_t)per_cu * cus;
}

// The argument block every kernel takes: buffers, geometry, planes and the
// weights converted to the accumulation type.  Tile counts and segmenting
// are the caller's.
template <typename A>
inline TbArgs<A> launch_args(const LaunchParams &p, int npts) {
  TbArgs<A> a{};
  a.in = p.in;
  a.out = p.out;
  a.buf_z0 = p.buf_z0;
  a.out_z0 = p.out_z0;
  a.plane = p.plane;
  a.nx = p.nx;
  a.ny = p.ny;
  a.per_x = p.per_x;
  a.per_y = p.per_y;
  a.n_axis = p.n_axis;
  a.in_lo = p.in_lo;
  a.in_hi = p.in_hi;
  a.out_lo = p.out_lo;
  a.out_hi = p.out_hi;
  for (int i = 0; i < npts; ++i) a.w.w[i] = (A)p.weights[i];
  return a;
}

template <typename T, int NDIM, bool BOX, int R, int KL, bool RAS = false>
int launch_one(const LaunchParams &p, hipStream_t stream, std::string *msg) {
  using A = typename Store<T>::A;
  using G = Tile<NDIM, R, KL>;
  using S = Stencil<NDIM, BOX, R>;
  if (p.npts != S::npts()) {
    if (msg) *msg = "weight count does not match the stencil";
    return -1;
  }
  TbArgs<A> a = launch_args<A>(p, S::npts());
  a.ntx = (int)((p.nx + G::OX - 1) / G::OX);
  a.nty = NDIM == 2 ? 1 : (int)((p.ny + G::OY - 1) / G::OY);
  const int64_t span = p.out_hi - p.out_lo;
  if (span <= 0) return 0;
  plan_segments(span, (int64_t)a.ntx * a.nty, &a.zseg, &a.nseg);
  const int64_t nwg = (int64_t)a.ntx * a.nty * a.nseg;
  if (nwg > 0x7fffffff) {
    if (msg) *msg = "grid too large for one launch";
    return -1;
  }
  constexpr size_t lds = tb_lds_bytes<T, NDIM, BOX, R, KL>();
  // once per instantiation; threads racing here both set the same value
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void *)tb_kernel<T, NDIM, BOX, R, KL, RAS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) {
      if (msg) *msg = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
      return -5;
    }
    attr_done.store(true, std::memory_order_release);
  }
  const int64_t grid = xcd_grid(nwg);
  hipLaunchKernelGGL((tb_kernel<T, NDIM, BOX, R, KL, RAS>), dim3((unsigned)grid), dim3(G::NT), lds, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    if (msg) *msg = std::string("kernel launch: ") + hipGetErrorString(e);
    return -5;
  }
  return 0;
}

// Whether the march kernel's layout fits this launch: whole VX-cell vectors
// per row, 32-bit byte offsets within a plane, 32-bit plane indices.
template <typename T, int VX>
inline bool march_fits(const LaunchParams &p) {
  // the kernels clamp loads into [max(in_lo, 0), min(in_hi, n_axis)): that
  // range must be non-empty
  return p.nx % VX == 0 && (uint64_t)p.plane * sizeof(T) < ((uint64_t)1 << 32) &&
         p.n_axis < ((int64_t)1 << 30) && p.in_lo > -((int64_t)1 << 29) && p.buf_z0 > -((int64_t)1 << 29) &&
         p.out_z0 > -((int64_t)1 << 29) && std::max<int64_t>(p.in_lo, 0) < std::min<int64_t>(p.in_hi, p.n_axis);
}

// One tile shape of march3d_kernel: its segmenting and predicted cost for a
// launch, and the launch itself.
template <typename T, bool BOX, int R, int KL, int NW, int M, int VX, int HB, int PF, int WPE = 1,
          bool RAS = false, int HA = VX>
struct March3d {
  using A = typename Store<T>::A;
  using G = StarTile<R, KL, NW, M, VX, HA>;
  using S = Stencil<3, BOX, R>;
  static constexpr auto kernel = march3d_kernel<T, BOX, R, KL, NW, M, VX, HB, PF, WPE, RAS, HA>;

  static int ntx(const LaunchParams &p) { return (int)((p.nx + G::OX - 1) / G::OX); }
  static int nty(const LaunchParams &p) { return (int)((p.ny + G::OY - 1) / G::OY); }

  // cached: the launch's planes fit the last-level cache
  static MarchPlan plan(const LaunchParams &p, bool cached = false, double scale = 1.0) {
    static std::atomic<int> per_cu{-1};
    const int64_t slots = resident_wgs((const void *)kernel, NW * 64, &per_cu);
    const int occ = std::max(1, per_cu.load(std::memory_order_relaxed));
    const int cus = slots > 0 ? (int)(slots / occ) : 256;
    MarchMemory mem;
    if (cached) mem = {(double)p.plane * sizeof(T) / kCacheBytesPerCycle, 2 * KL * R};
    return plan_march(p.out_hi - p.out_lo, (int64_t)ntx(p) * nty(p), 2 * KL * R + KL - 1, cus, occ, kMarchLatency,
                      march_issue(NW, M, VX, KL, S::npts()), 1, scale, mem);
  }

  static int launch(const LaunchParams &p, const MarchPlan &mp, hipStream_t stream, std::string *msg) {
    if (p.npts != S::npts()) {
      if (msg) *msg = "weight count does not match the stencil";
      return -1;
    }
    TbArgs<A> a = launch_args<A>(p, S::npts());
    a.ntx = ntx(p);
    a.nty = nty(p);
    a.zseg = mp.zseg;
    a.nseg = mp.nseg;
    const int64_t nwg = (int64_t)a.ntx * a.nty * a.nseg;
    if (nwg > 0x7fffffff) {
      if (msg) *msg = "grid too large for one launch";
      return -1;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(nwg)), dim3(NW * 64), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
      if (msg) *msg = std::string("kernel launch: ") + hipGetErrorString(e);
      return -5;
    }
    return 0;
  }
};

// Bytes that a launch reads and writes, and whether its planes fit the last-level
// cache.
template <typename T>
uint64_t launch_bytes(const LaunchParams &p) {
  return (uint64_t)(std::min(p.in_hi, p.n_axis) - std::max<int64_t>(p.in_lo, 0) + p.out_hi - p.out_lo) *
         (uint64_t)p.plane * sizeof(T);
}
template <typename T>
bool in_cache(const LaunchParams &p) { return launch_bytes<T>(p) <= kLastLevelCache; }

// Segmenting of one launch of a 2D kernel over row tiles G: `rows` input rows
// per step (a segment ends with a step where it can), `extra` rows' work besides
// its own per segment, `issue` and `lat` cycles per row as in plan_march.
template <typename T, typename G, typename A>
MarchPlan plan_rows(void (*kernel)(TbArgs<A>), const LaunchParams &p, int rows, int halo, int extra, double lat,
                    double issue, std::atomic<int> *per_cu) {
  const int64_t slots = resident_wgs((const void *)kernel, 64 * kRowWaves, per_cu);
  const int occ = std::max(1, per_cu->load(std::memory_order_relaxed));
  const int64_t span = p.out_hi - p.out_lo;
  MarchMemory mem;
  if (in_cache<T>(p)) mem = {(double)p.plane * sizeof(T) / kCacheBytesPerCycle2d, halo};
  MarchPlan mp = plan_march(span, (p.nx + G::OX - 1) / G::OX, extra, slots > 0 ? (int)(slots / occ) : 256, occ, lat,
                            issue, kRowWaves, 1.0, mem);
  mp.zseg = (mp.zseg + halo + rows - 1) / rows * rows - halo;
  mp.nseg = (int)((span + mp.zseg - 1) / mp.zseg);
  return mp;
}

template <typename S, typename G, typename A>
int launch_rows(void (*kernel)(TbArgs<A>), const LaunchParams &p, const MarchPlan &mp, hipStream_t stream,
                std::string *msg) {
  if (p.npts != S::npts()) {
    if (msg) *msg = "weight count does not match the stencil";
    return -1;
  }
  TbArgs<A> a = launch_args<A>(p, S::npts());
  a.ntx = (int)((p.nx + G::OX - 1) / G::OX);
  a.nty = 1;
  a.zseg = mp.zseg;
  a.nseg = mp.nseg;
  const int64_t nwg = ((int64_t)a.ntx * a.nseg + kRowWaves - 1) / kRowWaves;
  if (nwg > 0x7fffffff / kRowWaves) {
    if (msg) *msg = "grid too large for one launch";
    return -1;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(nwg)), dim3(64 * kRowWaves), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    if (msg) *msg = std::string("kernel launch: ") + hipGetErrorString(e);
    return -5;
  }
  return 0;
}

// One shape of march2d_kernel: its segmenting and predicted cost, and the launch.
template <typename T, bool BOX, int R, int KL, int VX, int PF, bool ROT, bool RAS = false>
struct March2d {
  using G = RowTile<R, KL, VX>;
  using S = Stencil<2, BOX, R>;
  static constexpr auto kernel = march2d_kernel<T, BOX, R, KL, VX, PF, ROT, RAS>;

  static MarchPlan plan(const LaunchParams &p) {
    // a wave's instructions per row (as for the 3D shapes) at 4 cycles each; the
    // latency from launches of 2, 3 and 4 waves per SIMD (12800 x 3260, two
    // levels of the radius-2 box: 93, 87, 86 us)
    constexpr double issue = 4.0 * (KL * (VX * S::npts() + 4.0) + 10.0), lat = 900.0;
    static std::atomic<int> per_cu{-1};
    return plan_rows<T, G>(kernel, p, 1, 2 * KL * R, 2 * KL * R + KL - 1, lat, issue, &per_cu);
  }
  static int launch(const LaunchParams &p, const MarchPlan &mp, hipStream_t stream, std::string *msg) {
    return launch_rows<S, G>(kernel, p, mp, stream, msg);
  }
};

// One shape of wide2d_kernel: its segmenting and predicted cost, and the launch.
template <typename T, int R, int VX, int U>
struct Wide2d {
  using G = RowTile<R, 1, VX>;
  using S = Stencil<2, true, R>;
  static constexpr auto kernel = wide2d_kernel<T, R, VX, U>;

  static MarchPlan plan(const LaunchParams &p) {
    // a segment's two ends cost about two rows: the rows of weights that none of
    // its outputs needs are skipped.  A latency of 1800 cycles per step chose
    // within 2 % of the best of 300 to 3000 on six grids (400 x 400 to 12800^2).
    constexpr double issue = 4.0 * (VX * S::npts() + 30.0), lat = 1800.0 / U;
    static std::atomic<int> per_cu{-1};
    return plan_rows<T, G>(kernel, p, U, 2 * R, 2, lat, issue, &per_cu);
  }
  static int launch(const LaunchParams &p, const MarchPlan &mp, hipStream_t stream, std::string *msg) {
    return launch_rows<S, G>(kernel, p, mp, stream, msg);
  }
};

// Bytes of the march kernel's halo buffers.
template <typename A, int KL, int NW, int R, int VX, int HB>
constexpr size_t march_lds() {
  return sizeof(A) * KL * HB * NW * 2 * R * 64 * VX;
}

// Kernel choice per depth, from measurements on MI355X (all variants give
// identical bits).
//
// 3D launches that stream from HBM (2048x1024x80 FP32 chunks) use wide rows:
//   * single-step launches 1 KiB rows (4 cells per lane, 16 waves of 2 rows):
//     0.26 ms, where one cell per lane takes 0.35;
//   * two fused steps of the radius-1 star: 1 KiB rows, 8 waves of 4 rows
//     (0.26 ms against 0.35);
//   * three fused steps of the radius-1 star and two of the radius-2 star:
//     512-byte rows, 8 waves of 6 rows (0.28 against 0.38 ms for the former;
//     taller tiles re-read fewer halo rows);
//   * other deeper fusion and the 27-point box: 512-byte rows, 8 waves of 4
//     rows (27-point at 2 levels 0.36 against 0.40 ms);
//   (the taller shapes hold FP32 sums only: FP64 keeps the 4-row tiles).
// Launches that fit the last-level cache take the shape of least cost
// (march_plan.hpp), mostly the narrow one: one cell per lane, 8 waves of 4 rows.
// Its tiles are a third to a sixth of the wide ones', so a mid-size grid divides
// evenly over the CUs, several workgroups share a CU and hide each other's
// barriers, and the tile overhang past the grid is smaller: 3 levels of the
// 7-point star on 256^3 44 us against 50 in the wide shape, 512x512x128 68
// against 85, 96x40x48 9 against 15; two levels of the BF16 13-point star on
// 320x320x26 19 against 23.  Rows that are not whole vectors have the narrow
// shapes only: the 27-point box on 301x257x203, two levels, 62 us, 85 in the
// register-column kernel that took them before.
// Planes of 4 GiB or more (and 2D rows of 4 GiB) take the LDS-plane kernel.
template <typename T, int NDIM, bool BOX, int R, int KL, bool RAS>
int launch_any(const LaunchParams &p, hipStream_t s, std::string *msg) {
  using A = typename Store<T>::A;
  constexpr size_t kLdsMax = 160 * 1024;
  if (p.out_hi <= p.out_lo) return 0;
  if constexpr (NDIM == 2) {
    // Unrolling by the stencil width is kept while the unrolled body stays
    // within 3000 FMAs (12 KiB of code; 2400 in FP64, whose FMAs take twice the
    // code): in this kernel one level of the radius-4 box, 2916 of them, took
    // 464 us on 12800^2 unrolled and 489 us with shifting sums.
    // FP64 lanes own two cells: four need 158 registers at 4 levels, three
    // waves per SIMD, and 93 us on 4800^2 where two need 82; two levels of the
    // radius-3 box gain 10 %.  One level of a box of radius 3 or 4 has a kernel
    // of its own, which is faster at every size (its header has the figures).
    // Grids that do not fill the chip take two cells per lane in FP32 and 16
    // bits as well, where the cost model says so: a wave's rows end sooner and
    // twice the tiles cover them.  us per launch on 400 x 400 (and 1201 x 1003),
    // two cells against four: 7 levels of the 5-point star 9.9 (14.7) and 11.6
    // (14.7), 6 of the radius-1 box 8.9 (13.9) and 10.7 (14.3), 3 of the radius-2
    // box 7.9 (12.9) and 10.3 (13.9), 2 of the radius-3 box 8.5 (14.2) and 11.8
    // (16.2), one of the radius-4 box 6.6 (11.3) and 9.1 (12.1).
    constexpr int VX = sizeof(T) == 8 ? 2 : 4;
    constexpr bool wide = BOX && R >= 3 && KL == 1;
    if (!p.plane_kernel && march_fits<T, 1>(p)) {
      auto shape = [&](auto vx) {
        constexpr int V = decltype(vx)::value;
        constexpr bool rot = (int64_t)KL * V * Stencil<2, BOX, R>::npts() * (2 * R + 1) > (sizeof(T) == 8 ? 2400 : 3000);
        using M = March2d<T, BOX, R, KL, V, 2, rot, RAS>;
        using W = Wide2d<T, R, V, 4>;
        return typename std::conditional<wide, W, M>::type{};
      };
      using Full = decltype(shape(std::integral_constant<int, VX>{}));
      const MarchPlan f = Full::plan(p);
      if constexpr (VX == 4) {
        using Half = decltype(shape(std::integral_constant<int, 2>{}));
        const MarchPlan h = Half::plan(p);
        if (h.cost < f.cost) return Half::launch(p, h, s, msg);
      }
      return Full::launch(p, f, s, msg);
    }
  }
  if constexpr (NDIM == 3) {
    constexpr bool single = KL == 1 && march_lds<A, KL, 16, R, 4, 2>() <= kLdsMax;
    constexpr bool a32 = sizeof(A) == 4;
    constexpr bool square = a32 && !BOX && R == 1 && KL == 2;
    constexpr bool tall = a32 && !BOX && ((R == 1 && KL == 3) || (R == 2 && KL == 2));
    // FP64 sums of two levels at radius 2 would spill in any wide shape
    constexpr bool no_wide = !a32 && R == 2 && KL == 2;
    constexpr int HB = march_lds<A, KL, 8, R, 2, 2>() <= 65536 ? 2 : 1;
    // Star tiles of 1 KiB FP32 rows (2 KiB FP64) take a 64-byte x halo: each
    // output row is then whole 128-byte lines.  Measured on 2048x1024
    // planes: single-step launches 3-8 % faster (FP32 7- and 13-point, FP64)
    // and the two-step 7-point launch 0-3 % faster than with the 4-cell halo,
    // whose output rows share lines with the neighbouring tiles.  The
    // 512-byte-row shapes of deeper fusion and the 27-point box lose more to
    // the wider halo's arithmetic than they gain; 16-bit rows gain nothing.
    constexpr int HA4 = BOX ? 4 : sizeof(T) == 4 ? 16 : sizeof(T) == 8 ? 8 : 4;
    constexpr int VXW = single || square ? 4 : 2;
    constexpr int NWW = single ? 16 : 8, MW = single ? 2 : tall ? 6 : 4;
    constexpr int HBW = single || square || tall ? 2 : HB, HAW = single || square ? HA4 : VXW;
    using Narrow = March3d<T, BOX, R, KL, 8, 4, 1, 2, 2, 1, RAS>;
    // half the waves and rows: a grid that does not fill the chip ends its march
    // steps sooner, and more tiles cover it (us, small against narrow: 3 levels
    // of the 7-point star on 48x40x30 5.7 and 7.3, 80x84x49 7.6 and 8.8; 2 of the
    // 13-point star 6.8 and 9.0, 9.2 and 11.1; 2 of the 27-point box 5.5 and 7.4)
    using Small = March3d<T, BOX, R, KL, 4, 4, 1, 2, 2, 1, RAS>;
    // two levels whose halo takes a quarter of 32 rows or whose box costs most
    // have a taller narrow shape, 8 waves of 6 rows: BF16 13-point on
    // 301x257x203 52 us against 57, 27-point 59 against 62
    constexpr bool two_narrow = a32 && KL == 2 && (BOX || R == 2);
    using Narrow6 = March3d<T, BOX, R, KL, 8, two_narrow ? 6 : 4, 1, 2, 2, 1, RAS>;
    if (!p.plane_kernel && march_fits<T, 1>(p)) {
      const bool cached = in_cache<T>(p);
      MarchPlan w;
      if constexpr (!no_wide) {
        using Wide = March3d<T, BOX, R, KL, NWW, MW, VXW, HBW, 2, 1, RAS, HAW>;
        constexpr double scale = wide_scale(BOX, a32, KL);
        if (march_fits<T, VXW>(p)) {
          if (!cached) return Wide::launch(p, Wide::plan(p), s, msg);
          if (scale > 0) w = Wide::plan(p, true, scale);
        }
        if constexpr (square) {   // rows of an odd number of 2-cell vectors
          using Mid = March3d<T, BOX, R, KL, 8, 4, 2, 2, 2, 1, RAS>;
          if (!cached && march_fits<T, 2>(p)) return Mid::launch(p, Mid::plan(p), s, msg);
        }
      }
      // the least cost; on a tie (the cache binds) the wider shape
      const MarchPlan n = Narrow::plan(p, cached), q = Small::plan(p, cached), n6 = Narrow6::plan(p, cached);
      const double least = std::min(n.cost, std::min(q.cost, n6.cost));
      if constexpr (!no_wide) {
        using Wide = March3d<T, BOX, R, KL, NWW, MW, VXW, HBW, 2, 1, RAS, HAW>;
        if (w.nseg > 0 && w.cost <= least) return Wide::launch(p, w, s, msg);
      }
      if (n.cost <= least) return Narrow::launch(p, n, s, msg);
      if (q.cost <= least) return Small::launch(p, q, s, msg);
      return Narrow6::launch(p, n6, s, msg);
    }
  }
  return launch_one<T, NDIM, BOX, R, KL, RAS>(p, s, msg);
}

// Expand one stencil's depths 1..MAXKL into a switch on p.kl.
template <typename T, int NDIM, bool BOX, int R, int MAXKL, bool RAS>
int launch_depth_r(const LaunchParams &p, hipStream_t s, std::string *msg) {
  switch (p.kl) {
    case 1: return launch_any<T, NDIM, BOX, R, 1, RAS>(p, s, msg);
    case 2: if constexpr (MAXKL >= 2) return launch_any<T, NDIM, BOX, R, 2, RAS>(p, s, msg); else break;
    case 3: if constexpr (MAXKL >= 3) return launch_any<T, NDIM, BOX, R, 3, RAS>(p, s, msg); else break;
    case 4: if constexpr (MAXKL >= 4) return launch_any<T, NDIM, BOX, R, 4, RAS>(p, s, msg); else break;
    case 5: if constexpr (MAXKL >= 5) return launch_any<T, NDIM, BOX, R, 5, RAS>(p, s, msg); else break;
    case 6: if constexpr (MAXKL >= 6) return launch_any<T, NDIM, BOX, R, 6, RAS>(p, s, msg); else break;
    case 7: if constexpr (MAXKL >= 7) return launch_any<T, NDIM, BOX, R, 7, RAS>(p, s, msg); else break;
    case 8: if constexpr (MAXKL >= 8) return launch_any<T, NDIM, BOX, R, 8, RAS>(p, s, msg); else break;
    default: break;
  }
  if (msg) *msg = "fused depth not built for this stencil";
  return -3;
}

// Round-at-store variants exist for the 16-bit storage types only: FP32 and
// FP64 storage rounds nothing between levels either way.
template <typename T, int NDIM, bool BOX, int R, int MAXKL>
int launch_depth(const LaunchParams &p, hipStream_t s, std::string *msg) {
  if constexpr (sizeof(T) == 2) {
    if (p.ras) return launch_depth_r<T, NDIM, BOX, R, MAXKL, true>(p, s, msg);
  }
  return launch_depth_r<T, NDIM, BOX, R, MAXKL, false>(p, s, msg);
}

}  // namespace so2dr
