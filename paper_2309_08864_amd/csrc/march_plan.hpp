// march_plan.hpp -- the cost model of a march launch: plain host code, with no
// device calls.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace so2dr {

// A launch's cost in clock cycles for segments of a given length, and the
// segmenting of least cost.  A workgroup's march step takes `lat` cycles of
// latency (barrier, LDS round trip, address work) plus its own issue time
// `issue` and that of the workgroups sharing its CU, and a segment of zseg
// output planes takes zseg + extra steps; workgroups run in rounds of CUs x
// per_cu.  Candidates fill k workgroups per CU, k = 1, 2, ..., which is where
// the rounds change; more, shorter segments only for a gain of 0.5 %, since each
// re-reads `extra` planes.  per_wg: tiles a workgroup takes (2D: one per wave).
// scale: the shape's march steps cost that much more than the model says.
// mem.plane > 0: no less than the planes read (reread more per segment) and
// written take at the last-level cache's rate, which launches of one level,
// and of FP64, reach; three tenths of the steps' time show even then.
//
// Measured on MI355X (3D 7-point FP32, 3 levels, tiles of 8 waves x 6 rows x 2
// cells): a 256^3 grid took 76 us in 336 workgroups of 16-plane segments (the
// former rule: 1.5 workgroups per slot, segments of at least 16 planes) and
// 50 us in 252 of 22 planes, one round instead of two; a 320 x 320 x 26 chunk
// 52 us in 24 workgroups and 19 us in 216.  2D: one level of the radius-3 box on
// 12800^2 took 329 us in 1027 workgroups, five on some CUs, and 290 us in
// 1014; five levels of the radius-1 box on 1020 x 767 rows 19 us in 17-row
// segments and 11 us in 4-row ones.  Over 323 launches of 47 shapes on 9
// grids the choice came within 3 % (geometric mean) of the best segmenting
// tried.  Over 420 3D launches beyond the cache (five grids, up to eight
// segments) it came within 1.2 % of the best and the former rule within 5.6 %;
// 19 of them are more than 1 % slower than by the former rule, 5 % at most, 206
// faster, and a price for the re-read planes loses there (1.4 to 1.9 % from the
// best where it is added to the steps, 3 to 7 % as a lower bound).
struct MarchPlan {
  int64_t zseg = 0;
  int nseg = 0;
  double cost = 0.0;
};

struct MarchMemory {
  double plane = 0.0;   // cycles one plane of the grid takes (0: no such bound)
  int reread = 0;       // planes a segment reads beside its own
};

inline MarchPlan plan_march(int64_t span, int64_t tiles, int extra, int cus, int per_cu, double lat, double issue,
                            int per_wg = 1, double scale = 1.0, MarchMemory mem = MarchMemory()) {
  constexpr int kMaxPerCu = 12;    // candidates; beyond, rounds no longer matter
  constexpr int kPrologue = 2;     // steps' worth of start-up per workgroup
  MarchPlan best;
  int64_t last = 0;
  for (int k = 1; k <= kMaxPerCu; ++k) {
    const int64_t want = std::min(span, std::max<int64_t>(1, (int64_t)k * cus * per_wg / tiles));
    if (want == last) continue;
    last = want;
    const int64_t zseg = (span + want - 1) / want, nseg = (span + zseg - 1) / zseg;
    const int64_t n = (tiles * nseg + per_wg - 1) / per_wg, full = n / ((int64_t)cus * per_cu), rest = n - full * cus * per_cu;
    const double t = (double)full * (lat + per_cu * issue) +
                     (rest > 0 ? lat + (double)((rest + cus - 1) / cus) * issue : 0.0);
    double c = scale * (double)(zseg + extra + kPrologue) * t;
    if (mem.plane > 0) c = std::max(c, mem.plane * (double)(2 * span + nseg * mem.reread)) + 0.3 * c;
    if (best.nseg == 0 || c < 0.995 * best.cost) best = {zseg, (int)nseg, c};
  }
  return best;
}

// Instructions of one wave per 3D march step, in clock cycles of the four SIMDs
// that NW waves share (a wave instruction takes 4): the multiply-adds, per row
// and level the lane shifts, halo rows and stores, and the plane's addresses.
constexpr double march_issue(int nw, int m, int vx, int kl, int npts) {
  return nw * (m * kl * (vx * npts + 4.0) + 20.0);
}
constexpr double kMarchLatency = 800.0;

// What 3D launches within the last-level cache choose a shape by.  The wide
// shapes' two waves per SIMD issue at 66 of the 73 TFLOP/s that the narrow ones'
// four reach, and hide less of a step's latency: their steps cost more (scale),
// least where a step is all multiply-adds or waits for the cache anyway; one
// level of the 27-point box and any of its FP64 ones never gained by them (0:
// not taken).  The cache carries 2600 bytes per cycle (6.2 TB/s).  Fitted to
// 842 launches (nine grids of 128 x 128 to 1024 x 1024, 12 to 100 planes, one to
// three levels, FP32, FP64 and BF16, each shape in up to 11 segmentings): 3.6 %
// from the best on average.  With one factor of 1/0.8 and no bound by the cache
// it was 4.4 %, and single launches were up to 33 % slower than the wide shape
// in the former rule's segments (now 14 %): us there, so, and now, 7-point FP32
// one level 512 x 512 x 64 24, 32 and 26; FP64 two levels 1024 x 512 x 24 38, 44
// and 38; 13-point FP64 one level 512 x 512 x 40 32, 38 and 32.
constexpr double wide_scale(bool box, bool fp32_sums, int levels) {
  if (box) return fp32_sums && levels > 1 ? 1.0 / 0.95 : 0.0;
  return levels > 1 ? 1.0 / 0.85 : fp32_sums ? 1.0 / 0.95 : 1.0 / 0.9;
}
constexpr double kCacheBytesPerCycle = 2600.0;
// The 2D kernels' (5.3 TB/s), fitted to 1350 launches of nine row lengths.  us by
// the former rule (segments for 1024 workgroups), without this bound, and with
// it: 5-point FP32 one level of 800 rows of 12800 cells 13.9, 16.5, 14.7; two
// levels of 3200 rows of 4800 21.6, 26.3, 21.8; 25-point FP64 one level of 800
// rows of 12800 29.2, 34.1, 28.9.
constexpr double kCacheBytesPerCycle2d = 2200.0;

}  // namespace so2dr
