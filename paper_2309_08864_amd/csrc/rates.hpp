// rates.hpp -- measured update rates of the fused-step kernels on MI355X,
// read by the planner (automatic fused depth) and the cost model.
//
// G cell-updates/s (output cells x fused levels per second) of one launch by
// storage type, stencil id and depth 1..8 (0 = depth not built), measured
// with so2dr_kernel_bench (`bench.py --kernel-rates --grid ...`) over an
// interior chunk of 64 output planes of a 2048 x 1024 plane in 3D and 1200
// output rows of 38400 cells in 2D.  The 2D chunks of 16-bit storage fit
// the 256 MiB last-level cache in part, which their rates include.
#pragma once
#include <stdint.h>

namespace so2dr {

// rows: so2dr_dtype F32, F64, BF16, F16; then StencilId; then depth - 1
constexpr double kRate[4][8][8] = {
    {
        // F32
        {624, 1178, 1688, 2251, 2725, 3121, 3255, 3359},  // 2D star r1
        {621, 1171, 1738, 2038, 2094, 2284, 2331, 2396},  // 2D box r1
        {604, 860, 890, 972, 0, 0, 0, 0},                 // 2D box r2
        {473, 478, 481, 473, 0, 0, 0, 0},                 // 2D box r3
        {315, 269, 275, 257, 0, 0, 0, 0},                 // 2D box r4
        {546, 1148, 1519, 1301, 0, 0, 0, 0},              // 3D star r1
        {556, 917, 0, 0, 0, 0, 0, 0},                     // 3D star r2
        {548, 771, 679, 530, 0, 0, 0, 0},                 // 3D box r1
    },
    {
        // F64
        {299, 574, 852, 1170, 0, 0, 0, 0},
        {296, 570, 859, 1171, 0, 0, 0, 0},
        {286, 580, 0, 0, 0, 0, 0, 0},
        {292, 319, 0, 0, 0, 0, 0, 0},
        {237, 168, 0, 0, 0, 0, 0, 0},
        {280, 517, 0, 0, 0, 0, 0, 0},
        {260, 446, 0, 0, 0, 0, 0, 0},
        {270, 511, 0, 0, 0, 0, 0, 0},
    },
    {
        // BF16
        {1504, 2724, 3144, 3129, 3041, 3103, 3068, 3084},
        {1453, 2261, 2306, 2362, 2268, 2252, 2244, 2232},
        {911, 971, 976, 999, 0, 0, 0, 0},
        {526, 549, 496, 463, 0, 0, 0, 0},
        {349, 284, 263, 255, 0, 0, 0, 0},
        {1002, 1490, 1545, 1241, 0, 0, 0, 0},
        {769, 913, 0, 0, 0, 0, 0, 0},
        {622, 818, 756, 516, 0, 0, 0, 0},
    },
    {
        // F16
        {1482, 2746, 2934, 2923, 3033, 3075, 3003, 2982},
        {1462, 2154, 2232, 2280, 2177, 2234, 2265, 2244},
        {898, 958, 991, 995, 0, 0, 0, 0},
        {519, 535, 495, 458, 0, 0, 0, 0},
        {347, 288, 268, 260, 0, 0, 0, 0},
        {992, 1365, 1445, 1164, 0, 0, 0, 0},
        {746, 886, 0, 0, 0, 0, 0, 0},
        {619, 788, 742, 511, 0, 0, 0, 0},
    },
};

// Measured rate of a launch fusing `levels` steps (0 when not measured or
// not built).
constexpr double kernel_rate(int dtype, int stencil, int levels) {
  return dtype >= 0 && dtype < 4 && stencil >= 0 && stencil < 8 && levels >= 1 && levels <= 8
             ? kRate[dtype][stencil][levels - 1]
             : 0.0;
}

// The rates by which the search for a round-at-store plan ranks (BF16, F16): a
// run of such a plan rounds once per launch, so that the depths found are part
// of its values, and of their accuracy.  They are the rates that those plans
// were first chosen by and are not measured again (up to a third below kRate
// in 2D, for wide boxes and few levels most).
constexpr double kRateAtStore[2][8][8] = {
    {
        // BF16
        {1538, 2584, 2846, 2923, 2700, 2729, 2744, 2659},
        {1423, 1950, 1993, 2019, 1899, 1914, 1906, 1911},
        {773, 832, 802, 799, 0, 0, 0, 0},
        {447, 413, 403, 384, 0, 0, 0, 0},
        {234, 224, 217, 198, 0, 0, 0, 0},
        {1004, 1330, 1486, 1234, 0, 0, 0, 0},
        {776, 914, 0, 0, 0, 0, 0, 0},
        {555, 802, 717, 514, 0, 0, 0, 0},
    },
    {
        // F16
        {1483, 2390, 2473, 2510, 2526, 2510, 2532, 2486},
        {1396, 1822, 1924, 1974, 1899, 1897, 1915, 1873},
        {729, 788, 772, 783, 0, 0, 0, 0},
        {427, 395, 386, 373, 0, 0, 0, 0},
        {228, 219, 214, 195, 0, 0, 0, 0},
        {993, 1290, 1414, 1162, 0, 0, 0, 0},
        {710, 876, 0, 0, 0, 0, 0, 0},
        {586, 769, 698, 510, 0, 0, 0, 0},
    },
};

// Fused depth (at most max_depth) for a plan that leaves k_on to the library.
// FP32 and FP64: the depth that costs least per level over grids from
// 400 x 400 to 12800 x 12800 (2D) and 64^3 to 640 x 512 x 256 (3D); deeper
// launches recompute more tile edges, which small grids have more of.  us per
// level on MI355X, (1201 x 1003, 12800 x 3360, 12800 x 12800):
//   FP32 2D 9-point box   5 levels 2.4 18.2 61.2, 6: 2.4 17.8 57.4, 8: 2.5 18.6 58.7
//   FP32 2D 25-point box  2 levels 4.5 43.4 147,  3: 4.6 42.0 139,  4: 4.9 42.4 139
//   FP32 2D 49-point box  1 level  8.0 87 296,    2: 8.4 78 261
//   FP32 2D 5-point star  6 levels 2.0 13.1 47.8, 7: 2.1 12.7 43.3, 8: 2.1 12.4 40.8
//   FP64 2D 49-point box  1 level  10.5 151 561,  2: 14.7 116 405 (4800 x 4800:
//     83 and 93): one level where a launch reads no more than the last-level
//     cache's 256 MiB (rows of 12800, 64, 96, 128, 160 and 280 MiB read: one
//     level 30 40 50 71 129, two 39 49 63 75 109)
// and for 251 x 190 x 163 and 640 x 512 x 256
//   FP64 3D 13-point star 1 level  29.3 288,      2: 20.1 198
// 16-bit storage: a round-at-store run rounds once per launch, so that its
// values depend on the depth, which is part of the plan's result and stays
// where it is (each is within 12 % of the best rate above).
constexpr int kDepth[4][8] = {
    {7, 6, 3, 2, 1, 3, 2, 2},
    {4, 4, 2, 2, 1, 2, 2, 2},
    {3, 3, 2, 1, 1, 3, 2, 2},
    {3, 3, 2, 1, 1, 3, 2, 2},
};
constexpr int preferred_depth(int dtype, int stencil, int max_depth, uint64_t launch_bytes) {
  int d = (dtype >= 0 && dtype < 4 && stencil >= 0 && stencil < 8) ? kDepth[dtype][stencil] : 1;
  if (dtype == 1 && stencil == 3 && launch_bytes <= (uint64_t)256 << 20) d = 1;
  return d < max_depth ? d : max_depth;
}

}  // namespace so2dr
