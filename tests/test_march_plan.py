"""The tile shape and the segments that 3D launches within the last-level
cache are given (march_plan.hpp, compiled for the host), against times
measured on MI355X: per launch (grid, stencil, storage, levels, output
planes), per shape its waves, rows per wave, cells per lane, tiles and resident
workgroups per CU, and us by number of segments."""
import subprocess

import pytest

from paper_2309_08864_amd import build as B

MEASURED = [
    ((512, 512, 'star', 1, 'f32', 1, 64), {
        "wide": ((16, 2, 4, 54, 2), {1: 66.4, 2: 37.1, 3: 27.6, 4: 24.1, 5: 32.7, 6: 33.1, 8: 30.6, 10: 33.3, 13: 34.1, 16: 29.9, 22: 35.6}),
        "narrow": ((8, 4, 1, 162, 4), {1: 42.5, 2: 31.8, 3: 26.2, 4: 27.6, 5: 30.4, 6: 32.1, 8: 31.5, 10: 32.1, 13: 35.1, 16: 31.5, 22: 38.6}),
        "small": ((4, 4, 1, 333, 8), {1: 35.7, 2: 26.4, 3: 26.1, 4: 27.6, 5: 27.5, 6: 29.3, 8: 30.1, 10: 30.6, 13: 33.7, 16: 30.9, 22: 37.4}),
    }),
    ((512, 512, 'star', 2, 'f64', 1, 40), {
        "wide": ((8, 4, 2, 95, 1), {1: 49.4, 2: 32.2, 3: 46.4, 4: 41.9, 5: 41.6, 6: 52.1, 8: 44.3, 10: 52.3, 14: 68.9, 20: 84.4}),
        "narrow": ((8, 4, 1, 171, 2), {1: 36.4, 2: 38.4, 3: 40.9, 4: 38.7, 5: 43.4, 6: 48.3, 8: 44.4, 10: 49.6, 14: 61.5, 20: 78.3}),
        "small": ((4, 4, 1, 387, 4), {1: 33.7, 2: 34.7, 3: 37.3, 4: 37.4, 5: 41.5, 6: 47.0, 8: 43.0, 10: 48.7, 14: 59.7, 20: 77.0}),
    }),
    ((512, 512, 'box', 1, 'f32', 2, 40), {
        "wide": ((8, 4, 2, 95, 2), {1: 90.6, 2: 51.4, 3: 65.9, 4: 51.9, 5: 45.2, 6: 57.8, 8: 49.2, 10: 54.7, 14: 68.2, 20: 77.3}),
        "narrow": ((8, 4, 1, 171, 4), {1: 56.9, 2: 51.8, 3: 53.5, 4: 42.9, 5: 47.5, 6: 51.1, 8: 51.1, 10: 50.8, 14: 61.0, 20: 72.7}),
        "small": ((4, 4, 1, 387, 8), {1: 54.4, 2: 50.0, 3: 45.6, 4: 46.6, 5: 46.0, 6: 49.6, 8: 51.9, 10: 53.9, 14: 62.6, 20: 74.1}),
        "narrow6": ((8, 6, 1, 108, 2), {1: 77.0, 2: 43.9, 3: 54.6, 4: 43.1, 5: 52.5, 6: 48.0, 8: 51.5, 10: 54.3, 14: 56.7, 20: 70.9}),
    }),
    ((1024, 512, 'star', 1, 'f64', 2, 24), {
        "wide": ((8, 4, 2, 171, 1), {1: 38.2, 2: 49.0, 3: 56.0, 4: 55.2, 5: 63.2, 6: 61.9, 8: 72.9, 12: 92.3}),
        "narrow": ((8, 4, 1, 342, 2), {1: 44.3, 2: 44.4, 3: 51.9, 4: 54.4, 5: 62.1, 6: 57.2, 8: 69.0, 12: 91.6}),
        "small": ((4, 4, 1, 774, 4), {1: 41.6, 2: 45.0, 3: 49.7, 4: 52.8, 5: 59.6, 6: 55.8, 8: 65.8, 12: 87.5}),
    }),
    ((1024, 512, 'star', 2, 'f64', 1, 24), {
        "wide": ((8, 4, 2, 171, 1), {1: 37.7, 2: 50.6, 3: 54.6, 4: 49.1, 5: 57.2, 6: 63.8, 8: 78.0, 12: 99.4}),
        "narrow": ((8, 4, 1, 342, 2), {1: 44.5, 2: 46.2, 3: 52.4, 4: 48.9, 5: 55.9, 6: 60.9, 8: 74.7, 12: 99.5}),
        "small": ((4, 4, 1, 774, 4), {1: 41.9, 2: 46.8, 3: 49.4, 4: 47.8, 5: 55.0, 6: 59.5, 8: 71.0, 12: 95.0}),
    }),
    ((640, 480, 'star', 1, 'f64', 2, 40), {
        "wide": ((8, 4, 2, 108, 1), {1: 54.9, 2: 36.7, 3: 52.4, 4: 42.5, 5: 57.9, 6: 50.5, 8: 62.5, 10: 60.1, 14: 73.1, 20: 92.0}),
        "narrow": ((8, 4, 1, 198, 2), {1: 40.1, 2: 42.4, 3: 47.1, 4: 44.8, 5: 47.7, 6: 48.4, 8: 58.0, 10: 53.5, 14: 66.6, 20: 85.8}),
        "small": ((4, 4, 1, 440, 4), {1: 37.6, 2: 42.8, 3: 43.5, 4: 41.7, 5: 47.9, 6: 47.9, 8: 54.4, 10: 53.7, 14: 65.9, 20: 83.8}),
    }),
    ((320, 320, 'star', 2, 'bf16', 2, 24), {
        "wide": ((8, 6, 2, 24, 1), {1: 62.4, 2: 40.0, 3: 31.9, 4: 27.2, 5: 25.6, 6: 24.1, 8: 22.8, 12: 38.4}),
        "narrow": ((8, 4, 1, 84, 2), {1: 32.4, 2: 21.9, 3: 18.1, 4: 21.9, 5: 20.6, 6: 19.8, 8: 25.4, 12: 30.2}),
        "small": ((4, 4, 1, 240, 5), {1: 23.6, 2: 20.6, 3: 20.4, 4: 20.7, 5: 22.5, 6: 24.5, 8: 27.9, 12: 35.1}),
        "narrow6": ((8, 6, 1, 48, 2), {1: 40.4, 2: 26.6, 3: 21.6, 4: 18.6, 5: 17.6, 6: 24.6, 8: 23.2, 12: 30.2}),
    }),
    ((256, 256, 'star', 1, 'f32', 3, 64), {
        "wide": ((8, 6, 2, 21, 1), {1: 116.3, 2: 65.2, 3: 48.2, 4: 38.5, 5: 33.5, 6: 31.1, 8: 26.6, 10: 24.4, 13: 38.8, 16: 35.1, 22: 33.3}),
        "narrow": ((8, 4, 1, 50, 3), {1: 61.1, 2: 35.0, 3: 26.6, 4: 21.8, 5: 19.3, 6: 24.6, 8: 21.3, 10: 19.6, 13: 21.7, 16: 23.9, 22: 25.9}),
        "small": ((4, 4, 1, 130, 6), {1: 45.0, 2: 33.5, 3: 25.3, 4: 24.9, 5: 22.0, 6: 23.7, 8: 22.9, 10: 23.3, 13: 23.1, 16: 24.3, 22: 27.5}),
    }),
    ((128, 128, 'star', 1, 'f32', 2, 64), {
        "wide": ((8, 4, 4, 5, 1), {1: 102.6, 2: 56.2, 3: 40.8, 4: 31.9, 5: 27.6, 6: 25.3, 8: 20.9, 10: 18.9, 13: 16.6, 16: 14.4, 22: 13.1}),
        "narrow": ((8, 4, 1, 15, 4), {1: 50.3, 2: 28.4, 3: 20.9, 4: 16.7, 5: 14.7, 6: 13.5, 8: 11.4, 10: 10.4, 13: 9.4, 16: 8.3, 22: 10.2}),
        "small": ((4, 4, 1, 33, 8), {1: 37.5, 2: 21.1, 3: 15.8, 4: 12.7, 5: 11.2, 6: 10.4, 8: 10.6, 10: 9.9, 13: 8.9, 16: 9.1, 22: 8.6}),
    }),
]

POINTS = {("star", 1): 7, ("star", 2): 13, ("box", 1): 27}
SIZE = {"f32": 4, "f64": 8, "bf16": 2}


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    """(shape arguments) -> (segments, cost), by the header itself."""
    d = tmp_path_factory.mktemp("march")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(r"""
#include <cstdio>
#include <cstdlib>
#include "march_plan.hpp"
using namespace so2dr;
int main(int, char **a) {
  auto I = [&](int k) { return std::atoi(a[k]); };
  // span tiles extra occ nw m vx kl npts wide box fp32 plane_bytes reread
  MarchMemory mem;
  mem.plane = std::atof(a[13]) / kCacheBytesPerCycle;
  mem.reread = I(14);
  const MarchPlan p = plan_march(I(1), I(2), I(3), 256, I(4), kMarchLatency, march_issue(I(5), I(6), I(7), I(8), I(9)), 1,
                                 I(10) ? wide_scale(I(11), I(12), I(8)) : 1.0, mem);
  std::printf("%d %.6g\n", p.nseg, p.cost);
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)

    def plan(*args):
        out = subprocess.run([str(exe)] + [str(int(x)) for x in args], capture_output=True, text=True, check=True)
        n, cost = out.stdout.split()
        return int(n), float(cost)
    return plan


def _near(times, n):
    """us at n segments, between the measured numbers on either side."""
    lo = max([k for k in times if k <= n], default=min(times))
    hi = min([k for k in times if k >= n], default=max(times))
    return times[lo] if lo == hi else times[lo] + (times[hi] - times[lo]) * (n - lo) / (hi - lo)


@pytest.mark.parametrize("launch,shapes", MEASURED, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else "")
def test_choice_is_near_the_best(planner, launch, shapes):
    nx, ny, shape, r, storage, kl, span = launch
    npts = POINTS[shape, r]
    best = None
    for name, ((nw, m, vx, tiles, occ), times) in shapes.items():
        if name == "wide" and shape == "box" and (storage == "f64" or kl == 1):
            continue      # not taken
        n, cost = planner(span, tiles, 2 * kl * r + kl - 1, occ, nw, m, vx, kl, npts, name == "wide", shape == "box",
                          storage != "f64", nx * ny * SIZE[storage], 2 * kl * r)
        if best is None or cost < best[0]:
            best = cost, name, n, _near(times, n)
    least = min(min(t.values()) for _, t in shapes.values())
    assert best[3] <= 1.12 * least, best
