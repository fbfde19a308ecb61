"""The segments that 2D launches within the last-level cache are given
(march_plan.hpp, compiled for the host), against times measured on MI355X with
four cells per lane (FP64: two): row length, stencil, storage, levels, output
rows; tiles, resident workgroups per CU, cells per lane; us by number of
segments.  Where the cache binds, more segments only re-read rows."""
import subprocess

import pytest

from paper_2309_08864_amd import build as B

MEASURED = [
    ((12800, "star", 1, "f32", 1, 800), (52, 8, 4),
     {17: 16.5, 21: 16.6, 25: 15.3, 34: 14.7, 40: 15.4, 50: 13.9, 67: 14.7, 80: 15.5, 100: 17.3, 134: 16.6}),
    ((4800, "star", 1, "f32", 2, 3200), (20, 8, 4),
     {48: 24.8, 60: 25.4, 72: 23.2, 95: 21.4, 119: 23.1, 140: 22.1, 189: 23.1, 229: 24.7, 267: 25.5, 356: 26.4}),
    ((6400, "star", 1, "f32", 1, 1600), (26, 8, 4),
     {35: 16.6, 43: 16.3, 52: 15.1, 70: 14.6, 85: 15.2, 100: 14.1, 134: 14.7, 160: 15.1, 200: 17.2, 267: 16.6}),
    ((12800, "box", 2, "f64", 1, 800), (104, 7, 2),
     {8: 32.1, 12: 29.8, 17: 27.6, 21: 29.9, 25: 28.4, 34: 29.1, 40: 30.3, 50: 30.3, 67: 33.9, 80: 32.4}),
]
POINTS = {("star", 1): 5, ("box", 1): 9, ("box", 2): 25}


@pytest.mark.parametrize("launch,tiles,times", MEASURED, ids=lambda v: "-".join(map(str, v)) if len(v) == 6 else "")
def test_segments_are_near_the_best(tmp_path, launch, tiles, times):
    nx, shape, r, storage, kl, span = launch
    size = 8 if storage == "f64" else 4
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    issue = 4.0 * (kl * (tiles[2] * POINTS[shape, r] + 4.0) + 10.0)
    src.write_text(f"""
#include <cstdio>
#include "march_plan.hpp"
using namespace so2dr;
int main() {{
  MarchMemory mem;
  mem.plane = {nx * size} / kCacheBytesPerCycle2d;
  mem.reread = {2 * kl * r};
  const MarchPlan p = plan_march({span}, {tiles[0]}, {2 * kl * r + kl - 1}, 256, {tiles[1]}, 900.0, {issue}, 4, 1.0, mem);
  std::printf("%d", p.nseg);
}}
""")
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    n = int(subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout)
    lo = max([k for k in times if k <= n], default=min(times))
    hi = min([k for k in times if k >= n], default=max(times))
    t = times[lo] if lo == hi else times[lo] + (times[hi] - times[lo]) * (n - lo) / (hi - lo)
    assert t <= 1.12 * min(times.values()), (n, t)
