"""The columns that the 2D kernels' lanes read, for every row length up to
several tiles, every tile shape and both boundary rules: each read lies inside
its row, the cells that a stored output depends on come from the column they
stand for, and every column is stored by some tile.  The kernels' own header
is compiled for the host and enumerated.  On the GPU, rows one to three cells
longer than a tile's output, whose last lanes wrap twice, against single-step
launches."""
import subprocess

import numpy as np
import pytest

from paper_2309_08864_amd import build as B

SOURCE = r"""
#include <cstdio>
#include "row_tile.hpp"
using namespace so2dr;

template <int R, int KL, int VX>
static int check() {
  if constexpr (R <= 2 * VX && 64 * VX > 2 * ((KL * R + VX - 1) / VX * VX)) {
    using G = RowTile<R, KL, VX>;
    int bad = 0;
    auto fail = [&](const char *what, int nx, int i, int gx, int src) {
      if (++bad <= 3) std::printf("R=%d KL=%d VX=%d nx=%d tile %d column %d reads %d: %s\n", R, KL, VX, nx, i, gx, src, what);
    };
    for (int nx = 1; nx <= 4 * G::TX + 40; ++nx)
      for (int wrap = 0; wrap < 2; ++wrap) {
        int stored = 0;   // columns [0, stored) have been stored
        for (int i = 0; i < (nx + G::OX - 1) / G::OX; ++i) {
          const RowStart s = row_start<G, VX>(i, nx);
          const int n = s.cells ? 1 : VX;   // cells of one read
          const int o0 = s.x_lo + G::HX, o1 = s.x_lo + G::TX - G::HX < nx ? s.x_lo + G::TX - G::HX : nx;
          if (o0 > stored) fail("column never stored", nx, i, stored, 0);
          stored = o1;
          for (int gx = s.x_lo; gx < s.x_lo + G::TX; gx += n) {
            const int src = row_source(gx, nx, n, wrap != 0);
            if (src < 0 || src + n > nx) fail("outside the row", nx, i, gx, src);
            for (int j = 0; j < n; ++j) {
              const int x = gx + j;
              if (x < o0 - KL * R || x >= o1 + KL * R) continue;   // no stored output needs it
              const bool in = x >= 0 && x < nx;
              if (in != (gx >= 0 && gx < nx)) fail("a read across the row's end", nx, i, gx, src);
              if ((in || wrap) && src + j != ((x % nx) + nx) % nx) fail("another column", nx, i, gx, src);
            }
          }
        }
        if (stored != nx) fail("columns left out", nx, -1, stored, 0);
      }
    return bad;
  } else {
    return 0;
  }
}
template <int VX>
static int all() {
  return check<1, 1, VX>() + check<1, 2, VX>() + check<1, 3, VX>() + check<1, 4, VX>() + check<1, 5, VX>() +
         check<1, 6, VX>() + check<1, 7, VX>() + check<1, 8, VX>() + check<2, 1, VX>() + check<2, 2, VX>() +
         check<2, 3, VX>() + check<2, 4, VX>() + check<3, 1, VX>() + check<3, 2, VX>() + check<3, 3, VX>() +
         check<3, 4, VX>() + check<4, 1, VX>() + check<4, 2, VX>() + check<4, 3, VX>() + check<4, 4, VX>();
}
int main() {
  const int bad = all<2>() + all<4>();
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_reads_stay_in_their_row(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("storage,shape,r,k_on,nx", [
    ("f64", "star", 1, 4, 121), ("f64", "box", 2, 2, 121), ("f64", "box", 4, 1, 121),
    ("f32", "star", 1, 7, 113), ("f32", "star", 1, 7, 242), ("f32", "box", 3, 2, 243), ("f32", "box", 4, 1, 121),
    ("bf16", "box", 2, 3, 241), ("f16", "box", 1, 6, 117),
])
def test_rows_just_past_a_tile_bitwise(storage, shape, r, k_on, nx):
    """The same sums in the same order whatever the depth: bit for bit."""
    import torch
    from helpers import gpu_run, to_storage
    from paper_2309_08864_amd import stencil_offsets
    offs = stencil_offsets(2, shape, r)
    rng = np.random.default_rng(nx + r)
    w = list(rng.random(len(offs)) / len(offs))
    u = to_storage(rng.random((151, nx)), storage)
    kw = dict(ndim=2, nx=nx, ny=151, shape=shape, radius=r, weights=w, T=k_on * 2, tb_depth=k_on * 2, n_chunks=1,
              storage=storage, bc=(1, 0, 0), budget=1 << 30)
    got, _, _ = gpu_run(dict(kw, k_on=k_on), u)
    # a row twice as long holds the periodic row twice; its lanes end elsewhere
    two, _, _ = gpu_run(dict(kw, nx=2 * nx, k_on=1), torch.cat([u, u], dim=1).contiguous())
    assert torch.equal(got, two[:, :nx]) and torch.equal(got, two[:, nx:])
