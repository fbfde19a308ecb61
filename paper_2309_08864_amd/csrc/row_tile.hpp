// row_tile.hpp -- the columns of a 2D tile: plain constant expressions, shared
// by the kernels and by whoever enumerates them on the host.
#pragma once

namespace so2dr {

// A wave's tile: 64 lanes of VX consecutive cells, the outer HX on either side
// overlapping the neighbouring tiles.
template <int R, int KL, int VX>
struct RowTile {
  static constexpr int TX = 64 * VX;
  static constexpr int HX = (KL * R + VX - 1) / VX * VX;
  static constexpr int OX = TX - 2 * HX;
  static_assert(R <= 2 * VX && OX > 0, "tile too small for this depth");
};

// First column of tile `i` of a row of nx cells.  A tile that reaches past the
// end of a row that is not whole vectors starts up to VX - 1 cells further left,
// so that a lane ends where the row does; where that would take it past the
// row's start too, it stays and its lanes go cell by cell (cells).
struct RowStart {
  int x_lo;
  bool cells;
};
template <typename G, int VX>
constexpr RowStart row_start(int i, int nx) {
  const int x_lo = i * G::OX - G::HX, over = nx % VX;
  if (over == 0 || x_lo + G::TX <= nx) return {x_lo, false};
  if (x_lo < VX) return {x_lo, true};
  return {x_lo - (VX - over), false};
}

// Where in its row a lane whose cells start at column gx reads `n` cells: at gx
// inside the row, beyond it at the wrapped column or (ghosts) at 0.  A row a few
// cells longer than a tile's output wraps twice within the last tile, and there
// the n cells may straddle the row's end: such lanes lie beyond the halo, no
// stored cell needs them, and they read the row's last n cells instead.
constexpr int row_source(int gx, int nx, int n, bool wrap) {
  if (gx >= 0 && gx < nx) return gx;
  if (!wrap) return 0;
  const int lx = ((gx % nx) + nx) % nx;
  return lx + n <= nx ? lx : nx - n;
}

}  // namespace so2dr
