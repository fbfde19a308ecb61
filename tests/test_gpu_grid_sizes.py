"""The tile shapes on both sides of their choice by grid size: grids that fill
the chip (2D: four cells per lane in FP32 and 16 bits; 3D: 8 waves of 4 rows)
with odd rows, and ones that do not (two cells per lane; 4 waves) at the small
shapes' tile edges (2D 128 cells less the halos, 3D 16 rows less the halos).
Against the C model of the documented arithmetic bit for bit, FP64 against the
oracle within 1e-13."""
import pytest

from test_gpu_tile_shapes import DEPTHS, DEPTHS_F64, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("shape,r", sorted(DEPTHS))
def test_3d_sizes(shape, r, storage):
    for k in (DEPTHS_F64 if storage == "f64" else DEPTHS)[(shape, r)]:
        oy = 16 - 2 * k * r
        _check(shape, r, k, storage, 65, oy, 7)
        _check(shape, r, k, storage, 63 - 2 * k * r, 2 * oy + 1, 12, bc=(1, 1, 0), T=2 * k)
        _check(shape, r, k, storage, 163, 130, 129)


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("shape,r", [("star", 1), ("box", 1), ("box", 2), ("box", 3), ("box", 4)])
def test_2d_sizes(shape, r, storage):
    deepest = {("star", 1): 8, ("box", 1): 8}.get((shape, r), 4)
    if storage == "f64":
        deepest //= 2
    for k in sorted({1, 2, deepest}):
        ox = 128 - 2 * ((k * r + 1) // 2 * 2)
        for i, nx in enumerate([ox - 1, ox, ox + 1, 2 * ox + 3]):
            _check(shape, r, k, storage, nx, 29 + 2 * k * r + i, 1, bc=(i & 1, 0, 0), T=2 * k, ndim=2)
    for k, nx, ny in ((deepest, 2051, 1301), (1, 4097, 2050)):
        _check(shape, r, k, storage, nx, ny, 1, ndim=2)
