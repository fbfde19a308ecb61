"""One level of a 2D box of radius 3 or 4 runs four input rows per step and
skips the rows of weights that none of a segment's outputs needs: grids of
every remainder of four rows, down to one row, in one segment and in several,
whole vectors and odd rows, give the bits of the C model of the documented
arithmetic (FP64: the oracle within 1e-13), as do rows that hold infinities
and NaN next to rows that must not see them."""
import numpy as np
import pytest
import torch

from helpers import gpu_run
from test_gpu_tile_shapes import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("r", [3, 4])
def test_rows_of_every_remainder(r, storage):
    for i, ny in enumerate([1, 2, 3, 5, 2 * r, 2 * r + 3, 40, 41, 42, 43, 1030]):
        _check("box", r, 1, storage, (300, 301, 516)[i % 3], ny, 1, bc=(i & 1, 0, 0), T=2, ndim=2)
    _check("box", r, 1, storage, 260, 203, 1, T=4, d=3, ndim=2)


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("r", [3, 4])
def test_non_finite_rows_stay_local(r, storage):
    dt = torch.float32 if storage == "f32" else torch.float64
    u = torch.rand(515, 400, dtype=dt)
    bad = u.clone()
    bad[250] = float("nan")
    bad[97, 33] = float("inf")
    n = (2 * r + 1) ** 2
    kw = dict(ndim=2, nx=400, ny=515, nz=1, shape="box", radius=r, weights=[1.0 / n] * n, T=1, tb_depth=1, n_chunks=1,
              k_on=1, budget=1 << 30, storage=storage)
    a, _, _ = gpu_run(kw, u)
    b, _, _ = gpu_run(kw, bad)
    near = torch.zeros(515, 400, dtype=torch.bool)
    near[250 - r:250 + r + 1] = True
    near[97 - r:97 + r + 1, 33 - r:33 + r + 1] = True
    assert torch.equal(a[~near], b[~near]) and not torch.isfinite(b[near]).any()
