"""Weight gradients over rows of every kind the reduction kernel tells apart:
whole 4-cell vectors, rows that are not (one cell per lane), rows shorter than
the stencil, periodic wraps, fewer vectors than lanes and several per lane, and
rounds deep enough that recomputed levels are reused.  FP64 storage against
the FP64 oracle; the bound is the one the gradient tests use (1e-10: some
1e5 FP64 roundings, with up to 1e3 of cancellation in a component)."""
import numpy as np
import pytest

import oracle
from helpers import STENCIL_CASES, pinned_copy, rel_l2, to_storage
from paper_2309_08864_amd import Plan

pytestmark = pytest.mark.gpu


def _case(ndim, shape, r, nx, ny, nz, T, K, d, per, k_on=0):
    rng = np.random.default_rng(nx + 10 * r + 100 * T)
    offs = oracle.stencil_offsets(ndim, shape, r)
    w = rng.uniform(0.2, 1.0, len(offs))
    w = w / w.sum()
    shp = (nz, ny, nx) if ndim == 3 else (ny, nx)
    u0, y = to_storage(rng.random(shp), "f64"), to_storage(rng.random(shp), "f64")
    print(f"[{ndim}D {shape} r={r}] {nx}x{ny}x{nz} T={T} K={K} d={d} per={per}", flush=True)
    p = Plan(ndim=ndim, nx=nx, ny=ny, nz=nz, shape=shape, radius=r, weights=list(w), T=T, tb_depth=K,
             n_chunks=d, k_on=k_on, budget=1 << 30, storage="f64", bc=per, adjoint=True).bind()
    loss, gu, gw, _ = p.adjoint(pinned_copy(u0), pinned_copy(y), T)
    p.close()
    rl, rgu, rgw, _ = oracle.adjoint(u0.numpy(), y.numpy(), offs, w, T, per)
    den = np.maximum(np.abs(rgw), 1e-3 * np.abs(rgw).max())
    assert abs(loss - rl) <= 1e-10 * abs(rl)
    assert rel_l2(gu.numpy(), rgu) <= 1e-10
    assert np.max(np.abs(gw - rgw) / den) <= 1e-10


@pytest.mark.parametrize("ndim,shape,r", STENCIL_CASES)
def test_weight_gradient_rows(ndim, shape, r):
    for i, nx in enumerate([1, 2, 4, 5, 8, 67, 72, 1030]):
        n = 8 * r + 1 + i
        if ndim == 3:
            _case(3, shape, r, nx, 5 + i, n, 4, 2, 2, (i & 1, (i >> 1) & 1, 0))
        else:
            _case(2, shape, r, nx, n, 1, 4, 2, 2, (i & 1, 0, 0))


@pytest.mark.parametrize("k_on", [1, 2, 4])
def test_deep_rounds_reuse_levels(k_on):
    _case(2, "star", 1, 516, 260, 1, 33, 17, 3, (0, 0, 0), k_on)
    _case(2, "box", 1, 131, 150, 1, 16, 16, 1, (1, 0, 0), k_on)
