"""The LDS-plane kernel, which only planes (2D: rows) of 4 GiB and more take by
themselves: every stencil, storage type and depth through the testing aid
so2dr_plan_set_plane_kernel, bit for bit against the march kernels (the same
sums in the same order)."""
import numpy as np
import pytest
import torch

from helpers import STENCIL_CASES, np_shape, pinned_copy, to_storage
from paper_2309_08864_amd import Plan, _lib, stencil_offsets

pytestmark = pytest.mark.gpu


def _plane_kernel(p):
    assert _lib.lib().so2dr_plan_set_plane_kernel(p._h, 1) == 0


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("ndim,shape,r", STENCIL_CASES)
def test_every_depth_bitwise(ndim, shape, r, storage):
    """Odd rows over several tiles and segments; periodic in x where a box."""
    offs = stencil_offsets(ndim, shape, r)
    rng = np.random.default_rng(31 + r)
    w = list(rng.random(len(offs)) / len(offs))
    nx, ny, nz = (1101, 83, 1) if ndim == 2 else (77, 45, 41)
    u = to_storage(rng.random(np_shape(ndim, nx, ny, nz)), storage)
    kw = dict(ndim=ndim, nx=nx, ny=ny, nz=nz, shape=shape, radius=r, weights=w, storage=storage, budget=1 << 30,
              bc=(1 if shape == "box" else 0, 0, 0), n_chunks=2)
    deepest = Plan(T=1, tb_depth=1, **kw).info()["max_k_on"]
    for k_on in range(1, deepest + 1):
        print(f"{ndim}D {shape} r={r} {storage} levels {k_on}", flush=True)
        K = k_on + 1 if 4 * r * (k_on + 1) <= (ny if ndim == 2 else nz) else k_on
        p = Plan(T=2 * K, tb_depth=K, k_on=k_on, **kw).bind()
        want, got = pinned_copy(u), pinned_copy(u)
        p.run(want)
        _plane_kernel(p)
        p.run(got)
        p.close()
        assert torch.equal(got, want), k_on


@pytest.mark.parametrize("storage", ["bf16", "f16"])
@pytest.mark.parametrize("ndim,shape,r", [(2, "box", 1), (3, "star", 2)])
def test_round_at_store_bitwise(ndim, shape, r, storage):
    offs = stencil_offsets(ndim, shape, r)
    rng = np.random.default_rng(37)
    w = list(rng.random(len(offs)) / len(offs))
    nx, ny, nz = (1030, 40, 1) if ndim == 2 else (70, 35, 20)
    u = to_storage(rng.random(np_shape(ndim, nx, ny, nz)), storage)
    p = Plan(ndim=ndim, nx=nx, ny=ny, nz=nz, shape=shape, radius=r, weights=w, storage=storage, T=5, tb_depth=5, k_on=2,
             n_chunks=1, rounding="at_store", budget=1 << 30).bind()
    want, got = pinned_copy(u), pinned_copy(u)
    p.run(want)
    _plane_kernel(p)
    p.run(got)
    p.close()
    assert torch.equal(got, want)


def test_gradient_bitwise():
    offs = stencil_offsets(3, "box", 1)
    rng = np.random.default_rng(41)
    w = list(rng.random(len(offs)) / len(offs))
    u, y = (to_storage(rng.random((30, 33, 61)), "f64") for _ in range(2))
    res = []
    for aid in (False, True):
        p = Plan(ndim=3, nx=61, ny=33, nz=30, shape="box", radius=1, weights=w, storage="f64", T=6, tb_depth=3, n_chunks=3,
                 adjoint=True, budget=1 << 30).bind()
        if aid:
            _plane_kernel(p)
        loss, gu, gw, _ = p.adjoint(pinned_copy(u), pinned_copy(y), 3)
        res.append((loss, gu.clone(), gw.copy()))
        p.close()
    assert res[0][0] == res[1][0] and torch.equal(res[0][1], res[1][1]) and np.array_equal(res[0][2], res[1][2])
