"""Bit-for-bit parity of the tile shapes at the edges of their choice.

launch_any takes a wide shape (2 or 4 cells per lane) for launches whose
planes exceed the last-level cache and a narrow one (1 cell per lane, any row
length) otherwise and for rows that are not whole vectors; the cut axis is
split by a cost model into segments of any length.  Cases: rows and columns
just below, at and above the narrow tiles' output sizes (64 - 2 levels r
columns, 32 - 2 levels r rows), single rows and columns, odd rows, spans from
one plane up; and grids whose in and out planes exceed 256 MiB, with whole and
with odd rows.  2D rows of any length take one kernel whose waves load whole
vectors inside the row and single cells at its ends: lengths around the tile's
columns, shorter than a vector, and odd ones, so that every row starts at
another alignment.  FP32 and 16-bit results equal the C model of the documented
arithmetic bit for bit; FP64 agrees with the oracle to 1e-13 (a few hundred
FP64 roundings of weights that sum to at most 1)."""
import numpy as np
import pytest

import oracle

from helpers import fp32_weights, gpu_run, rel_l2, to_storage

pytestmark = pytest.mark.gpu

DEPTHS = {("star", 1): (1, 2, 3, 4), ("star", 2): (1, 2), ("box", 1): (1, 2, 4)}
DEPTHS_F64 = {("star", 1): (1, 2), ("star", 2): (1, 2), ("box", 1): (1, 2)}


def _check(shape, r, k_on, storage, nx, ny, nz, bc=(0, 0, 0), T=None, d=1, ndim=3):
    from oracle import emulator
    rng = np.random.default_rng(nx + 7 * ny + 31 * nz + 100 * r + k_on)
    offs = oracle.stencil_offsets(ndim, shape, r)
    w = rng.uniform(-1.0, 1.0, len(offs))
    w = w / np.abs(w).sum()
    if storage != "f64":
        w = fp32_weights(w)
    dims = (nz, ny, nx) if ndim == 3 else (ny, nx)
    us = to_storage(rng.standard_normal(dims, dtype=np.float32).astype(np.float64), storage)
    T = T or k_on
    kw = dict(ndim=ndim, nx=nx, ny=ny, nz=nz, shape=shape, radius=r, weights=list(w), T=T, tb_depth=T,
              n_chunks=d, k_on=k_on, budget=4 << 30, storage=storage, bc=bc)
    print(f"[{storage} {shape} r={r} k_on={k_on} T={T} d={d} bc={bc}] {nx}x{ny}x{nz}", flush=True)
    got, _, info = gpu_run(kw, us)
    assert info["k_on"] == k_on
    if storage == "f64":
        assert rel_l2(got.numpy(), oracle.sweep(us.numpy(), offs, w, T, bc)) <= 1e-13
        return
    model = emulator.sweep_bits_c(us.float().numpy(), offs, w, T, storage, bc)
    g = np.ascontiguousarray(got.float().numpy())
    assert int(np.sum(g.view(np.uint32) != model.view(np.uint32))) == 0


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("shape,r", sorted(DEPTHS))
def test_narrow_tiles_at_their_edges(shape, r, storage):
    for k in (DEPTHS_F64 if storage == "f64" else DEPTHS)[(shape, r)]:
        ox, oy = 64 - 2 * k * r, 32 - 2 * k * r
        _check(shape, r, k, storage, ox - 1, oy + 1, 9)
        _check(shape, r, k, storage, ox, oy, 1)
        _check(shape, r, k, storage, 2 * ox + 1, 2 * oy - 1, 23, bc=(1, 1, 0))
        _check(shape, r, k, storage, 1, 3, 40, T=2 * k)
        _check(shape, r, k, storage, 301, 1, 5, bc=(1, 0, 0))
        _check(shape, r, k, storage, 131, 53, 8 * k * r + 3, T=2 * k, d=2, bc=(0, 1, 0))


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16"])
@pytest.mark.parametrize("shape,r", sorted(DEPTHS))
def test_tiles_of_grids_beyond_the_cache(shape, r, storage):
    nx, ny = 1032, 1030
    nz = {2: 72, 4: 36, 8: 20}[{"f32": 4, "f64": 8, "bf16": 2}[storage]]
    for k in (DEPTHS_F64 if storage == "f64" else DEPTHS)[(shape, r)]:
        _check(shape, r, k, storage, nx, ny, nz)
    _check(shape, r, 2, storage, nx - 2, ny, nz)         # an odd number of 2-cell vectors
    _check(shape, r, 2, storage, nx - 1, ny, nz, bc=(1, 1, 0))


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("shape,r", [("star", 1), ("box", 1), ("box", 2), ("box", 3), ("box", 4)])
def test_2d_rows_of_any_length(shape, r, storage):
    deepest = {("star", 1): 8, ("box", 1): 8}.get((shape, r), 4)
    if storage == "f64":
        deepest //= 2
    for k in sorted({1, 2, deepest - 1, deepest}):
        ox = (128 if storage == "f64" else 256) - 2 * ((k * r + 3) // 4 * 4)
        for i, nx in enumerate([1, 3, ox - 1, ox + 1, 2 * ox + 3, 1021]):
            ny = 4 * k * r + 1 + i
            _check(shape, r, k, storage, nx, ny, 1, bc=(i & 1, 0, 0), T=2 * k, ndim=2)
        _check(shape, r, k, storage, 517, 8 * k * r + 5, 1, T=2 * k, d=2, ndim=2)
