"""One-buffer ("lean") plans spend what their budget leaves on taller
sub-blocks; every budget between the least one and the two-buffer layout has
to give a schedule that stays inside its buffers and replays to the oracle's
values (FP64 on both sides: 16 steps of at most 25 FMAs, far below 1e-12)."""
import numpy as np
import pytest

import oracle
from paper_2309_08864_amd import Plan, So2drError
from paper_2309_08864_amd import stencil_offsets
from test_planner import simulate


@pytest.mark.parametrize("ndim,shape,r,n,T,K,d,k_on,slots", [
    (2, "star", 1, 256, 10, 4, 4, 4, 1),
    (2, "box", 2, 211, 7, 3, 3, 2, 1),
    (3, "star", 1, 150, 9, 4, 3, 2, 2),
    (3, "box", 1, 33, 5, 5, 1, 2, 1),
])
def test_lean_blocks_fill_the_budget(ndim, shape, r, n, T, K, d, k_on, slots):
    offs = stencil_offsets(ndim, shape, r)
    rng = np.random.default_rng(5)
    w = rng.random(len(offs)) / len(offs)
    kw = dict(ndim=ndim, nx=16, ny=n if ndim == 2 else 5, nz=1 if ndim == 2 else n, shape=shape, radius=r,
              weights=list(w), T=T, tb_depth=K, n_chunks=d, k_on=k_on, n_slots=slots, storage="f64")
    full = Plan(budget=1 << 30, **kw).info()
    lo, hi = 0, full["workspace_bytes"] - 1          # least budget that any plan fits, by bisection
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            Plan(budget=mid, **kw)
            hi = mid
        except So2drError:
            lo = mid
    u0 = rng.random((n, 1 if ndim == 2 else 5, 16))
    ref = oracle.sweep(u0[:, 0, :] if ndim == 2 else u0, offs, w, T)
    ref = ref[:, None, :] if ndim == 2 else ref
    blocks, ops = [], []
    for budget in np.linspace(hi, full["workspace_bytes"] - 1, 7).astype(int):
        p = Plan(budget=int(budget), **kw)
        i = p.info()
        assert i["lean"] == 1 and i["workspace_bytes"] <= budget
        blocks.append(i["lean_block"])
        ops.append(i["n_ops"])
        host, lv = simulate(p, offs, w, u0, 0, 0, ndim)
        assert np.all(lv == T) and np.allclose(host, ref, rtol=1e-12, atol=1e-12)
    assert blocks == sorted(blocks) and ops == sorted(ops, reverse=True)
    assert blocks[-1] > blocks[0] and ops[-1] < ops[0]
