"""One-buffer ("lean") plans and so2dr_run_noalloc: growing the sub-blocks
must not take a plan out of the static workspace that its least layout fits."""
import numpy as np
import pytest

from paper_2309_08864_amd import Plan
from paper_2309_08864_amd._lib import NOALLOC_MAX_BYTES

MIB = 1 << 20


def _kw(ny, budget_mib, T=64):
    return dict(ndim=2, nx=4096, ny=ny, shape="star", radius=1, weights=[0.2] * 5, T=T, tb_depth=T, n_chunks=1,
                budget=budget_mib * MIB)


@pytest.mark.parametrize("budget_mib", [110, 127, 140, 180, 195])
def test_growth_stops_at_the_static_workspace(budget_mib):
    """The least layout takes 104 MiB: the plan is not grown beyond the 128
    that so2dr_run_noalloc has, whatever the budget, and what the smaller of
    the two leaves is still spent on taller blocks."""
    i = Plan(**_kw(6400, budget_mib)).info()
    assert i["lean"] == 1 and i["lean_block"] > 16
    assert i["workspace_bytes"] <= min(budget_mib * MIB, NOALLOC_MAX_BYTES)


def test_growth_beyond_the_static_workspace():
    """A least layout above the static workspace grows up to the budget."""
    i = Plan(**_kw(12800, 390)).info()
    assert i["lean"] == 1 and i["lean_block"] > 1000
    assert NOALLOC_MAX_BYTES < i["workspace_bytes"] <= 390 * MIB


@pytest.mark.gpu
def test_lean_plan_runs_without_allocation():
    """Under a budget above the static workspace; the bits of the two-buffer
    plan."""
    import torch
    from helpers import gpu_run, pinned_copy, to_storage
    u = to_storage(np.random.default_rng(3).random((6400, 4096)), "f32")
    want, _, i = gpu_run(_kw(6400, 1024, T=16), u)
    assert i["lean"] == 0
    p = Plan(**_kw(6400, 180, T=16))
    assert p.info()["lean"] == 1
    h = pinned_copy(u)
    p.run_noalloc(h)
    p.close()
    assert torch.equal(h, want)
