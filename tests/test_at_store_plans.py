"""The depths that the plan search finds for round-at-store plans.  Such a run
rounds once per launch and at the end of each round, so that tb_depth and
k_on decide its values: they stay what they were when the kernels or the
copies become faster.  (tb_depth, n_chunks, k_on, n_slots) as first found."""
import pytest

from paper_2309_08864_amd import Plan, stencil_offsets, suggest

MIB = 1 << 20

# storage, ndim, grid, shape, radius, T, budget as a share of the field -> found
FOUND = [
    ("bf16", 3, (512, 512, 512), "star", 2, 64, 0.3, (4, 29, 2, 2)),      # one-buffer plans
    ("bf16", 3, (2048, 1024, 1024), "star", 1, 64, 0.3, (16, 29, 3, 2)),
    ("f16", 3, (512, 512, 512), "box", 1, 64, 0.3, (8, 29, 2, 2)),
    ("bf16", 2, (12800, 12800, 1), "box", 4, 40, 0.3, (20, 17, 2, 2)),
    ("bf16", 2, (12800, 12800, 1), "box", 4, 40, 0.6, (10, 11, 2, 3)),
    ("f16", 2, (12800, 12800, 1), "box", 4, 40, 8, (10, 4, 1, 3)),
    ("f16", 2, (12800, 12800, 1), "box", 1, 160, 0.6, (80, 12, 7, 3)),
    ("bf16", 2, (12800, 12800, 1), "box", 2, 80, 0.3, (40, 17, 4, 2)),
]


def _kw(storage, ndim, grid, shape, r, T, share):
    n = len(stencil_offsets(ndim, shape, r))
    return dict(ndim=ndim, nx=grid[0], ny=grid[1], nz=grid[2], shape=shape, radius=r, weights=[1.0 / n] * n, T=T,
                storage=storage, budget=int(grid[0] * grid[1] * grid[2] * 2 * share) + MIB)


@pytest.mark.parametrize("case", FOUND, ids=lambda c: f"{c[0]}-{c[1]}d-{c[3]}{c[4]}-{c[6]}")
def test_found_depths_stay(case):
    kw, ms = suggest(rounding="at_store", **_kw(*case[:-1]))
    assert (kw["tb_depth"], kw["n_chunks"], kw["k_on"], kw["n_slots"]) == case[-1]
    # the time is the plan's own prediction, by the present figures
    assert ms == pytest.approx(Plan(**kw).predict(), rel=1e-9)
    # runs that round every step do not depend on the schedule: the fastest is taken
    _, every = suggest(**_kw(*case[:-1]))
    assert every <= ms * 1.01
