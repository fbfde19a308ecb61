"""The automatic fused depth of FP64 radius-3 boxes goes by what one launch
reads, the tallest chunk with its halo, not by the whole field."""
import pytest

from paper_2309_08864_amd import Plan, So2drError

MIB = 1 << 20


def _plan(ny, d, K=8, budget=64 << 30, **kw):
    return Plan(ndim=2, nx=12800, ny=ny, shape="box", radius=3, weights=[1 / 49] * 49, T=K, tb_depth=K, n_chunks=d,
                storage="f64", budget=budget, **kw)


@pytest.mark.parametrize("ny,d,k_on", [
    (2600, 1, 1),        # 254 MiB
    (2700, 1, 2),        # 264 MiB
    (12800, 1, 2),
    (12800, 4, 2),       # 3200 + 48 rows: 317 MiB
    (12800, 5, 1),       # 2560 + 48 rows: 255 MiB
    (12800, 16, 1),      # 83 MiB
])
@pytest.mark.parametrize("adjoint", [False, True])
def test_depth_by_the_launch(ny, d, k_on, adjoint):
    i = _plan(ny, d, adjoint=adjoint).info()
    assert i["k_on"] == k_on and not i["lean"]
    assert _plan(ny, d, k_on=2, adjoint=adjoint).info()["k_on"] == 2      # a depth asked for is kept


def test_one_buffer_plans_keep_a_depth_that_fits():
    """One level needs more spare planes than two: a one-buffer plan that only
    two levels fit keeps them, and with room takes one."""
    kw = dict(ny=12800, d=16, n_slots=1)
    full = _plan(**kw).info()["workspace_bytes"]
    lo, hi = 0, full - 1
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        try:
            _plan(budget=mid, **kw)
            hi = mid
        except So2drError:
            lo = mid
    two = lo, hi
    lo, hi = 0, full - 1
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        try:
            _plan(budget=mid, k_on=2, **kw)
            hi = mid
        except So2drError:
            lo = mid
    assert two == (lo, hi)
    least, roomy = _plan(budget=hi, **kw).info(), _plan(budget=full - 1, **kw).info()
    assert least["lean"] and least["k_on"] == 2 and least["workspace_bytes"] <= hi
    assert roomy["lean"] and roomy["k_on"] == 1 and roomy["workspace_bytes"] < full
