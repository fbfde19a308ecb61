"""Predictions of plans whose copies and launches share one stream: each
operation follows the one before, each copy goes at its direction's own rate."""
import pytest

from paper_2309_08864_amd import Plan


def _chain_ms(p, elem):
    i, m = p.info(), p.machine()
    t = 0.0
    for op in p.ops():
        n = (op["z1"] - op["z0"]) * i["plane_elems"]
        if op["kind"] == "H2D":
            t += n * elem / (m["h2d_gbps"] * 1e9)
        elif op["kind"] == "D2H":
            t += n * elem / (m["d2h_gbps"] * 1e9)
        elif op["kind"] == "KERNEL":
            t += m["launch_us"] * 1e-6 + n * op["levels"] / (m["gupd"][op["levels"] - 1] * 1e9)
        else:
            t += m["launch_us"] * 1e-6 + 2 * n * elem / (m["d2d_gbps"] * 1e9)
    return 1e3 * t


@pytest.mark.parametrize("d,T,K,engine", [
    (1, 8, 8, 2),        # one slot
    (4, 9, 3, 2),        # three slots, pieces below half a MiB
    (8, 12, 4, 2),
    (16, 48, 4, 3),      # more than 256 copies: out by kernels, still on one stream
])
def test_serial_plans_are_predicted_as_a_chain(d, T, K, engine):
    p = Plan(ndim=3, nx=64, ny=40, nz=160, shape="star", radius=1, weights=[1 / 7] * 7, T=T, tb_depth=K, n_chunks=d,
             budget=1 << 30)
    assert p.info()["copy_engine"] == engine and p.info()["n_slots"] == min(3, d)
    # rounds after the third are extrapolated
    assert p.predict() == pytest.approx(_chain_ms(p, 4), rel=1e-6)


def test_overlapping_plans_are_predicted_shorter_than_their_chain():
    p = Plan(ndim=3, nx=64, ny=40, nz=160, shape="star", radius=1, weights=[1 / 7] * 7, T=12, tb_depth=4, n_chunks=8,
             budget=1 << 30, copy_engine="dma")
    assert p.predict() < 0.9 * _chain_ms(p, 4)
