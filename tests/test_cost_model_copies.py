"""Predictions of sweeps that the link binds, against times measured on
MI355X: 7-point FP32, 1024 x 512 x 512, 16 steps of K = 8, three slots."""
import pytest

from paper_2309_08864_amd import Plan


@pytest.mark.parametrize("chunks,engine,measured_ms", [
    (16, "dma", 45.4), (16, "kernel", 66.3), (16, "kernel_out", 50.2),      # 64 MiB per copy
    (32, "dma", 45.7), (32, "kernel", 69.9), (32, "kernel_out", 52.1),      # 32 MiB
])
def test_prediction_near_the_measurement(chunks, engine, measured_ms):
    p = Plan(ndim=3, nx=1024, ny=512, nz=512, shape="star", radius=1, weights=[1 / 7] * 7, T=16, tb_depth=8,
             n_chunks=chunks, budget=4 << 30, copy_engine=engine)
    assert p.info()["n_slots"] == 3
    assert p.predict() == pytest.approx(measured_ms, rel=0.05)
