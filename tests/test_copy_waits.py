"""Who waits before a DMA copy-out of the reverse sweep: the rule (copy_rule.hpp,
compiled for the host) at the sizes it was measured at, and on the GPU gradients
on either side of it, and forward runs of large copies against the in-core bits."""
import subprocess

import numpy as np
import pytest

from paper_2309_08864_amd import build as B

MIB = 1 << 20

REVERSE = [   # MiB per copy, chunks, does the host wait
    (146, 28, 0), (512, 4, 0), (256, 16, 0), (128, 16, 0), (64, 16, 0), (64, 8, 0),
    (64, 32, 1), (32, 16, 1), (32, 32, 1), (16, 32, 1), (6, 20, 1),
]


def test_rule_at_the_measured_points(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    body = "".join(f'  std::printf("%d\\n", (int)so2dr::host_waits_reverse((size_t){m} << 20, {d}));\n'
                   for m, d, _ in REVERSE)
    src.write_text('#include <cstdio>\n#include "copy_rule.hpp"\nint main() {\n' + body + "}\n")
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    assert got == [w for *_, w in REVERSE]


@pytest.mark.gpu
@pytest.mark.parametrize("d,slots,K", [(4, 2, 4), (4, 2, 1), (4, 3, 4)])   # 16 and 64 copies of 64 MiB; three slots
def test_large_copies_bitwise(d, slots, K):
    import torch
    from paper_2309_08864_amd import Plan, pinned_empty
    nx, ny, nz, T = 512, 512, 256, 8
    kw = dict(ndim=3, nx=nx, ny=ny, nz=nz, shape="star", radius=1, weights=[0.1, 0.1, 0.1, 0.4, 0.1, 0.1, 0.1], T=T,
              budget=4 << 30)
    u = pinned_empty((nz, ny, nx), torch.float32)
    u.copy_(torch.from_numpy(np.random.default_rng(8).random((nz, ny, nx), dtype=np.float32)))
    outs = []
    for more in (dict(tb_depth=T, n_chunks=1), dict(tb_depth=K, n_chunks=d, n_slots=slots, copy_engine="dma")):
        p = Plan(**kw, **more).bind()
        o = pinned_empty(u.shape, u.dtype)
        p.run_steps(u, o, T)
        outs.append(o.clone())
        o.copy_(u)
        p.run(o)
        outs.append(o.clone())
        p.close()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


@pytest.mark.gpu
def test_large_copies_gradient_bitwise():
    """64 MiB copies in four chunks (the device waits) and 8 MiB ones in 32 (the
    host waits) of the same field: the gradient arrays agree bit for bit, the
    FP64 sums to their rounding."""
    import torch
    from paper_2309_08864_amd import Plan, adjoint_buffers_needed, pinned_empty
    nx, ny, nz, T = 512, 512, 256, 4
    rng = np.random.default_rng(9)
    u, y = (pinned_empty((nz, ny, nx), torch.float32) for _ in range(2))
    u.copy_(torch.from_numpy(rng.random((nz, ny, nx), dtype=np.float32)))
    y.copy_(torch.from_numpy(rng.random((nz, ny, nx), dtype=np.float32)))
    res = []
    for d, slots in ((4, 2), (4, 3), (32, 3)):
        p = Plan(ndim=3, nx=nx, ny=ny, nz=nz, shape="star", radius=1, weights=[0.1, 0.1, 0.1, 0.4, 0.1, 0.1, 0.1], T=T,
                 tb_depth=2, n_chunks=d, n_slots=slots, adjoint=True, copy_engine="dma", budget=4 << 30).bind()
        bufs = [pinned_empty(u.shape, u.dtype) for _ in range(adjoint_buffers_needed(T, 2, 4))]
        loss, gu, gw, _ = p.adjoint(u, y, 4, ckpt=bufs)
        res.append((loss, gu.clone(), gw.copy()))
        p.close()
    for loss, gu, gw in res[1:]:
        assert torch.equal(gu, res[0][1])
        assert loss == pytest.approx(res[0][0], rel=1e-12) and np.allclose(gw, res[0][2], rtol=1e-10, atol=0)
