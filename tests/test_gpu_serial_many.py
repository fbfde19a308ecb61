"""Small pieces in several slots and more than 256 host copies: copies in by
the DMA engines and out by kernels, all on the launches' stream.  The bits of
the DMA plan on three streams, in and out of place."""
import numpy as np
import pytest
import torch

from helpers import pinned_copy, to_storage
from paper_2309_08864_amd import Plan, stencil_offsets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,dims,storage,T,K,d", [
    (2, (512, 512), "f32", 68, 4, 8),
    (2, (333, 240), "bf16", 130, 2, 3),
    (3, (37, 29, 50), "f64", 132, 1, 2),
])
def test_many_small_pieces_bitwise(ndim, dims, storage, T, K, d):
    offs = stencil_offsets(ndim, "star", 1)
    rng = np.random.default_rng(43)
    w = list(rng.random(len(offs)) / len(offs))
    u = to_storage(rng.random(dims[::-1]), storage)
    kw = dict(ndim=ndim, nx=dims[0], ny=dims[1], nz=dims[2] if ndim == 3 else 1, shape="star", radius=1, weights=w,
              T=T, tb_depth=K, n_chunks=d, storage=storage, budget=1 << 30)
    outs = []
    for engine, want in (("dma", 1), ("auto", 3)):
        p = Plan(copy_engine=engine, **kw).bind()
        assert p.info()["copy_engine"] == want and p.info()["n_slots"] > 1
        h, o = pinned_copy(u), pinned_copy(u)
        for _ in range(2):
            p.run_steps(h, o, T)
            outs.append(o.clone())
        assert torch.equal(h, u)
        p.run(h)
        outs.append(h.clone())
        p.close()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
