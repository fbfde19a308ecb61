"""Plans whose host copies run as copy kernels on the launches' stream (one
slot, or several with small pieces): rows of any length, host arrays at any
element offset and pieces down to a few cells give the bits of the DMA
engines and touch nothing beside the output array."""
import numpy as np
import pytest
import torch

from helpers import to_storage
from paper_2309_08864_amd import Plan, stencil_offsets

pytestmark = pytest.mark.gpu


def _at(t, shift):
    """Pinned copy of t that begins `shift` elements into its allocation, with
    guard elements on both sides."""
    big = torch.full((t.numel() + shift + 160,), 7.0, dtype=t.dtype).pin_memory()
    v = big[shift:shift + t.numel()].view(t.shape)
    v.copy_(t)
    return big, v


@pytest.mark.parametrize("ndim,dims,storage,T,K,d", [
    (2, (3, 9), "f16", 3, 3, 1),            # a field of 54 bytes: no whole 16 at the aligned side
    (2, (71, 67), "bf16", 9, 4, 1),
    (2, (1021, 130), "f32", 9, 4, 4),       # small pieces, several slots
    (3, (37, 29, 50), "f16", 7, 3, 3),
    (3, (64, 40, 33), "f32", 8, 8, 1),
    (3, (33, 21, 70), "f64", 6, 2, 4),
    (2, (2101, 700), "f64", 5, 5, 1),       # 11 MiB: many steps per lane
])
@pytest.mark.parametrize("shift_in,shift_out", [(0, 0), (1, 3), (64, 37)])
def test_serial_copies_bitwise(ndim, dims, storage, T, K, d, shift_in, shift_out):
    offs = stencil_offsets(ndim, "star", 1)
    rng = np.random.default_rng(17)
    w = list(rng.random(len(offs)) / len(offs))
    u = to_storage(rng.random(dims[::-1]), storage)
    kw = dict(ndim=ndim, nx=dims[0], ny=dims[1], nz=dims[2] if ndim == 3 else 1, shape="star", radius=1, weights=w,
              T=T, tb_depth=K, n_chunks=d, storage=storage, budget=1 << 30)
    outs = []
    for engine in ("dma", "auto"):
        p = Plan(copy_engine=engine, **kw).bind()
        assert p.info()["copy_engine"] == (1 if engine == "dma" else 2)
        _, h = _at(u, shift_in)
        big, o = _at(torch.zeros_like(u), shift_out)
        p.run_steps(h, o, T)
        assert torch.equal(h, u)
        assert torch.all(big[:shift_out] == 7) and torch.all(big[shift_out + u.numel():] == 7)
        p.run(h)                             # in place, every round re-reads its own output
        outs += [o.clone(), h.clone()]
        p.close()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


NONCOHERENT = 0x80000000   # hipHostMallocNonCoherent


@pytest.mark.parametrize("engine,want", [("auto", 2), ("dma", 1)])
def test_non_coherent_host_memory(engine, want):
    """Host memory that the device may cache is left to the DMA engines."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    u = to_storage(np.random.default_rng(23).random((40, 50)), "f32")
    ptr = ctypes.c_void_p()
    assert hip.hipHostMalloc(ctypes.byref(ptr), ctypes.c_size_t(u.numel() * 4), ctypes.c_uint(NONCOHERENT)) == 0
    h = torch.frombuffer((ctypes.c_char * (u.numel() * 4)).from_address(ptr.value), dtype=torch.float32).view(u.shape)
    p = Plan(ndim=2, nx=50, ny=40, shape="star", radius=1, weights=[0.2] * 5, T=6, tb_depth=3, copy_engine=engine,
             budget=1 << 30).bind()
    assert p.info()["copy_engine"] == want
    ref = u.clone().pin_memory()
    for _ in range(3):                      # the host rewrites the array between runs
        h.copy_(u)
        p.run(h)
        ref.copy_(u)
        p.run(ref)
        assert torch.equal(h, ref)
        u = u * 0.5 + 1
    p.close()
    assert hip.hipHostFree(ptr) == 0


@pytest.mark.parametrize("dims,d", [((101, 67), 1), ((515, 96), 3)])
def test_serial_adjoint_bitwise(dims, d):
    offs = stencil_offsets(2, "box", 1)
    rng = np.random.default_rng(19)
    w = list(rng.random(len(offs)) / len(offs))
    u, y = (to_storage(rng.random(dims[::-1]), "f32") for _ in range(2))
    res = []
    for engine in ("dma", "auto"):
        p = Plan(ndim=2, nx=dims[0], ny=dims[1], shape="box", radius=1, weights=w, T=7, tb_depth=3, n_chunks=d,
                 adjoint=True, copy_engine=engine, budget=1 << 30).bind()
        assert p.info()["copy_engine"] == (1 if engine == "dma" else 2)
        loss, gu, gw, _ = p.adjoint(_at(u, 5)[1], _at(y, 2)[1], 3)
        res.append((loss, gu.clone(), gw.copy()))
        p.close()
    assert res[0][0] == res[1][0] and torch.equal(res[0][1], res[1][1]) and np.array_equal(res[0][2], res[1][2])
