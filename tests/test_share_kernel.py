"""The region-sharing kernel keeps what it moves in registers (a private array
of the HIP vector class lands in LDS, which takes 16 us per launch at any
size), and shared launches of every kind give the bits of single copies."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2309_08864_amd import build as B

LLVM = "/opt/rocm/llvm/bin/llvm-objdump"


def test_no_lds_and_no_scratch(tmp_path):
    obj = os.path.join(B.OBJ, "aux_kernels.hip.o")
    if not os.path.exists(obj) or not os.path.exists(LLVM):
        pytest.skip("library not built here, or no llvm-objdump")
    local = tmp_path / "aux.o"
    shutil.copy(obj, local)
    subprocess.run([LLVM, "--offloading", str(local)], cwd=tmp_path, check=True, capture_output=True)
    dev = [f for f in os.listdir(tmp_path) if f.startswith("aux.o.") and "gfx950" in f]
    assert len(dev) == 1
    asm = subprocess.run([LLVM, "-d", str(tmp_path / dev[0])], capture_output=True, text=True, check=True).stdout
    bodies = re.findall(r"<(\S*share_kernel\S*)>:\n(.*?)(?=\n\n|\Z)", asm, re.S)
    assert bodies
    for name, body in bodies:
        assert "global_load_dwordx4" in body, name
        assert not re.search(r"\b(ds_|scratch_|buffer_)", body), name


@pytest.mark.gpu
@pytest.mark.parametrize("method,d", [("so2dr", 2), ("so2dr", 5), ("resreu", 4)])
@pytest.mark.parametrize("nx,ny", [(64, 8), (61, 7)])     # whole 16-byte words, and not
def test_shared_planes_bitwise(method, d, nx, ny):
    import torch
    from helpers import gpu_run, to_storage
    u = to_storage(np.random.default_rng(d).random((60, ny, nx)), "f32")
    kw = dict(ndim=3, nx=nx, ny=ny, nz=60, shape="star", radius=1, weights=[0.1] * 7, T=10, budget=1 << 30)
    want, _, _ = gpu_run(dict(kw, tb_depth=10, n_chunks=1), u)
    got, _, _ = gpu_run(dict(kw, tb_depth=4, n_chunks=d, method=method), u)
    assert torch.equal(got, want)


@pytest.mark.gpu
def test_large_halos_bitwise():
    """Halos of 128 MiB, which are shared by single copies."""
    import torch
    from paper_2309_08864_amd import Plan, pinned_empty
    nx, ny, nz, T = 2048, 2048, 48, 4
    u = pinned_empty((nz, ny, nx), torch.float32)
    u.copy_(torch.from_numpy(np.random.default_rng(2).random((nz, ny, nx), dtype=np.float32)))
    outs = []
    for K, d in ((4, 1), (4, 3)):
        p = Plan(ndim=3, nx=nx, ny=ny, nz=nz, shape="star", radius=1, weights=[0.1] * 7, T=T, tb_depth=K, n_chunks=d,
                 budget=8 << 30).bind()
        o = pinned_empty(u.shape, u.dtype)
        p.run_steps(u, o, T)
        outs.append(o.clone())
        p.close()
    assert torch.equal(outs[0], outs[1])
