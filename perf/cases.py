"""Representative work of a user of this library, as cases that can be timed.

A case is one call of a public entry point on data in pinned host memory, as
the library is meant to be used: ``Plan.run_steps`` (a sweep, out of place so
that it can be repeated on the same input), ``Plan.adjoint`` (loss and
gradients with caller-kept checkpoint buffers) or ``StencilLoss`` (the same
through torch.autograd, which plans and binds on every call).  Grids, stencils
and schedules are those of workloads/configs.py, the smoke check and the
tests, scaled so that a pass takes well under a second; row lengths include
odd ones."""
import math

import torch

from paper_2309_08864_amd import (Plan, StencilLoss, adjoint_buffers_needed, pinned_empty,
                                  stencil_offsets, suggest)

MIB = 1 << 20
TORCH = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16,
         "f16": torch.float16}
SIZE = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2}


def _case(name, mode, ndim, nx, ny, nz, shape, radius, storage, T, K, chunks, budget_mib, **more):
    c = dict(name=name, mode=mode, ndim=ndim, nx=nx, ny=ny, nz=nz, shape=shape, radius=radius,
             storage=storage, T=T, K=K, chunks=chunks, budget_mib=budget_mib, periodic=False,
             rounding="every_step", ckpt=0, auto=False)
    c.update(more)
    return c


def listed():
    return [
        # the smoke check's grid: a small 3D sweep held in core, where the
        # call's own latency counts
        _case("small_3d7pt", "run", 3, 96, 40, 48, "star", 1, "f32", 8, 8, 1, 64),
        # the 2D 5-point Jacobi workload under its 4 MiB budget, FP64 (one
        # buffer per slot, many short launches)
        _case("2d5pt_4mib_f64", "run", 2, 1024, 1024, 1, "star", 1, "f64", 16, 4, 4, 4),
        # a mid-size simulation held in core for a long run
        _case("incore_3d7pt_256", "run", 3, 256, 256, 256, "star", 1, "f32", 256, 256, 1, 256),
        # 27-point box, periodic in x and y, odd extents, in core
        _case("incore_3d27pt_odd", "run", 3, 301, 257, 203, "box", 1, "f32", 64, 64, 1, 256,
              periodic=True),
        # the headline 7-point workload's schedule (16 chunks, K = 8, T = 64,
        # half the field as budget) on an eighth of its grid
        _case("ooc_3d7pt", "run", 3, 1024, 512, 512, "star", 1, "f32", 64, 8, 16, 512),
        # the same sweep with chunks, depth and slots left to the cost model
        _case("auto_3d7pt", "run", 3, 1024, 512, 512, "star", 1, "f32", 64, 0, 0, 512, auto=True),
        # 13-point star in BF16 storage, the precision workload's form with a
        # deeper round
        _case("ooc_3d13pt_bf16", "run", 3, 512, 512, 512, "star", 2, "bf16", 64, 16, 4, 512),
        # 13-point star in FP64, odd rows, in core
        _case("incore_3d13pt_f64_odd", "run", 3, 251, 190, 163, "star", 2, "f64", 48, 48, 1, 512),
        # the paper's in-core 2D box dataset at radius 1: 12800^2, 640 steps
        _case("incore_box2d1r", "run", 2, 12800, 12800, 1, "box", 1, "f32", 640, 640, 1, 2048),
        # the paper's 2D box at radius 4, chunked with its S_TB = 40
        _case("ooc_box2d4r", "run", 2, 12800, 12800, 1, "box", 4, "f32", 80, 40, 4, 2048),
        # gradient of the 7-point sweep, checkpoints every 16 steps, under a
        # budget of about half a field as in the adjoint workload
        _case("adjoint_3d7pt", "adjoint", 3, 320, 320, 320, "star", 1, "f32", 64, 8, 0, 128,
              ckpt=16),
        # learning 2D box weights through autograd, odd rows
        _case("loss_2d9pt_odd", "loss", 2, 1021, 767, 1, "box", 1, "f32", 16, 8, 1, 64, ckpt=8),
    ]


_STENCILS = [(2, "star", 1), (2, "box", 1), (2, "box", 2), (2, "box", 3), (2, "box", 4),
             (3, "star", 1), (3, "star", 2), (3, "box", 1)]


def draw(rng):
    ndim, shape, r = rng.choice(_STENCILS)
    mode = rng.choice(["run", "run", "run", "run", "adjoint", "loss"])
    storage = (rng.choice(["f32", "f32", "f32", "f64", "bf16", "f16"]) if mode == "run"
               else rng.choice(["f32", "f32", "f64"]))
    cells = 2.0 ** rng.uniform(17, 26.5 if mode == "run" else 24.0)
    if ndim == 3:
        nx = int(cells ** (1 / 3) * 2.0 ** rng.uniform(-0.5, 1.0))
        ny = int(math.sqrt(cells / nx) * 2.0 ** rng.uniform(-0.4, 0.4))
        nz = int(cells / (nx * ny))
    else:
        nx = int(math.sqrt(cells) * 2.0 ** rng.uniform(-0.7, 0.7))
        ny, nz = int(cells / nx), 1
    kind = rng.choice(["round", "even", "odd"])   # row length: whole 64s, even or odd
    nx = max(40, nx)
    nx = (nx + 32) // 64 * 64 if kind == "round" and nx >= 64 else nx // 2 * 2 + (kind == "odd")
    ny, nz = max(24, ny), (max(24, nz) if ndim == 3 else 1)
    n_axis = nz if ndim == 3 else ny
    T = int(2.0 ** rng.uniform(3, 7.5 if mode == "run" else 5.0))
    K = min(T, rng.choice([4, 8, 16, 40, 160]))
    if mode != "run":
        K = min(K, 16)
    chunks = rng.choice([1, 1, 2, 4, 8])
    while chunks > 1 and n_axis // chunks < 2 * r * K:
        chunks -= 1
    if chunks == 1 and mode == "run":
        K = T
    ckpt = 0 if mode == "run" else rng.choice([K, 2 * K, T])
    # room for three slots of two buffers (the adjoint: three working buffers
    # more and two sharing buffers)
    plane = nx * (ny if ndim == 3 else 1) * SIZE[storage]
    halo = 2 * r * K if chunks > 1 else 0
    bufs = 2 * min(3, chunks) + (0 if mode == "run" else 3)
    need = plane * ((-(-n_axis // chunks) + halo) * bufs + 2 * halo) + 2 * MIB
    c = _case("", mode, ndim, nx, ny, nz, shape, r, storage, T, K, chunks, -(-need // MIB),
              ckpt=ckpt, periodic=rng.random() < 0.3)
    if storage in ("bf16", "f16") and rng.random() < 0.25:
        c["rounding"] = "at_store"
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _shape(c):
    return (c["nz"], c["ny"], c["nx"]) if c["ndim"] == 3 else (c["ny"], c["nx"])


def _bc(c):
    if not c["periodic"]:
        return (0, 0, 0)
    return (1, 1, 0) if c["ndim"] == 3 else (1, 0, 0)


def _weights(c, gen):
    """Centre/arm weights for stars, random positive ones of sum 1 for boxes."""
    offs = stencil_offsets(c["ndim"], c["shape"], c["radius"])
    if c["shape"] == "box":
        w = 0.5 + torch.rand(len(offs), generator=gen, dtype=torch.float64)
        w = w / w.sum()
        return [float(x) for x in (w if c["storage"] == "f64" else w.float().double())]
    if c["ndim"] == 2:
        table = [0.2, 0.2]
    else:
        table = [0.4, 0.1] if c["radius"] == 1 else [0.28, 0.1, 0.02]
    w = [table[max(abs(a) for a in o)] for o in offs]
    return w if c["storage"] == "f64" else [float(torch.tensor(x)) for x in w]


def _field(c, seed, salt):
    """The field on the GPU, in FP64 rounded to the storage type: uniform
    [0, 1) for the radius-1 star and the 2D boxes, a Gaussian bump with noise
    for the 13-point star, Fourier modes with noise for the 27-point box."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 16 + salt)
    shape = _shape(c)
    u = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32)
    if c["ndim"] == 3 and c["radius"] == 2:
        u = (u - 0.5) * 2e-3
        g = 1.0
        for axis, n in enumerate(shape):
            x = torch.arange(n, device="cuda", dtype=torch.float32)
            e = torch.exp(-0.5 * ((x - (n - 1) / 2) / (n / 8)) ** 2)
            g = g * e.reshape([-1 if a == axis else 1 for a in range(3)])
        u += g
    elif c["ndim"] == 3 and c["shape"] == "box":
        u = (u - 0.5) * 0.03
        nz, ny, nx = shape
        x = torch.arange(nx, device="cuda", dtype=torch.float32)
        y = torch.arange(ny, device="cuda", dtype=torch.float32)[:, None]
        z = torch.arange(nz, device="cuda", dtype=torch.float32)[:, None, None]
        for kx, ky, m, a in ((1, 2, 1, 0.3), (5, 3, 2, 0.2), (9, 12, 4, 0.15)):
            u += a * torch.cos(2 * math.pi * (kx * x / nx + ky * y / ny)) * torch.sin(
                math.pi * m * (z + 1) / (nz + 1))
    return u.to(TORCH[c["storage"]])


def _inputs(c, seed):
    gen = torch.Generator().manual_seed(seed)
    return _weights(c, gen), _field(c, seed, 1), (_field(c, seed, 2) if c["mode"] != "run" else None)


def _pinned(c, values=None):
    t = pinned_empty(_shape(c), TORCH[c["storage"]])
    if values is not None:
        t.copy_(values)
    return t


def _spec(c):
    return dict(ndim=c["ndim"], nx=c["nx"], ny=c["ny"], nz=c["nz"], shape=c["shape"],
                radius=c["radius"], T=c["T"], tb_depth=c["K"], n_chunks=c["chunks"],
                budget=c["budget_mib"] * MIB, storage=c["storage"], bc=_bc(c),
                rounding=c["rounding"])


def prepare(case, seed):
    c = case
    w, u0, target = _inputs(c, seed)
    s = {"mode": c["mode"], "T": c["T"], "ckpt": c["ckpt"], "u0": _pinned(c, u0)}
    if c["mode"] == "loss":
        s["target"] = _pinned(c, target)
        s["spec"] = dict(_spec(c), ckpt_every=c["ckpt"])
        s["w"] = torch.tensor(w, dtype=torch.float64, requires_grad=True)
        s["u0"].requires_grad_(True)
        return s
    spec = dict(_spec(c), weights=w)
    if c["auto"]:
        spec, _ = suggest(**spec)
    if c["mode"] == "adjoint":
        s["target"] = _pinned(c, target)
        s["plan"] = Plan(adjoint=True, **spec).bind()
        n = adjoint_buffers_needed(c["T"], s["plan"].info()["tb_depth"], c["ckpt"])
        s["buffers"] = [_pinned(c) for _ in range(n)]
        s["grad"] = _pinned(c)
    else:
        s["plan"] = Plan(**spec).bind()
        s["out"] = _pinned(c)
    return s


def run(state):
    s = state
    if s["mode"] == "run":
        s["plan"].run_steps(s["u0"], s["out"], s["T"])
        return s["out"]
    if s["mode"] == "adjoint":
        loss, grad, grad_w, _ = s["plan"].adjoint(s["u0"], s["target"], s["ckpt"],
                                                  ckpt=s["buffers"], grad_u0=s["grad"])
        return {"loss": loss, "grad_u0": grad, "grad_w": grad_w}
    loss = StencilLoss.apply(s["u0"], s["w"], s["target"], s["spec"])
    grad, grad_w = torch.autograd.grad(loss, (s["u0"], s["w"]))
    return {"loss": loss.detach(), "grad_u0": grad, "grad_w": grad_w}


def _cells(c):
    return c["nx"] * c["ny"] * c["nz"]


def work(case):
    c = case
    points = len(stencil_offsets(c["ndim"], c["shape"], c["radius"]))
    sweep = _cells(c) * c["T"] * (2 * points - 1)
    field = _cells(c) * SIZE[c["storage"]]
    if c["mode"] == "run":
        return {"bytes": 2 * field, "flops": sweep}
    # forward, transpose steps and weight gradients; u0 and target in, the
    # gradient out
    return {"bytes": 3 * field, "flops": 2 * sweep + 2 * points * _cells(c) * c["T"]}


# ------------------------------------------------------------------- exact
def _shift(v, off, bc):
    """View pairs (destination slices, source tensor) of v displaced by off:
    out[x] += w v[x + off], zero outside, wrapped on periodic axes."""
    dst, src = [], v
    for axis, (d, per) in enumerate(zip(off, bc)):
        n = v.shape[axis]
        if d == 0:
            dst.append(slice(None))
        elif per:
            src = torch.roll(src, -d, axis)
            dst.append(slice(None))
        else:
            src = src.narrow(axis, max(0, d), n - abs(d))
            dst.append(slice(max(0, -d), n - max(0, d)))
    return tuple(dst), src


def _apply(v, offs, w, bc):
    out = torch.zeros_like(v)
    for o, x in zip(offs, w):
        dst, src = _shift(v, o, bc)
        out[dst].add_(src, alpha=x)
    return out


def exact(case, seed):
    c = case
    offs = stencil_offsets(c["ndim"], c["shape"], c["radius"])
    steps = c["T"] if c["mode"] == "run" else 4 * c["T"]
    passes = _cells(c) * len(offs) * steps * (2.0 if c["periodic"] else 1.0)
    if passes > 2.5e12 or (c["mode"] != "run" and _cells(c) * (c["T"] + 4) * 8 > 60e9):
        return None
    w, u0, target = _inputs(c, seed)
    bc = _bc(c)
    bc = (bc[2], bc[1], bc[0]) if c["ndim"] == 3 else (bc[1], bc[0])
    offs = offs if c["ndim"] == 3 else [o[1:] for o in offs]
    u = u0.double()
    del u0
    if c["mode"] == "run":
        for _ in range(c["T"]):
            u = _apply(u, offs, w, bc)
        return u
    states = [u]
    for _ in range(c["T"]):
        states.append(_apply(states[-1], offs, w, bc))
    lam = states.pop() - target.double()
    loss = 0.5 * float((lam * lam).sum())
    grad_w = torch.zeros(len(offs), dtype=torch.float64, device="cuda")
    back = [tuple(-d for d in o) for o in offs]
    while states:
        v = states.pop()
        for k, o in enumerate(offs):
            dst, src = _shift(v, o, bc)
            grad_w[k] += (lam[dst] * src).sum()
        lam = _apply(lam, back, w, bc)
    loss = torch.tensor(loss, dtype=torch.float64) if c["mode"] == "loss" else loss
    return {"loss": loss, "grad_u0": lam, "grad_w": grad_w.cpu()}
