"""Performance cases of the stencil library: what its users run, through the
public entry points (`Plan(...).run` and `run_batch`).

A case is one call: `steps` time steps of a box or star stencil on a dense
grid (or one batched call over several grids), with the plan, the input grid
and the output buffer already in hand.  The listed cases are the workloads of
the benchmark and of the served stream at their own sizes, with odd and small
grids beside them; `draw` gives further cases of the same ranges: d = 2 with
sides 256..8192, d = 3 with sides 64..512, radius 1..3, fusion depth 1..4
(1..3 for d = 3), both boundaries, every storage type, and batches of mixed
grids.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2603_00477_amd as stl

_BYTES = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "bf16x3": 4}
_MAX_FLOPS = 1.3e11   # flops of the largest listed case
_MAX_BYTES = 1.0e9    # bytes in and out of a drawn case


def _grid(name, shape, d, r, dims, T, dtype, boundary, steps, halo=0.0, data="uniform"):
    dims = tuple(dims) + (1,) * (3 - d)
    c = dict(kind="grid", shape=shape, d=d, r=r, n0=dims[0], n1=dims[1], n2=dims[2], T=T, dtype=dtype,
             boundary=boundary, steps=steps, halo=halo, data=data)
    return dict(c, name=name) if name else c


def listed():
    return [
        # Jacobi relaxation on a small grid: the smallest call, where each of
        # the ten one-step launches is shorter than the way to start it
        _grid("jacobi2d_512_f64", "star", 2, 1, (512, 512), 1, "f64", "dirichlet", 10),
        # the benchmark's headline: a large compute-bound box in float64
        _grid("box2d3r_8192_f64_t2", "box", 2, 3, (8192, 8192), 2, "f64", "dirichlet", 20),
        # a large star fused four deep in float32 (seismic-like reach)
        _grid("star2d3r_8192_f32_t4", "star", 2, 3, (8192, 8192), 4, "f32", "dirichlet", 20),
        # odd sides: rows that are no whole number of vectors, a remainder
        # pass, and a halo value
        _grid("box2d2r_odd_f32_t2", "box", 2, 2, (3001, 4093), 2, "f32", "dirichlet", 9, halo=0.25),
        # 16-bit storage on the matrix cores, the benchmark's precision
        # workload: large, periodic, four steps per pass
        _grid("box2d2r_16384_bf16_t4", "box", 2, 2, (16384, 16384), 4, "bf16", "periodic", 12, data="smooth"),
        # 16-bit storage, middling grid, fixed boundary (its band is redone
        # step by step), a remainder pass
        _grid("star2d2r_1500_f16_t4", "star", 2, 2, (1500, 2200), 4, "f16", "dirichlet", 18),
        # the compensated mode: float32 storage on bf16 matrix products
        _grid("box2d2r_4096_x3_t2", "box", 2, 2, (4096, 4096), 2, "bf16x3", "periodic", 10, data="smooth"),
        # three-dimensional workload, float64 star fused three deep
        _grid("star3d2r_512_f64_t3", "star", 3, 2, (512, 512, 512), 3, "f64", "periodic", 9),
        # three-dimensional workload, float32 27-point box
        _grid("box3d1r_512_f32_t2", "box", 3, 1, (512, 512, 512), 2, "f32", "periodic", 8),
        # small volume of the served stream, odd sides
        _grid("star3d1r_97_f32_t2", "star", 3, 1, (97, 97, 97), 2, "f32", "dirichlet", 16),
        # compute-bound 125-point box of the served stream
        _grid("box3d2r_200_f32_t1", "box", 3, 2, (200, 200, 200), 1, "f32", "dirichlet", 8),
        # one call over sixteen mixed grids, as the server's rounds make them
        dict(name="batch16_f32", kind="batch", jobs=16, mix=5000, side2=2048, side3=192, steps=8),
    ]


def _points(d, r, shape):
    return (2 * r + 1) ** d if shape == "box" else 2 * d * r + 1


def _log_side(rng, lo, hi):
    """A side spread over the logarithm of its range: as drawn (odd ones as
    often as even ones), or rounded to a multiple of 32."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return n if rng.random() < 0.6 else max(lo, n // 32 * 32)


def draw(rng):
    if rng.random() < 0.12:
        return dict(kind="batch", jobs=rng.randint(4, 24), mix=rng.randint(1, 10 ** 6),
                    side2=rng.choice([512, 1024, 2048]), side3=rng.choice([96, 128, 192]), steps=rng.randint(2, 10))
    shape = rng.choice(["star", "box"])
    r = rng.randint(1, 3)
    boundary = rng.choice(["dirichlet", "periodic"])
    halo = rng.choice([0.0, 0.25]) if boundary == "dirichlet" else 0.0
    if rng.random() < 0.6:
        d, T = 2, rng.randint(1, 4)
        dtype = rng.choice(["f64", "f32", "f64", "f32", "bf16", "f16", "bf16x3"])
        dims = (_log_side(rng, 256, 8192), _log_side(rng, 256, 8192))
    else:
        d, T = 3, rng.randint(1, 3)
        dtype = rng.choice(["f64", "f32"])
        dims = tuple(_log_side(rng, 64, 512) for _ in range(3))
        if shape == "box" and r > 1:
            T = 1  # the large boxes are swept one step per pass
    points = math.prod(dims)
    most = _MAX_FLOPS / (2.0 * _points(d, r, shape) * points)
    steps = max(1, min(rng.randint(1, 24), int(most)))
    while 2.0 * points * _BYTES[dtype] > _MAX_BYTES or 2.0 * _points(d, r, shape) * points > _MAX_FLOPS:
        dims = (max(64, dims[0] // 2),) + dims[1:]
        points = math.prod(dims)
    return _grid(None, shape, d, r, dims, T, dtype, boundary, steps, halo=halo)


def _batch_jobs(case):
    """The grids of a batched call: shapes, radii and sides of the served
    stream (sides spread over their logarithm), fused as the server's tuner
    fuses them: stars deep, boxes two steps, large 3D boxes not at all."""
    rng = random.Random(case["mix"])
    jobs = []
    for i in range(case["jobs"]):
        shape, d, r = rng.choice(["star", "box"]), 2 + i % 2, rng.randint(1, 3)
        lo, hi = (256, case["side2"]) if d == 2 else (64, case["side3"])
        side = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        if d == 2:
            T = 4 if shape == "star" else 2
        else:
            T = 2 if shape == "star" or r == 1 else 1
        jobs.append(_grid(None, shape, d, r, (side,) * d, T, "f32", rng.choice(["dirichlet", "periodic"]),
                          rng.randint(1, case["steps"])))
    return jobs


def _members(case):
    return _batch_jobs(case) if case["kind"] == "batch" else [case]


def _dims(c):
    return (c["n0"], c["n1"], c["n2"])[:c["d"]]


def _weights(c, seed):
    w = np.random.Generator(np.random.PCG64(seed)).random(_points(c["d"], c["r"], c["shape"]))
    return w / w.sum()


def _input(c, seed):
    """The input grid in its storage type: uniform on [0, 1), or the smooth
    field sin(2 pi x) sin(2 pi y) with 1e-3 of uniform noise."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dims = _dims(c)
    tdt = stl.torch_dtype(c["dtype"])
    if c["data"] == "smooth":
        y, x = (torch.sin(torch.arange(n, device="cuda", dtype=torch.float64) * (2 * math.pi / n)) for n in dims)
        u = torch.outer(y, x)
        u += 1e-3 * torch.rand(dims, generator=g, device="cuda", dtype=torch.float64)
    else:
        u = torch.rand(dims, generator=g, device="cuda",
                       dtype=torch.float64 if c["dtype"] == "f64" else torch.float32)
    return u.to(tdt).contiguous()


def _seeds(seed, i):
    return 1000003 * seed + 2 * i, 1000003 * seed + 2 * i + 1


def prepare(case, seed):
    plans, ins, outs, steps = [], [], [], []
    for i, c in enumerate(_members(case)):
        ds, ws = _seeds(seed, i)
        # the path is left to the plan: the model's predicted winner
        plans.append(stl.Plan(c["shape"], c["d"], c["r"], _weights(c, ws), _dims(c), T=c["T"], dtype=c["dtype"],
                              boundary=c["boundary"], halo=c["halo"]))
        ins.append(_input(c, ds))
        outs.append(torch.empty_like(ins[-1]))
        steps.append(c["steps"])
    return dict(batch=case["kind"] == "batch", plans=plans, ins=ins, outs=outs, steps=steps)


def run(state):
    if state["batch"]:
        stl.run_batch(state["plans"], state["ins"], state["outs"], state["steps"])
        return state["outs"]
    return state["plans"][0].run(state["ins"][0], state["outs"][0], state["steps"][0])


def work(case):
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _members(case):
        points = math.prod(_dims(c))
        total["bytes"] += 2.0 * points * _BYTES[c["dtype"]]
        total["flops"] += 2.0 * _points(c["d"], c["r"], c["shape"]) * points * c["steps"]
    return total


def _offsets(c):
    """Offsets in the canonical weight order: boxes row-major with the last
    axis fastest; stars the centre, then each axis from -r to r."""
    d, r = c["d"], c["r"]
    if c["shape"] == "box":
        return [tuple(o) for o in np.ndindex(*(2 * r + 1,) * d)]
    offs = [(r,) * d]
    for ax in range(d):
        for k in list(range(-r, 0)) + list(range(1, r + 1)):
            offs.append(tuple(r + (k if i == ax else 0) for i in range(d)))
    return offs


def _exact_one(c, ds, ws):
    w = _weights(c, ws)
    u = _input(c, ds).to(torch.float64)
    r, dims = c["r"], _dims(c)
    offs = _offsets(c)
    inner = tuple(slice(r, r + n) for n in dims)
    pad = torch.full([n + 2 * r for n in dims], float(c["halo"]), device="cuda", dtype=torch.float64)
    for _ in range(c["steps"]):
        pad[inner] = u
        if c["boundary"] == "periodic":
            for ax, n in enumerate(dims):
                pad.narrow(ax, 0, r).copy_(pad.narrow(ax, n, r))
                pad.narrow(ax, r + n, r).copy_(pad.narrow(ax, r, r))
        u.zero_()
        for o, wk in zip(offs, w):
            u.add_(pad[tuple(slice(a, a + n) for a, n in zip(o, dims))], alpha=float(wk))
    return u


def exact(case, seed):
    got = [_exact_one(c, *_seeds(seed, i)) for i, c in enumerate(_members(case))]
    return got if case["kind"] == "batch" else got[0]
