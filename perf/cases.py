"""The transforms whose speed is followed, through the package's public entry points.

A case is one call (or a forward and backward pair) as a program makes it:
plans are made once, inputs lie in device memory, output buffers are kept by
the caller's loop.  Kinds:

  grid   offt.Plan of three axes, natural output order, with a batch
  cba    offt.Plan with the reversed (cba) output order
  nd     offt.Plan of four axes
  many   offt.ManyPlan, an uneven batch in one packed buffer

"plan" is "default" (the plan a program gets without asking for tuning) or
"cached" (the tuned plan of the committed plan cache, as bench.py runs it).
Directions: "fwd", "bwd" (with 1/N) and "pair" (forward, then backward with
1/N, whose outputs are both returned).
"""
from __future__ import annotations

import math
import os

import torch

import paper_1501_07350_amd as offt

DTYPES = {"c128": torch.complex128, "c64": torch.complex64}
ELEM = {"c128": 16, "c64": 8}
PLAN_CACHE = os.path.join(os.path.dirname(os.path.abspath(offt.__file__)), "data", "plan_cache_mi355x.txt")
# axis lengths of the uneven batches (the bench's workload of 64 grids)
BATCH_AXES = (48, 60, 64, 80, 96, 120, 128, 150, 160)


def _case(kind, shape, dtype, direction, batch=1, plan="default", name=None):
    c = {"kind": kind, "shape": "x".join(str(n) for n in shape), "dtype": dtype, "direction": direction,
         "batch": batch, "plan": plan}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call in use: a 32^3 convolution step (forward, then
        # inverse with 1/N); launches and latency count
        _case("grid", (32, 32, 32), "c128", "pair", name="cube32_c128_pair"),
        # one small single-precision grid, forward
        _case("grid", (64, 64, 64), "c64", "fwd", name="cube64_c64_fwd"),
        # a batch of equal small grids with ragged sides, inverse
        _case("grid", (48, 60, 50), "c64", "bwd", batch=8, name="batch8_48x60x50_c64_bwd"),
        # the paper's smallest grid, a simulation step in double precision
        _case("grid", (128, 128, 128), "c128", "pair", name="cube128_c128_pair"),
        # the paper's 256^3 grid
        _case("grid", (256, 256, 256), "c128", "fwd", name="cube256_c128_fwd"),
        # the headline: 512^3 with the tuned plan, both precisions
        _case("grid", (512, 512, 512), "c128", "fwd", plan="cached", name="cube512_c128_fwd_cached"),
        _case("grid", (512, 512, 512), "c64", "fwd", plan="cached", name="cube512_c64_fwd_cached"),
        # the paper's largest grid, single precision (8 GiB), tuned plan
        _case("grid", (1024, 1024, 1024), "c64", "fwd", plan="cached", name="cube1024_c64_fwd_cached"),
        # a large box with sides that are no powers of two, inverse, default plan
        _case("grid", (450, 480, 500), "c128", "bwd", name="box450x480x500_c128_bwd"),
        # reversed output order, the distribution the paper's transform ends in
        _case("cba", (256, 320, 384), "c64", "fwd", name="cba256x320x384_c64_fwd"),
        # a four-dimensional grid (2 GiB), default plan
        _case("nd", (128, 128, 128, 128), "c64", "fwd", name="nd128x4_c64_fwd"),
        # 64 grids of unequal shapes in one call
        _case("many", (64,), "c64", "fwd", name="many64_c64_fwd"),
    ]


def _smooth(lo, hi):
    out = []
    for n in range(lo, hi + 1):
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            out.append(n)
    return out


def _near(lengths, x):
    return min(lengths, key=lambda n: (abs(math.log(n / x)), n))


def draw(rng):
    """Grids of 2^12 to 2^27.5 points: cubes and boxes in equal parts, sides
    any 2/3/5-smooth length, batches of 1 to 8, both precisions."""
    kind = rng.choice(("grid", "grid", "grid", "grid", "grid", "cba", "nd", "many"))
    dtype = rng.choice(("c128", "c64"))
    if kind == "many":
        return _case("many", (rng.randint(12, 64),), "c64", rng.choice(("fwd", "bwd")))
    direction = rng.choice(("fwd", "bwd", "pair"))
    lengths = _smooth(8, 640)
    points = 2.0 ** rng.uniform(12, 27.5)
    batch = rng.choice((1, 1, 1, 2, 4, 8)) if kind == "grid" else 1
    ndim = 4 if kind == "nd" else 3
    side = max(8.0, (points / batch) ** (1.0 / ndim))
    if rng.random() < 0.5:
        shape = (_near(lengths, side),) * ndim
    else:
        shape = tuple(_near(lengths, side * 2.0 ** rng.uniform(-0.8, 0.8)) for _ in range(ndim))
    return _case(kind, shape, dtype, direction, batch=batch)


def _dims(case):
    return tuple(int(v) for v in case["shape"].split("x"))


def _many_dims(case):
    """The shapes of an uneven batch: sides cycled through BATCH_AXES with
    co-prime steps, so that every length occurs on every axis."""
    n = len(BATCH_AXES)
    return [(BATCH_AXES[(5 * g + 2) % n], BATCH_AXES[(7 * g + g // n) % n], BATCH_AXES[(4 * g + 1) % n])
            for g in range(_dims(case)[0])]


def _rand(n, dtype, seed):
    """n values with real and imaginary parts uniform in [-1, 1)."""
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1501 + int(seed))
    x = torch.empty((n, 2), dtype=real, device="cuda").uniform_(-1.0, 1.0, generator=gen)
    return torch.view_as_complex(x)


def _many_offsets(dims, elem):
    """Element offset of every grid in the packed buffer (grids start on
    256-byte boundaries), and the buffer's length."""
    offs, at = [], 0
    align = 256 // elem
    for d in dims:
        offs.append(at)
        at += -(-(d[0] * d[1] * d[2]) // align) * align
    return offs, at


def _inputs(case, seed):
    dtype = DTYPES[case["dtype"]]
    if case["kind"] == "many":
        dims = _many_dims(case)
        offs, total = _many_offsets(dims, ELEM[case["dtype"]])
        x = torch.zeros(total, dtype=dtype, device="cuda")
        vals = _rand(total, dtype, seed)
        for o, d in zip(offs, dims):
            n = d[0] * d[1] * d[2]
            x[o:o + n] = vals[o:o + n]
        return x
    shape = _dims(case)
    if case["kind"] == "cba" and case["direction"] == "bwd":
        shape = shape[::-1]
    n = case["batch"] * math.prod(shape)
    full = ((case["batch"],) if case["batch"] > 1 else ()) + shape
    return _rand(n, dtype, seed).view(full)


def prepare(case, seed):
    dtype = DTYPES[case["dtype"]]
    x = _inputs(case, seed)
    if case["kind"] == "many":
        plan = offt.ManyPlan(_many_dims(case), dtype=dtype, normalize_inverse=True)
        return {"case": case, "plan": plan, "x": x, "out": torch.zeros_like(x)}
    opts = {}
    if case["plan"] == "cached":
        opts = {"tune": "exhaustive", "cache_path": PLAN_CACHE}
    plan = offt.Plan(_dims(case), dtype=dtype, batch=case["batch"], normalize_inverse=True,
                     layout="cba" if case["kind"] == "cba" else "natural", **opts)
    lead = (case["batch"],) if case["batch"] > 1 else ()
    y = torch.empty(lead + tuple(plan.spectral_shape), dtype=dtype, device="cuda")
    z = torch.empty(lead + tuple(plan.shape), dtype=dtype, device="cuda")
    return {"case": case, "plan": plan, "x": x, "y": y, "z": z}


def run(state):
    plan, x, direction = state["plan"], state["x"], state["case"]["direction"]
    if state["case"]["kind"] == "many":
        return plan.forward(x, state["out"]) if direction == "fwd" else plan.backward(x, state["out"])
    if direction == "fwd":
        return plan.forward(x, state["y"])
    if direction == "bwd":
        return plan.backward(x, state["z"])
    return plan.forward(x, state["y"]), plan.backward(state["y"], state["z"])


def _points(case):
    if case["kind"] == "many":
        return [math.prod(d) for d in _many_dims(case)]
    return [math.prod(_dims(case))] * case["batch"]


def work(case):
    """Each transform reads its grid once and writes it once; 5 N log2 N
    operations."""
    calls = 2 if case["direction"] == "pair" else 1
    pts = _points(case)
    return {"bytes": calls * 2 * ELEM[case["dtype"]] * sum(pts),
            "flops": calls * sum(5.0 * n * math.log2(n) for n in pts)}


def exact(case, seed):
    x = _inputs(case, seed).to(torch.complex128)

    def whole(v, nd, inverse):
        axes = tuple(range(v.dim() - nd, v.dim()))
        return torch.fft.ifftn(v, dim=axes) if inverse else torch.fft.fftn(v, dim=axes)

    if case["kind"] == "many":
        dims = _many_dims(case)
        offs, total = _many_offsets(dims, ELEM[case["dtype"]])
        out = torch.zeros(total, dtype=torch.complex128, device="cuda")
        for o, d in zip(offs, dims):
            n = math.prod(d)
            out[o:o + n] = whole(x[o:o + n].view(d), 3, case["direction"] == "bwd").reshape(-1)
        return out
    nd = len(_dims(case))

    def flip(v):
        """The last three axes in reversed order."""
        return v.transpose(-1, -3).contiguous()

    if case["direction"] == "bwd":
        return whole(flip(x) if case["kind"] == "cba" else x, nd, True)
    y = whole(x, nd, False)
    y = flip(y) if case["kind"] == "cba" else y
    return (y, x) if case["direction"] == "pair" else y
