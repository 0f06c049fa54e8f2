"""Which launches a plan makes: passes over the last axes of small planes and
grids run as one block launch in default and tuned plans and in the plan that
their string names, with the bits of the passes one by one."""
import importlib.util
import os

import pytest
import torch

import paper_1501_07350_amd as offt
import synth

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
CSRC = os.path.join(os.path.dirname(os.path.abspath(offt.__file__)), "csrc")


def _kernels(plan, x):
    """Names of the kernels of one forward transform."""
    out = torch.empty(_out_shape(plan, x), dtype=x.dtype, device="cuda")
    plan.forward(x, out=out)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        plan.forward(x, out=out)
        torch.cuda.synchronize()
    return sorted(e.key for e in prof.key_averages() for _ in range(e.count) if "fft_" in e.key)


def _out_shape(plan, x):
    spectral = tuple(plan.spectral_shape)
    return tuple(x.shape[:x.dim() - len(spectral)]) + spectral


def _pass_by_pass(plan, x):
    y = torch.empty(_out_shape(plan, x), dtype=x.dtype, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for i in range(plan.npasses()):
        plan.exec_pass(i, offt.FORWARD, x.data_ptr(), y.data_ptr(), st)
    torch.cuda.synchronize()
    return y


# (shape, batch, layout, launches, of which block kernels); the last two on both
# sides of the limit on small blocks
CASES = [((16, 16, 16), 3, "natural", 1, 1), ((32, 32, 32), 1, "natural", 2, 1), ((40, 24, 36), 1, "cba", 2, 1),
         ((6, 9, 24, 20), 1, "natural", 3, 1), ((64, 120, 30), 6, "natural", 2, 1),
         ((1, 4, 6), 8192, "natural", 1, 1), ((1, 4, 6), 8193, "natural", 2, 0)]


@pytest.mark.parametrize("shape,batch,layout,launches,blocks", CASES,
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_launches_of_a_plan_and_of_its_string(shape, batch, layout, launches, blocks, dtype):
    full = ((batch,) if batch > 1 else ()) + shape
    x = synth.complex_grid((batch,) + shape if len(shape) == 3 else shape, dtype, device="cuda").reshape(full)
    plan = offt.Plan(shape, dtype=dtype, batch=batch, layout=layout)
    named = offt.Plan(shape, dtype=dtype, batch=batch, layout=layout, tune="forced", forced_plan=plan.describe())
    k = _kernels(plan, x)
    assert len(k) == launches and sum("fft_block" in n for n in k) == blocks, k
    assert _kernels(named, x) == k
    y, yn, yp = plan.forward(x), named.forward(x), _pass_by_pass(plan, x)
    torch.cuda.synchronize()
    assert torch.equal(y, yn) and torch.equal(y, yp)


@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_tuned_plan_runs_as_timed(dtype, tmp_path):
    """A tuned plan, the same from its cache entry and named by its string."""
    shape, cache = (24, 20, 18), str(tmp_path / "plans.txt")
    x = synth.complex_grid(shape, dtype, device="cuda")
    tuned = offt.Plan(shape, dtype=dtype, tune="exhaustive", cache_path=cache)
    again = offt.Plan(shape, dtype=dtype, tune="exhaustive", cache_path=cache)
    named = offt.Plan(shape, dtype=dtype, tune="forced", forced_plan=tuned.describe())
    k = _kernels(tuned, x)
    assert _kernels(again, x) == k and _kernels(named, x) == k
    y = tuned.forward(x)
    assert torch.equal(named.forward(x), y) and torch.equal(_pass_by_pass(tuned, x), y)


@pytest.mark.parametrize("prec,dtype", [("f64", C128), ("f32", C64)])
def test_default_kernels_pass_by_pass(prec, dtype):
    """The default table's kernels of lengths that blocks take, as passes of
    their own: the bits of the whole transform, which may run as blocks."""
    spec = importlib.util.spec_from_file_location("gen_kernels_launches", os.path.join(CSRC, "gen_kernels.py"))
    gk = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gk)
    ran = 0
    for p, kind, L, specs in gk.default_lines():
        if p != prec or kind == "t" or L > gk.BLOCK_MAX_L:
            continue
        axis, shape = ("a", (L, 3, 9)) if kind == "s" else ("c", (5, 9, L))
        x = synth.complex_grid(shape, dtype, key=synth.SEED + L, device="cuda")
        for s in sorted(set(specs)):
            plan = offt.Plan(shape, dtype=dtype, tune="forced", forced_plan=f"order=cba;{axis}={s}")
            assert torch.equal(_pass_by_pass(plan, x), plan.forward(x)), (kind, L, s)
            plan.close()
            ran += 1
    assert ran > 100
