"""The measured default kernels (csrc/kernel_defaults.txt) on the GPU: every
spec of the table, in the pass form its line stands for, against the oracle."""
import importlib.util
import os

import numpy as np
import pytest
import torch

import oracle
import paper_1501_07350_amd as offt
import synth
from oracle import layout

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1501_07350_amd", "csrc")
DTYPES = {"f64": torch.complex128, "f32": torch.complex64}


def _lines(prec, kind):
    spec = importlib.util.spec_from_file_location("gen_kernels_defaults", os.path.join(CSRC, "gen_kernels.py"))
    gk = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gk)
    return [(L, specs) for p, k, L, specs in gk.default_lines() if p == prec and k == kind]


# strided lines: 3 x 9 = 27 columns, contiguous: 45 lines, transposing: 3 x 5
# lines -- none a multiple of a tile width, so that the last tile is ragged
FORMS = {"s": ("a", lambda L: (L, 3, 9), "natural"),
         "c": ("c", lambda L: (5, 9, L), "natural"),
         "t": ("a", lambda L: (L, 3, 5), "cba")}


@pytest.mark.parametrize("kind", sorted(FORMS))
@pytest.mark.parametrize("prec", sorted(DTYPES))
def test_every_default_kernel_vs_oracle(prec, kind):
    axis, shape_of, order = FORMS[kind]
    dtype = DTYPES[prec]
    bad, ran = [], 0
    for L, specs in _lines(prec, kind):
        shape = shape_of(L)
        x = synth.complex_grid(shape, dtype, key=synth.SEED + L, device="cuda")
        xh = x.cpu().numpy().astype(np.complex128)
        ref = layout.fft3_reversed(xh) if kind == "t" else oracle.fft3(xh)
        for spec in sorted(set(specs)):
            plan = "order=cba;" + ("rev=a;" if kind == "t" else "") + f"{axis}={spec}"
            p = offt.Plan(shape, dtype=dtype, tune="forced", forced_plan=plan, layout=order)
            assert f";{axis}={spec}" in p.describe()
            y = p.forward(x)
            torch.cuda.synchronize()
            p.close()
            e = oracle.rel_l2(y.cpu().numpy(), ref)
            ran += 1
            if not e <= oracle.tolerance(x.numel(), dtype == torch.complex64):
                bad.append((L, spec, e))
    print(f"{prec} {kind}: {ran} kernels", flush=True)
    assert ran > 0 and not bad, bad[:10]


@pytest.mark.parametrize("shape,batch", [((24, 50, 48), 1), ((24, 50, 48), 8), ((100, 90, 108), 4), ((225, 250, 243), 2)],
                         ids=["small", "small-batch8", "medium", "large"])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
def test_default_plan_of_each_size_class(shape, batch, dtype):
    """The default plan of a batch in each size class (the class follows the
    bytes of the whole batch): grid by grid against the oracle, and the
    normalised round trip."""
    x = torch.stack([synth.complex_grid(shape, dtype, key=synth.SEED + g, device="cuda") for g in range(batch)])
    plan = offt.Plan(shape, dtype=dtype, batch=batch, normalize_inverse=True)
    x = x if batch > 1 else x[0]
    y = plan.forward(x)
    z = plan.backward(y)
    torch.cuda.synchronize()
    n = int(np.prod(shape))
    tol = oracle.tolerance(n, dtype == torch.complex64)
    for g in range(batch):
        xg, yg = (x[g], y[g]) if batch > 1 else (x, y)
        assert oracle.rel_l2(yg.cpu().numpy(), oracle.fft3(xg.cpu().numpy().astype(np.complex128))) <= tol
    assert oracle.rel_l2(z.cpu().numpy(), x.cpu().numpy()) <= tol
