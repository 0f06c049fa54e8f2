"""Block kernels on the GPU: plans whose passes over c and b (and a) run as one
launch give the same bits as the same plan named explicitly (which runs pass
by pass), and match the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1501_07350_amd as offt
import synth
from oracle import layout, ndim

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128

# whole grids (up to 4096 points; more from 512 grids on), planes (several and
# one round of lines, rows of one and of three stages, one block to a CU), and
# lengths on both sides of the two kernels' limit of 100 points
SHAPES = [((2, 2, 2), 1), ((16, 16, 16), 3), ((9, 5, 27), 2), ((12, 10, 18), 520), ((32, 32, 32), 1), ((24, 50, 48), 9),
          ((64, 81, 100), 1), ((64, 108, 45), 1), ((128, 128, 128), 1), ((1, 64, 60), 5), ((5, 162, 20), 1), ((3, 4, 250), 40)]


def _grids(shape, batch, dtype):
    x = torch.stack([synth.complex_grid(shape, dtype, key=synth.SEED + g, device="cuda") for g in range(batch)])
    return x if batch > 1 else x[0]


@pytest.mark.parametrize("shape,batch", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"b{v}")
@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_block_plans_match_pass_by_pass(shape, batch, dtype):
    x = _grids(shape, batch, dtype)
    plan = offt.Plan(shape, dtype=dtype, batch=batch, normalize_inverse=True)
    alone = offt.Plan(shape, dtype=dtype, batch=batch, normalize_inverse=True, tune="forced", forced_plan=plan.describe())
    assert alone.describe() == plan.describe()
    y, ya = plan.forward(x), alone.forward(x)
    z, za = plan.backward(y), alone.backward(ya)
    inplace = x.clone()
    plan.forward(inplace, out=inplace)
    # pass by pass through the same plan object
    yp = torch.empty_like(x)
    st = torch.cuda.current_stream().cuda_stream
    for i in range(plan.npasses()):
        plan.exec_pass(i, offt.FORWARD, x.data_ptr(), yp.data_ptr(), st)
    torch.cuda.synchronize()
    assert torch.equal(y, ya) and torch.equal(z, za) and torch.equal(inplace, y) and torch.equal(yp, y)
    tol = oracle.tolerance(int(np.prod(shape)), dtype == C64)
    for g in sorted({0, batch - 1}):
        xg, yg, zg = (x[g], y[g], z[g]) if batch > 1 else (x, y, z)
        xh = xg.cpu().numpy().astype(np.complex128)
        assert oracle.rel_l2(yg.cpu().numpy(), oracle.fft3(xh)) <= tol
        assert oracle.rel_l2(zg.cpu().numpy(), xh) <= tol


@pytest.mark.parametrize("dtype", [C128, C64], ids=["c128", "c64"])
def test_block_planes_in_other_plans(dtype):
    """Reversed output order (the planes go through the workspace), four axes
    (with the plan named explicitly beside it) and graph replay on new
    buffers."""
    shape = (20, 40, 36)
    x = synth.complex_grid(shape, dtype, device="cuda")
    xh = x.cpu().numpy().astype(np.complex128)
    tol = oracle.tolerance(x.numel(), dtype == C64)
    rev = offt.Plan(shape, dtype=dtype, layout="cba", normalize_inverse=True)
    named = offt.Plan(shape, dtype=dtype, layout="cba", normalize_inverse=True, tune="forced", forced_plan=rev.describe())
    y = rev.forward(x)
    z = rev.backward(y)
    torch.cuda.synchronize()
    assert torch.equal(y, named.forward(x))
    assert oracle.rel_l2(y.cpu().numpy(), layout.fft3_reversed(xh)) <= tol
    assert oracle.rel_l2(z.cpu().numpy(), xh) <= tol
    shape4 = (6, 9, 24, 20)
    x4 = synth.complex_grid(shape4, dtype, device="cuda")
    p4 = offt.Plan(shape4, dtype=dtype)
    n4 = offt.Plan(shape4, dtype=dtype, tune="forced", forced_plan=p4.describe())
    y4 = p4.forward(x4)
    torch.cuda.synchronize()
    assert torch.equal(y4, n4.forward(x4))
    assert oracle.rel_l2(y4.cpu().numpy(), ndim.fftn(x4.cpu().numpy().astype(np.complex128))) <= oracle.tolerance(x4.numel(), dtype == C64)
    graph = offt.Plan(shape, dtype=dtype, use_graph=True)
    direct = offt.Plan(shape, dtype=dtype)
    for k in range(3):
        xk = synth.complex_grid(shape, dtype, key=synth.SEED + 40 + k, device="cuda")
        out = torch.empty_like(xk)
        for _ in range(2):
            graph.forward(xk, out=out)
            torch.cuda.synchronize()
            assert torch.equal(out, direct.forward(xk))
