"""Contiguous lines in the level kernels: rows are staged several elements a
thread at a time with a remainder, so batches whose row counts end inside a
tile, at its edge and one row after it give the same bits as the stand-alone
passes, and match the oracle."""
import pytest
import torch

import oracle
import paper_1501_07350_amd as offt
import synth
from test_gpu_many import C64, C128, check_against_oracle, packed_input, same_grids

pytestmark = pytest.mark.gpu

ROWS = [1, 2, 3, 5, 8, 9, 15, 16, 25, 27, 32, 64, 81]


@pytest.mark.parametrize("lengths", [(6, 8, 27), (48, 50, 54), (60, 64, 75), (96, 100, 128), (144, 150, 160)],
                         ids=lambda v: "x".join(map(str, v)))
@pytest.mark.parametrize("dtype", [C64, C128], ids=["c64", "c128"])
def test_rows_around_tile_edges(lengths, dtype):
    dims = [(1, r, L) for L in lengths for r in ROWS]
    plan = offt.ManyPlan(dims, dtype=dtype, normalize_inverse=True)
    grids, x = packed_input(plan, dims, dtype, key0=synth.SEED + 500)
    y = plan.execute(x, use_graph=3)
    sep = plan.execute(x, use_graph=-2)
    back = plan.execute(y, use_graph=3, direction=offt.BACKWARD)
    torch.cuda.synchronize()
    assert same_grids(plan, y, sep)
    check_against_oracle(plan, grids, y, dtype)
    for a, b in zip(grids, plan.unpack(back)):
        assert oracle.rel_l2(b.cpu().numpy(), a.cpu().numpy()) <= oracle.tolerance(a.numel(), dtype == C64)
