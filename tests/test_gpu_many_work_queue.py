"""The work-queue kernel of uneven batches in both precisions: every length of
its case set on every axis, bit for bit against the same plans as separate
launches, directly and replayed from its graph."""
import pytest
import torch

import paper_1501_07350_amd as offt
import synth
from test_gpu_many import C64, C128, check_against_oracle, packed_input, same_grids

pytestmark = pytest.mark.gpu

LENGTHS = (48, 60, 64, 80, 96, 120, 128, 150, 160)


@pytest.mark.parametrize("dtype", [C64, C128], ids=["c64", "c128"])
def test_work_queue_every_length(dtype):
    dims = [(LENGTHS[i], LENGTHS[(i + 4) % 9], LENGTHS[(i + 7) % 9]) for i in range(9)]
    plan = offt.ManyPlan(dims, dtype=dtype, normalize_inverse=True)
    print(plan.describe().splitlines()[0], flush=True)
    assert "executor batch" in plan.describe()
    grids, x = packed_input(plan, dims, dtype, key0=synth.SEED + 600)
    sep = plan.execute(x, use_graph=offt.MANY_SEPARATE_TUNED)
    for form in (offt.MANY_PERSISTENT, offt.MANY_PERSISTENT_GRAPH, offt.MANY_PERSISTENT_GRAPH):
        print(f"form {form}", flush=True)
        y = plan.execute(x, use_graph=form)
        torch.cuda.synchronize()
        assert plan.status() == 0
        assert same_grids(plan, y, sep)
    check_against_oracle(plan, grids, y, dtype)
