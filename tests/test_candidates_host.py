"""The learned selector's candidates follow the batch, host side."""
import importlib.util
import os

import pytest

import paper_1501_07350_amd as offt
from paper_1501_07350_amd import selector

CSRC = os.path.join(os.path.dirname(os.path.abspath(offt.__file__)), "csrc")


@pytest.fixture(scope="module")
def gk():
    spec = importlib.util.spec_from_file_location("gen_kernels_candidates", os.path.join(CSRC, "gen_kernels.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("prec,dtype", [("f64", 0), ("f32", 1)])
@pytest.mark.parametrize("batch,cls", [(1, 1), (32, 2)])
def test_first_candidate_is_the_batch_default(gk, prec, dtype, batch, cls):
    """90 x 100 x 300 alone and 32 times (above 256 MiB): the first candidate
    and what the others vary have the kernels of the whole batch's bytes."""
    shape = (90, 100, 300)
    table = {(p, k, n): s for p, k, n, s in gk.default_lines()}
    plans, _ = selector.candidates(shape, batch, dtype)
    want = {}
    for ax, n in zip("abc", shape):
        want[ax] = gk.parse_spec(n, table[(prec, "c" if ax == "c" else "s", n)][cls])
    fields = [dict(f.split("=", 1) for f in p.split(";")) for p in plans]
    same = [[gk.parse_spec(n, f[ax].replace("/x", "").replace("/s", "").replace("/c", "")) == want[ax]
             for ax, n in zip("abc", shape)] for f in fields]
    assert all(same[0])
    assert all(sum(s) >= 2 for s in same)      # the others change one axis's kernel at most


@pytest.mark.parametrize("shape,dtype", [((64, 64, 64), 1), ((48, 48, 48), 0), ((16, 12, 18), 1)])
def test_candidates_keep_the_block_launch(shape, dtype):
    """Where the default runs passes c and b (and a) as blocks, every candidate
    does: c before b, with the default's kernels."""
    plans, feats = selector.candidates(shape, 1, dtype)
    fields = [dict(f.split("=", 1) for f in p.split(";")) for p in plans]
    assert len(plans) > 4 and len(feats) == len(plans)
    assert all(f["order"].startswith("cb") or f["order"] == "acb" for f in fields)
    assert all(f[ax].split("/")[0] == fields[0][ax].split("/")[0] for f in fields for ax in "bc")


def test_candidates_of_separate_passes_have_every_order():
    plans, _ = selector.candidates((40, 450, 500), 1, 1)
    assert len({p.split(";")[0] for p in plans}) == 6
