"""The measured default kernels (csrc/kernel_defaults.txt), host side: every
spec names a compiled kernel, and default plans follow the table's size
classes and its line threshold."""
import importlib.util
import os

import pytest
import torch

import paper_1501_07350_amd as offt

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1501_07350_amd", "csrc")
DTYPES = {"f64": torch.complex128, "f32": torch.complex64}


@pytest.fixture(scope="module")
def gk():
    spec = importlib.util.spec_from_file_location("gen_kernels_defaults", os.path.join(CSRC, "gen_kernels.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _fields(plan):
    return dict(f.split("=", 1) for f in plan.split("|")[0].split(";"))


def test_every_spec_names_a_compiled_kernel(gk):
    compiled = {prec: {(L, tuple(seq), tpl, P) for L, seq, tpl, P in gk.entries(prec)} for prec in DTYPES}
    for prec, kind, L, specs in gk.default_lines():
        assert len(specs) == 3
        for s in specs:
            seq, tpl, P = gk.parse_spec(L, s)
            assert (L, tuple(seq), tpl, P) in compiled[prec]
            axis, shape, lay = {"s": ("a", (L, 2, 8), "natural"), "c": ("c", (2, 4, L), "natural"),
                                "t": ("a", (L, 2, 8), "cba")}[kind]
            plan = "order=cba;" + ("rev=a;" if kind == "t" else "") + f"{axis}={s}"
            plan = offt.plan_string(shape, DTYPES[prec], lay,
                                    plan if lay == "natural" else plan + "|" + offt.plan_string(shape[::-1], DTYPES[prec], "cba").split("|")[0])
            assert _fields(plan)[axis] == s


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_default_plans_follow_the_size_classes(gk, prec):
    table = {(p, k, L): specs for p, k, L, specs in gk.default_lines()}

    def kernel(L, spec):
        return gk.parse_spec(L, spec.replace("/x", ""))
    es = 16 if prec == "f64" else 8
    # rows longer than a block kernel's (256 points), so that every pass runs alone
    for shape in [(16, 20, 270), (32, 60, 288), (90, 100, 300), (128, 128, 320), (225, 320, 300), (512, 480, 450)]:
        n = shape[0] * shape[1] * shape[2]
        limit = 256 << 20
        cls = 0 if n * es <= 8 << 20 else (1 if n * es <= limit else 2)
        f = _fields(offt.default_plan_string(shape, DTYPES[prec]))
        for i, ax in enumerate("abc"):
            L = shape[i]
            assert n // L >= 256
            assert kernel(L, f[ax]) == kernel(L, table[(prec, "c" if ax == "c" else "s", L)][cls])


def test_few_lines_keep_the_rules_kernels(gk):
    # 2 x 100 = 200 lines of 480 points against 3 x 100 = 300
    few = _fields(offt.default_plan_string((2, 100, 480), torch.complex128))["c"]
    many = _fields(offt.default_plan_string((3, 100, 480), torch.complex128))["c"]
    assert few.split("/")[0] == "16x5x3x2"
    assert gk.parse_spec(480, many) == gk.parse_spec(480, {(p, k, L): s for p, k, L, s in gk.default_lines()}[("f64", "c", 480)][0])
