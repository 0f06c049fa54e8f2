"""Default kernels of streaming strided passes by the stride, host side."""
import ctypes
import importlib.util
import os

import pytest
import torch

import paper_1501_07350_amd as offt

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1501_07350_amd", "csrc")
DTYPES = {"f64": torch.complex128, "f32": torch.complex64}


@pytest.fixture(scope="module")
def gk():
    spec = importlib.util.spec_from_file_location("gen_kernels_strided", os.path.join(CSRC, "gen_kernels.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _fields(plan):
    return dict(f.split("=", 1) for f in plan.split(";"))


@pytest.mark.parametrize("prec,stride,from_table", [("f64", 5, False), ("f64", 6, False), ("f64", 8, True), ("f32", 5, False),
                                                    ("f32", 15, False), ("f32", 16, True)])
def test_strides_below_a_cache_line(gk, prec, stride, from_table):
    """Axis c of a 4-D grid above 256 MiB, 300 points on a stride of `stride`
    elements: from 128 bytes on the table's kernel, below one of the rules."""
    shape = (90, 400, 300, stride)
    plan = offt.plan_string_nd(shape, DTYPES[prec])
    seq, tpl, P = gk.parse_spec(300, _fields(plan)["c"].replace("/x", ""))
    table = {(p, k, L): specs for p, k, L, specs in gk.default_lines()}[(prec, "s", 300)]
    assert ((seq, tpl, P) == gk.parse_spec(300, table[2])) == from_table
    assert from_table or gk.legacy(prec, 300, seq, tpl, P)


@pytest.mark.parametrize("L,listed", [(75, True), (125, True), (80, False), (100, False)])
@pytest.mark.parametrize("columns", [500, 512, 540, 640])
def test_width_by_row_alignment(gk, L, listed, columns):
    """Streaming strided lines of a length in the half list: the table's width
    where rows are no whole cache lines, half of it where they are; other
    lengths keep the width.  (Lengths whose tiles fit any device's LDS.)"""
    assert (L in gk.half_lengths("f32")) == listed
    spec = {(p, k, n): s for p, k, n, s in gk.default_lines()}[("f32", "s", L)][2].split("/")
    got = _fields(offt.default_plan_string((1000, L, columns), DTYPES["f32"]))["b"].split("/")
    assert got[0] == spec[0]
    assert int(got[1]) == int(spec[1]) // (2 if listed and columns * 8 % 128 == 0 else 1)


def test_large_transposing_pass_of_512():
    """Reversed 512^3, complex128: the transposing pass of a large grid takes
    16 x 16 x 2 (8 x 8 x 8 took 1.09 of its time; the width is the device's)."""
    plan = offt.plan_string((512, 512, 512), DTYPES["f64"], "cba")
    assert [_fields(p)["a"].split("/")[0] for p in plan.split("|")] == ["16x16x2"] * 2


@pytest.mark.parametrize("prec,m,half_row,half", [
    ("f64", (360, 360), 256, True), ("f64", (480, 500), 256, False),    # complex128: the line at 2 MiB
    ("f64", (512, 256), 256, True), ("f64", (400, 400), 256, False),    # above it at powers of two only
    ("f64", (512, 256), 128, False), ("f64", (360, 360), 128, True),    # halves of 128 bytes below it only
    ("f32", (512, 500), 128, True), ("f32", (512, 512), 128, False),
    ("f32", (512, 512), 256, True), ("f32", (800, 600), 256, True),
    ("f32", (801, 601), 256, False), ("f32", (1, 5), 256, True)])       # rows of partial lines
def test_width_by_row_distance(prec, m, half_row, half):
    """Streaming strided lines whose rows lie m elements apart: half of the
    width or not."""
    es = 16 if prec == "f64" else 8
    assert bool(offt._lib.load().offt_test_halves_width(ctypes.c_int64(m[0] * m[1] * es), ctypes.c_int64(2 * half_row),
                                                        ctypes.c_int64(es))) == half
