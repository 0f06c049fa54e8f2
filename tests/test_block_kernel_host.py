"""The block kernel's body (csrc/fft_block.hpp: the passes of a plane or of a
whole small grid in LDS) on CPU threads under AddressSanitizer and UBSan, with
exactly the launch's LDS, against the oracle; and the rule that chooses it."""
import fcntl
import hashlib
import importlib.util
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_1501_07350_amd as offt

HERE = os.path.dirname(os.path.abspath(__file__))
EMU, DRIVER = os.path.join(HERE, "emu"), os.path.join(HERE, "emu_block", "block_driver.cpp")
CSRC = os.path.join(os.path.dirname(HERE), "paper_1501_07350_amd", "csrc")
BUILD = os.path.join(HERE, "emu_block", "_build")
LENGTHS = (2, 5, 9, 12, 15, 16, 18, 27, 30, 48)


@pytest.fixture(scope="module")
def gk():
    spec = importlib.util.spec_from_file_location("gen_kernels_block", os.path.join(CSRC, "gen_kernels.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.fixture(scope="module")
def driver(gk):
    text = ("namespace offt {\ntemplate <typename V> struct EmuPass { void operator()(const BlockArgs& a, V* lds, const V* tw, "
            "V* go, int axis, int tid) const { switch (a.kid[axis]) {\n")
    for L in LENGTHS:
        seq = gk.block_seq(L)
        text += f"case {L}: block_pass<V, {L}, {L // min(seq)}, {', '.join(map(str, seq))}>(a, lds, tw, go, axis, tid); break;\n"
    text += "default: break; } } };\n}\n"
    h = hashlib.sha256(text.encode())
    for p in (DRIVER, os.path.join(EMU, "hip_emu.h"), os.path.join(CSRC, "fft_block.hpp"), os.path.join(CSRC, "fft_device.hpp")):
        h.update(open(p, "rb").read())
    out = os.path.join(BUILD, h.hexdigest()[:16])
    exe = os.path.join(out, "block_driver")
    os.makedirs(out, exist_ok=True)
    with open(os.path.join(BUILD, "lock"), "w") as lk:
        fcntl.flock(lk, fcntl.LOCK_EX)
        if not os.path.exists(exe):
            with open(os.path.join(out, "block_cases_emu.inc"), "w") as f:
                f.write(text)
            subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined",
                            "-fno-sanitize-recover=undefined", "-I", EMU, "-I", out, "-I", CSRC, DRIVER, "-o", exe + ".tmp"],
                           check=True)
            os.replace(exe + ".tmp", exe)
    return exe


# (A, B, C, naxes, threads, blocks): planes and whole grids; several rounds of
# lines with a ragged last one, threads beyond the last whole line, a single
# round, one-stage and three-stage lines
CASES = [(1, 12, 30, 2, 64, 2), (1, 48, 5, 2, 64, 1), (1, 2, 27, 2, 64, 3), (1, 30, 48, 2, 128, 1), (1, 16, 16, 2, 256, 1),
         (9, 5, 12, 3, 64, 2), (2, 18, 15, 3, 128, 1), (16, 2, 9, 3, 64, 1), (5, 9, 18, 3, 192, 1)]


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128], ids=["c64", "c128"])
@pytest.mark.parametrize("backward", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_emulated_block(driver, dtype, case, backward):
    A, B, C, naxes, threads, blocks = case
    args = [driver, "0" if dtype == torch.complex128 else "1"] + [str(v) for v in (A, B, C, naxes, threads, blocks, backward, C, B, A)]
    r = subprocess.run(args, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = r.stdout.splitlines()
    assert lines[0] == "OK"
    vals = np.array([[float(t) for t in ln.split()] for ln in lines[1:]])
    got = (vals[:, 0] + 1j * vals[:, 1]).reshape(blocks, A, B, C)
    i = np.arange(got.size)
    x = np.sin(0.37 * i + 0.1) + 1j * np.cos(0.91 * i)
    if dtype == torch.complex64:
        x = x.astype(np.complex64).astype(np.complex128)
    x = x.reshape(got.shape)
    for k in range(blocks):
        want = oracle.fft3(np.conj(x[k])).conj() / x[k].size if backward else oracle.fft3(x[k])
        assert oracle.rel_l2(got[k], want) <= oracle.tolerance(x[k].size, dtype == torch.complex64)


def _default_sequences(shape, dtype):
    f = dict(t.split("=", 1) for t in offt.default_plan_string(shape, dtype).split(";"))
    return [[int(r) for r in f[ax].split("/")[0].split("x")] for ax in "abc"]


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128], ids=["c64", "c128"])
def test_default_plans_name_the_block_sequences(gk, dtype):
    """The default plan's passes that run as a block kernel carry its radix
    sequences: every axis of a 12^3 grid; the planes' axes, not a, of 60^3 in
    complex64 (60 x 65 x 8 bytes: two planes to a CU); none of 12 x 150 x 60
    in complex128 (a 150 x 60 plane fills a CU, and only 12 of them)."""
    assert _default_sequences((12, 12, 12), dtype) == [gk.block_seq(12)] * 3
    assert _default_sequences((8, 9, 32), dtype) == [gk.block_seq(n) for n in (8, 9, 32)]
    assert _default_sequences((8, 8, 32), dtype)[2] == ([16, 2] if dtype == torch.complex128 else [8, 4])
    if dtype == torch.complex64:
        assert _default_sequences((60, 64, 60), dtype)[1:] == [gk.block_seq(64), gk.block_seq(60)]
    else:
        prec = {(p, k, L): s for p, k, L, s in gk.default_lines()}
        assert _default_sequences((12, 150, 60), dtype)[2] == gk.parse_spec(60, prec[("f64", "c", 60)][0])[0]


def test_block_index_helpers():
    """f div C by multiplication with ceil(2^32 / C), for every f < 2^16 and
    every row length."""
    f = np.arange(1 << 16, dtype=np.uint64)
    for C in range(2, 1025):
        m = np.uint64(((1 << 32) + C - 1) // C)
        assert np.array_equal((f * m) >> np.uint64(32), f // np.uint64(C))
