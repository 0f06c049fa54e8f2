"""Machine code of the batch executors, cross-compiled for gfx950 without a GPU.

A conditional branch of this target reaches 128 KiB.  In a larger function the
compiler inserts branches through a register pair, and in a device function
that calls nothing it takes s[30:31] for that -- the return address, which
such a function keeps there without saving it.  The return then jumps to the
last of those targets instead of the caller: the kernel never ends.  So no
out-of-line function may be that large; the executors' case switches are the
only ones that can grow to it."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

import paper_1501_07350_amd as offt
from paper_1501_07350_amd import build

PKG = os.path.dirname(os.path.abspath(offt.__file__))
CSRC = os.path.join(PKG, "csrc")


def _gen_many():
    spec = importlib.util.spec_from_file_location("gen_many_code", os.path.join(CSRC, "gen_many.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _functions(asm):
    """(name, text) of every device function of an assembly listing (kernels
    end the program and have no return address)."""
    for m in re.finditer(r"^(_Z\w+):.*?^\.Lfunc_end\d+:", asm, re.M | re.S):
        if "s_setpc_b64 s[30:31]" in m.group(0):
            yield m.group(1), m.group(0)


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="hipcc is not installed")
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_out_of_line_code_keeps_its_return_address(tmp_path, prec):
    """The compiled work-queue kernels."""
    cases = "batch"
    gm = _gen_many()
    (vt, dcode), = [(v, d) for p, v, d in gm.PRECISIONS if p == prec]
    src = gm._executor_file(str(tmp_path), cases, True, prec, vt, dcode, gm.many_cases(prec, cases, rules_only=True))
    asm = str(tmp_path / "executor.s")
    r = subprocess.run([build.HIPCC, "-x", "hip", "-S", "--cuda-device-only", src, "-o", asm] + build.FLAGS,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(asm) as f:
        text = f.read()
    assert f"many_kernel_{cases}_{prec}" in text
    bad = [name for name, body in _functions(text) if "s_getpc_b64 s[30:31]" in body]
    assert not bad, bad
    assert len(list(_functions(text))) > 0
