"""Generate the explicit instantiations of the pass kernels and their registry.

For every 2/3/5-smooth length L <= 1024 and both precisions, one kernel per
radix sequence is compiled.  Radix sequences: the power-of-two part of L is
split into as few stages as possible with radix <= 16 (balanced), a
variant with radix <= 8 (balanced) and a greedy one (radix-16 stages plus one
remainder stage), and for 512 and 1024 also two radix-32-sized stages; each
factor 5 and 3 is its own stage.  Stages
run largest radix first.  Threads per line = L / (largest radix), so the
largest-radix stage does one butterfly per thread.  Beside these come the
kernels that kernel_defaults.txt names (the measured defaults, with composite
radices 6 to 30 and other thread counts).

Output: <outdir>/kernels_<prec>_<part>.hip, each holding a slice of the
instantiations and a table; <outdir>/registry_parts.inc lists the tables and
<outdir>/kernel_defaults.inc holds kernel_defaults.txt for the planner.
"""
from __future__ import annotations

import functools
import itertools
import math
import os
import sys

MAX_L = 1024
PARTS = 8  # translation units per precision (compiled in parallel)


def smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


def exponents(n):
    e = []
    for p in (2, 3, 5):
        k = 0
        while n % p == 0:
            n //= p
            k += 1
        e.append(k)
    return e


def split_pow2(p, maxbits):
    """Split 2^p into the fewest stages of at most 2^maxbits, balanced."""
    if p == 0:
        return []
    ns = -(-p // maxbits)
    base, extra = divmod(p, ns)
    bits = [base + (1 if i < extra else 0) for i in range(ns)]
    return [1 << b for b in bits]


def radix_seqs(L):
    """Radix sequences of L: the power-of-two part split balanced with radix
    <= 16, balanced with radix <= 8, greedily into radix-16 stages, and (for
    2^9 and 2^10, where it saves a stage and so an LDS exchange) balanced
    with radix <= 32; each 3 and 5 is its own stage."""
    if L == 1:
        return []
    p, q, r = exponents(L)
    seqs = []
    greedy = [16] * (p // 4) + ([1 << (p % 4)] if p % 4 else [])
    splits2 = [split_pow2(p, 4), split_pow2(p, 3), greedy]
    if p >= 9:
        splits2.append(split_pow2(p, 5))
    for twos in splits2:
        seq = sorted(twos + [5] * r + [3] * q, reverse=True)
        if seq not in seqs:
            seqs.append(seq)
    return seqs


def max_threads(prec, L=None, seq=None, tpl=None):
    """Launch bound of a stand-alone pass kernel: 512 threads for binary64;
    1024 for binary32, except the variants with half the threads per line
    (two largest-radix butterflies per thread), which get 512 so that their
    registers fit without spilling (a strided tile of 32 columns still fits:
    that is what they are for).  A few binary32 kernels of L = 1024 at the
    1024 bound, and binary64 ones of radix 32 x 32, still spill 8-76 bytes
    per lane; the tuner weighs them like any other candidate."""
    if prec != "f32":
        return 512
    if seq is not None and tpl < L // max(seq):
        return 512
    return 1024


def lengths():
    return [n for n in range(2, MAX_L + 1) if smooth(n)]


def splits(L, seq, P):
    """Whether every LDS exchange of the radix sequence can run in P parts:
    P divides the next radix and the span times radix of the stage before
    divides L/P (fft_device.hpp, exchange_splits)."""
    if P == 1:
        return True
    if len(seq) < 2 or L % P:
        return False
    ns = 1
    for r, r2 in zip(seq, seq[1:]):
        if r2 % P or (L // P) % (ns * r):
            return False
        ns *= r
    return True


# Launch bound of the transposing kernels in both precisions: their row table
# and row-side copy add registers, and at 1024 threads (128 registers) the
# binary32 ones would spill.
TRANSPOSE_MAX_THREADS = 512


def transposes(seq, P):
    """Whether a kernel also comes as a transposing pass: with P parts its row
    side moves part by part, which needs P to divide the first radix (rows
    in) and the last radix (rows out)."""
    return P == 1 or (seq[0] % P == 0 and seq[-1] % P == 0)


# Lengths whose strided tiles also get kernels with LDS exchanges in 2 and 4
# parts: a wide tile of these fills the LDS, and only part of each line then
# needs to be resident at a time.
PARTS_MIN_L = 256


DEFAULTS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "kernel_defaults.txt")


def parse_spec(L, spec):
    """(radix sequence, threads per line, parts) of a kernel spec
    "<radices>/<width>[/<threads per line>][/p<parts>]"."""
    seq_s, _, *rest = spec.split("/")
    seq = [int(r) for r in seq_s.split("x")]
    tpl, P = L // max(seq), 1
    for t in rest:
        if t.startswith("p"):
            P = int(t[1:])
        else:
            tpl = int(t)
    return seq, tpl, P


@functools.lru_cache(maxsize=None)
def _default_rows():
    with open(DEFAULTS) as f:
        return tuple(tuple(ln.split()) for ln in f if ln.strip() and not ln.startswith("#"))


@functools.lru_cache(maxsize=None)
def default_lines():
    """(precision, line kind, length, specs) of every line of
    kernel_defaults.txt that names kernels."""
    return tuple((r[0], r[1], int(r[2]), tuple(r[3:])) for r in _default_rows() if r[0] != "half")


def half_lengths(prec):
    """Lengths whose strided lines take half of the width on aligned rows."""
    return {int(n) for r in _default_rows() if r[:2] == ("half", prec) for n in r[2:]}


def default_entries(prec, L):
    """Kernels of length L that kernel_defaults.txt names, in file order."""
    out = []
    for p, _, n, specs in default_lines():
        if p == prec and n == L:
            for s in specs:
                seq, tpl, P = parse_spec(L, s)
                if (seq, tpl, P) not in out:
                    out.append((seq, tpl, P))
    return out


def entries(prec="f64", parts=True):
    """(L, radix sequence, threads per line, parts).  The default thread count
    is L / (largest radix); binary32 kernels of L >= 384 also come with half
    as many threads per line (two largest-radix butterflies per thread), which
    lets a strided tile span 32 columns (256-byte rows) under the thread
    limit.  Kernels of L >= PARTS_MIN_L whose exchanges split also come with
    2 and 4 parts (strided lines only).  Last come the kernels of
    kernel_defaults.txt."""
    out = []
    for L in lengths():
        for seq in radix_seqs(L):
            tpl = L // max(seq)
            tpls = [tpl] + ([tpl // 2] if prec == "f32" and L >= 384 and tpl % 2 == 0 else [])
            for t in tpls:
                out.append((L, seq, t, 1))
            if parts and L >= PARTS_MIN_L:
                for P in (2, 4):
                    if splits(L, seq, P):
                        for t in tpls:
                            out.append((L, seq, t, P))
        # the block kernels' sequences (their stand-alone passes) and the
        # measured defaults, where the sequences above do not hold them
        if L <= BLOCK_MAX_L and block_seq(L):
            e = (L, block_seq(L), L // max(block_seq(L)), 1)
            if e not in out:
                out.append(e)
        for seq, t, P in default_entries(prec, L):
            if (parts or P == 1) and (L, seq, t, P) not in out:
                out.append((L, seq, t, P))
    return out


def legacy(prec, L, seq, tpl, P):
    """Whether a kernel is one of the radix-sequence rules' (entries without
    kernel_defaults.txt)."""
    t0 = L // max(seq)
    tpls = [t0] + ([t0 // 2] if prec == "f32" and L >= 384 and t0 % 2 == 0 else [])
    return seq in radix_seqs(L) and tpl in tpls and (P == 1 or (L >= PARTS_MIN_L and P in (2, 4) and splits(L, seq, P)))


# Longest line of a block kernel (fft_block.hpp).
BLOCK_MAX_L = 256
# A precision has two block kernels.  Lines of up to 100 points have radices up
# to 10 and fit 80 registers in binary32 (six waves per SIMD) and 128 in
# binary64; the longer lines' radices 12 to 16 take up to 128, and in binary64
# more than 1024 threads leave.  (kernel, longest line, threads, waves per SIMD
# that its registers leave: 80, 128, 116 and 181 of them, attribute)
BLOCK_KERNELS = {"f64": (("short", 100, 1024, 4, ""), ("long", BLOCK_MAX_L, 512, 2, "")),
                 "f32": (("short", 100, 1024, 6, "__attribute__((amdgpu_waves_per_eu(6))) "),
                         ("long", BLOCK_MAX_L, 1024, 4, ""))}
# Radices of the block kernels' stages.
BLOCK_RADICES = (2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16)


@functools.lru_cache(maxsize=None)
def block_seq(L):
    """Radix sequence of a block kernel's lines: the fewest stages, of those
    the most even radices (one butterfly per thread in every stage, so uneven
    ones leave threads idle), largest first; None if the radices do not
    reach L in three stages."""
    best = None
    for n in (1, 2, 3):
        for seq in itertools.combinations_with_replacement(BLOCK_RADICES, n):
            if math.prod(seq) == L and (n > 1 or L <= 10):
                key = seq[-1] / seq[0]
                if best is None or key < best[0]:
                    best = (key, sorted(seq, reverse=True))
        if best:
            return best[1]
    return None


def block_cases(prec):
    """Kernel cases (L, radix sequence, threads per line) of the block kernel:
    one per length up to BLOCK_MAX_L, one butterfly per thread in every
    stage."""
    return [(L, block_seq(L), L // min(block_seq(L))) for L in lengths() if L <= BLOCK_MAX_L and block_seq(L)]


def emit_block(outdir):
    """block_<kernel>_<prec>.hip (the block kernels of a precision, a switch
    over their cases per axis) and block_cases.inc (the cases for the
    planner)."""
    files, inc = [], []
    for prec, vt, dcode in (("f64", "double2", 0), ("f32", "float2", 1)):
        cases = block_cases(prec)
        for name, max_l, threads, _, attr in BLOCK_KERNELS[prec]:
            lines = ["// generated by gen_kernels.py -- do not edit",
                     '#include "offt_internal.h"',
                     '#include "fft_block.hpp"',
                     "namespace offt {",
                     "namespace {",
                     "struct Pass {",
                     f"    __device__ __forceinline__ void operator()(const BlockArgs& a, {vt}* lds, const {vt}* tw, {vt}* go, "
                     "int axis, int tid) const {",
                     "        switch (a.kid[axis]) {"]
            for i, (L, seq, tpl) in enumerate(cases):
                if L <= max_l:
                    lines.append(f"            case {i}: block_pass<{vt}, {L}, {tpl}, {', '.join(map(str, seq))}>(a, lds, tw, go, axis, tid); break;")
            lines += ["            default: break;", "        }", "    }", "};",
                      f"__global__ void __launch_bounds__({threads}) {attr}fft_block_{name}_{prec}(BlockArgs a) {{",
                      "    extern __shared__ __align__(16) unsigned char smem_raw[];",
                      f"    block_body<{vt}>(a, reinterpret_cast<{vt}*>(smem_raw), (int64_t)blockIdx.x, Pass{{}});",
                      "}",
                      "}  // namespace",
                      f"hipError_t launch_block_{name}_{prec}(const BlockArgs& a, int64_t nblocks, int threads, size_t lds, "
                      "hipStream_t s) {",
                      "    static std::atomic<uint64_t> lds_raised{0};",
                      f"    return launch_kernel(&fft_block_{name}_{prec}, lds_raised, a, nblocks, threads, lds, s);",
                      "}",
                      "}  // namespace offt"]
            path = os.path.join(outdir, f"block_{name}_{prec}.hip")
            _write(path, "\n".join(lines) + "\n")
            files.append(path)
        for L, seq, tpl in cases:
            padded = ", ".join(str(x) for x in (list(seq) + [0] * (8 - len(seq))))
            inc.append(f"    {{{dcode}, {L}, {len(seq)}, {{{padded}}}, {tpl}}},")
    _write(os.path.join(outdir, "block_cases.inc"), "\n".join(inc) + "\n")
    protos = []
    for prec in BLOCK_KERNELS:
        for name, *_ in BLOCK_KERNELS[prec]:
            protos.append(f"hipError_t launch_block_{name}_{prec}(const BlockArgs& a, int64_t nblocks, int threads, size_t lds, hipStream_t s);")
    protos.append("struct BlockKernel { int dtype; int max_l; int threads; int waves; hipError_t (*launch)(const BlockArgs&, int64_t, int, size_t, hipStream_t); };")
    protos.append(f"constexpr int kBlockMaxLine = {BLOCK_MAX_L};")
    protos.append("static const BlockKernel kBlockKernels[] = {")
    for prec, dcode in (("f64", 0), ("f32", 1)):
        for name, max_l, threads, waves, _ in BLOCK_KERNELS[prec]:
            protos.append(f"    {{{dcode}, {max_l}, {threads}, {waves}, &launch_block_{name}_{prec}}},")
    protos.append("};")
    _write(os.path.join(outdir, "block_kernels.inc"), "\n".join(protos) + "\n")
    return files


def _write(path, text):
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)


def emit_defaults(outdir):
    """kernel_defaults.inc: {dtype, line kind, L, {spec per size class}, half
    of the last width on aligned rows} rows."""
    rows = []
    for prec, kind, L, specs in default_lines():
        for s in specs:
            seq, tpl, P = parse_spec(L, s)
            assert len(specs) == 3 and (P == 1 or (kind != "c" and splits(L, seq, P))), (prec, kind, L, s)
            assert kind != "t" or transposes(seq, P), (prec, kind, L, s)
        half = kind == "s" and L in half_lengths(prec)
        assert not half or int(specs[2].split("/")[1]) > 1
        rows.append(f"    {{{0 if prec == 'f64' else 1}, {'cst'.index(kind)}, {L}, "
                    f"{{{', '.join(chr(34) + s + chr(34) for s in specs)}}}, {int(half)}}},")
    text = "\n".join(rows) + "\n"
    _write(os.path.join(outdir, "kernel_defaults.inc"), text)


def emit(outdir):
    os.makedirs(outdir, exist_ok=True)
    emit_defaults(outdir)
    tables = []
    for prec, vt, dcode in (("f64", "double2", 0), ("f32", "float2", 1)):
        ents = entries(prec)
        extras = [e for e in ents if not legacy(prec, *e)]
        for part in range(PARTS):
            mine = ents[part::PARTS]
            name = f"kernels_{prec}_{part}"
            lines = [
                "// generated by gen_kernels.py -- do not edit",
                '#include "offt_internal.h"',
                '#include "fft_kernel.hpp"',
                "namespace offt {",
                "namespace {",
                "template <int MAXT, int L, int TPL, int P, int... Rs>",
                "hipError_t launch_one(const PassArgs& a, int64_t nblocks, int threads, size_t lds, hipStream_t s) {",
                f"    auto* k = &fft_pass_kernel<{vt}, MAXT, L, TPL, P, Rs...>;",
                "    static std::atomic<uint64_t> lds_raised{0};",
                "    return launch_kernel(k, lds_raised, a, nblocks, threads, lds, s);",
                "}",
                "template <int L, int TPL, int P, int... Rs>",
                "hipError_t launch_t_one(const PassArgs& a, int64_t nblocks, int threads, size_t lds, hipStream_t s) {",
                f"    auto* k = &fft_tpass_kernel<{vt}, {TRANSPOSE_MAX_THREADS}, L, TPL, P, Rs...>;",
                "    static std::atomic<uint64_t> lds_raised{0};",
                "    return launch_kernel(k, lds_raised, a, nblocks, threads, lds, s);",
                "}",
                "}  // namespace",
                f"extern KernelEntry g_{name}[];",
                f"extern const int g_{name}_n;",
                f"KernelEntry g_{name}[] = {{",
            ]
            for L, seq, tpl, P in mine:
                # (what kernel_defaults.txt adds is not among the learned
                # selector's candidates, whose training data it did not have)
                extra = int((L, seq, tpl, P) in extras)
                rad = ", ".join(str(x) for x in seq)
                padded = ", ".join(str(x) for x in (seq + [0] * (8 - len(seq))))
                # whole-line kernels, and kernels in parts whose first and last
                # radix split into the parts, also come as transposing passes
                lt = f"&launch_t_one<{L}, {tpl}, {P}, {rad}>" if transposes(seq, P) else "nullptr"
                mt = max_threads(prec, L, seq, tpl)
                lines.append(f"    {{{dcode}, {L}, {len(seq)}, {{{padded}}}, {tpl}, {mt}, {P}, "
                             f"&launch_one<{mt}, {L}, {tpl}, {P}, {rad}>, {lt}, {extra}}},")
            lines.append("};")
            lines.append(f"const int g_{name}_n = {len(mine)};")
            lines.append("}  // namespace offt")
            path = os.path.join(outdir, name + ".hip")
            _write(path, "\n".join(lines) + "\n")
            tables.append(name)
    inc = []
    for t in tables:
        inc.append(f"extern KernelEntry g_{t}[]; extern const int g_{t}_n;")
    inc.append("#define OFFT_REGISTRY_TABLES \\")
    inc.append(" \\\n".join(f"    {{g_{t}, g_{t}_n}}," for t in tables))
    text = "\n".join(inc) + "\n"
    _write(os.path.join(outdir, "registry_parts.inc"), text)
    return [os.path.join(outdir, t + ".hip") for t in tables] + emit_block(outdir)


if __name__ == "__main__":
    outdir = sys.argv[1] if len(sys.argv) > 1 else os.path.join(os.path.dirname(__file__), "_gen")
    files = emit(outdir)
    print(len(entries("f64")), "+", len(entries("f32")), "kernels in", len(files), "files")
