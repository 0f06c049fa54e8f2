"""Generate the batch executors of uneven batches (many-plans).

An executor compiles the tile code of a set of kernel cases (length, radix
sequence, threads per line) behind one switch, so that a single kernel can
run a tile of any grid of a batch: the level kernels (one tile per
workgroup, one launch per pass level), and for some executors the
persistent forms (a work-queue kernel and a level-synchronous kernel, each
one launch for the whole batch).  A plan uses the first executor whose set
covers all its passes; register use of an executor is that of its hungriest
case, so the lengths of the uneven-batch workload get a compact executor of
their own.

Output: <outdir>/many_<executor>_<prec>.hip (level and work-queue kernels),
<outdir>/many_sync_<executor>_<prec>.hip (level-synchronous kernel), and
<outdir>/many_executors.inc (the executor list and the lookup of the
level-synchronous kernels).
"""
from __future__ import annotations

import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gen_kernels import entries, legacy  # noqa: E402

sys.path.pop(0)

MANY_MAX_L = 160  # longest axis a batch executor dispatches

BATCH_LENGTHS = (48, 60, 64, 80, 96, 120, 128, 150, 160)
CASE_SETS = {"batch": lambda L: L in BATCH_LENGTHS, "all": lambda L: L <= MANY_MAX_L}

# Executors compiled into the library: (name, case set, persistent forms).
# The "all" set (every length <= 160) has its level kernels only.
EXECUTORS = (("batch", "batch", True), ("all", "all", False))


def many_cases(prec, which="all", rules_only=False):
    """Kernel cases (L, radix sequence, threads per line) of one case set;
    rules_only: without the kernels that only kernel_defaults.txt names, which
    the executors do not compile (many-plans choose among the others)."""
    keep = CASE_SETS[which]
    return [e[:3] for e in entries(prec, parts=False) if keep(e[0]) and not (rules_only and not legacy(prec, *e))]


# waves per SIMD the level-synchronous kernel is compiled for: 4, two
# 512-thread workgroups per CU (128 registers).  Its loop runs every case's
# tile code inline, which needs about 126 registers for complex64 (with the
# opaque thread index; without it the hoisted index math spills); asked for
# 6 waves (80 registers) it spills, and behind an out-of-line call (80
# registers, no spills) each tile pays the call's stack traffic and ran
# slower.
SYNC_WAVES_PER_EU = {"f32": 4, "f64": 4}

PRECISIONS = (("f64", "double2", 0), ("f32", "float2", 1))


def _write(path, lines):
    text = "\n".join(lines) + "\n"
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)
    return path


def _switch(fn, inline, tile, name, vt, cases):
    """A dispatch function: case i of the switch runs the tile code `tile`
    of kernel case i."""
    out = [f"__device__ {inline} void {fn}_{name}(int kid, const PassArgs& a, {vt}* lds, int64_t l0) {{",
           "    switch (kid) {"]
    for i, (L, seq, tpl) in enumerate(cases):
        rad = ", ".join(str(x) for x in seq)
        out.append(f"        case {i}: {tile}<{vt}, {L}, {tpl}, {rad}>(a, lds, l0); break;")
    out += ["        default: break;", "    }", "}"]
    return out


def _calls(name, vt, cases):
    """The persistent kernel's dispatch: one out-of-line function per kernel
    case and an inline switch that calls them.  (Inlined into the persistent
    loop, loop-invariant code of every case would be hoisted and kept live
    together.)  One function around the whole switch is not safe: beyond the
    128 KiB that a conditional branch reaches the compiler adds branches
    through s[30:31], where a function that calls nothing keeps its return
    address unsaved; the return then jumps to the last such target and the
    workgroup never ends (complex128, 15 cases: 157 KB; complex64: 125 KB with
    15 cases, 184 KB with 25, 307 KB with 50).  A case's tile is 3 to 17 KB.
    The case is uniform in the workgroup (readfirstlane: a scalar branch)."""
    out = []
    for i, (L, seq, tpl) in enumerate(cases):
        rad = ", ".join(str(x) for x in seq)
        out += [f"__device__ __noinline__ void tile_{name}_{i}(const PassArgs& a, {vt}* lds, int64_t l0) {{",
                f"    pass_tile_coherent<{vt}, {L}, {tpl}, {rad}>(a, lds, l0);",
                "}"]
    out += [f"__device__ __forceinline__ void dispatch_{name}(int kid, const PassArgs& a, {vt}* lds, int64_t l0) {{",
            "    switch (__builtin_amdgcn_readfirstlane(kid)) {"]
    out += [f"        case {i}: tile_{name}_{i}(a, lds, l0); break;" for i in range(len(cases))]
    out += ["        default: break;", "    }", "}"]
    return out


def _functor(struct, fn, name, vt):
    return [f"struct {struct}_{name} {{",
            f"    __device__ __forceinline__ void operator()(int kid, const PassArgs& a, {vt}* lds, int64_t l0) const {{",
            f"        {fn}_{name}(kid, a, lds, l0);",
            "    }",
            "};"]


def _executor_file(outdir, ex, persistent, prec, vt, dcode, cases):
    name = f"{ex}_{prec}"
    lines = ["// generated by gen_many.py -- do not edit",
             '#include "offt_internal.h"',
             '#include "many_device.hpp"',
             "namespace offt {",
             "namespace {"]
    if persistent:
        lines += _calls(name, vt, cases)
    # the level kernels are ordered by kernel boundaries: plain stores; one
    # tile per workgroup and no loop to hoist out of, so their dispatch is
    # inlined (no call frame)
    lines += _switch("dispatch_plain", "__forceinline__", "pass_tile", name, vt, cases)
    if persistent:
        lines += _functor("Dispatch", "dispatch", name, vt)
    lines += _functor("DispatchPlain", "dispatch_plain", name, vt)
    lines.append("}  // namespace")
    if persistent:
        lines += [f"__global__ void __launch_bounds__(512) many_kernel_{name}(ManyArgs a) {{",
                  "    extern __shared__ __align__(16) unsigned char smem_raw[];",
                  f"    many_body<{vt}>(a, reinterpret_cast<{vt}*>(smem_raw), Dispatch_{name}{{}});",
                  "}"]
    lines += [f"__global__ void __launch_bounds__(512) many_level_kernel_{name}(ManyArgs a, int64_t tile_begin) {{",
              "    extern __shared__ __align__(16) unsigned char smem_raw[];",
              f"    many_level_body<{vt}>(a, tile_begin, reinterpret_cast<{vt}*>(smem_raw), DispatchPlain_{name}{{}});",
              "}",
              f"static const ManyCase cases_{name}[] = {{"]
    for L, seq, tpl in cases:
        padded = ", ".join(str(x) for x in (seq + [0] * (8 - len(seq))))
        lines.append(f"    {{{dcode}, {L}, {len(seq)}, {{{padded}}}, {tpl}}},")
    kernel = f"reinterpret_cast<const void*>(&many_kernel_{name})" if persistent else "nullptr"
    lines += ["};",
              f"extern const ManyExecutor g_many_{name};",
              f"const ManyExecutor g_many_{name} = {{\"{ex}\", {dcode}, cases_{name}, {len(cases)}, "
              f"{kernel}, reinterpret_cast<const void*>(&many_level_kernel_{name})}};",
              "}  // namespace offt"]
    return _write(os.path.join(outdir, f"many_{name}.hip"), lines)


def _sync_file(outdir, ex, prec, vt, cases):
    """Level-synchronous persistent kernel: the plain tile code inlined into
    its loop, each tile's thread index opaque."""
    name = f"{ex}_{prec}"
    lines = ["// generated by gen_many.py -- do not edit",
             '#include "offt_internal.h"',
             '#include "many_device.hpp"',
             "namespace offt {",
             "namespace {"]
    lines += _switch("dispatch_looped", "__forceinline__", "pass_tile_looped", name, vt, cases)
    lines += _functor("DispatchLooped", "dispatch_looped", name, vt)
    lines += ["}  // namespace",
              f"__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu({SYNC_WAVES_PER_EU[prec]}))) "
              f"many_sync_kernel_{name}(ManyArgs a, ManySyncArgs g) {{",
              "    extern __shared__ __align__(16) unsigned char smem_raw[];",
              f"    many_sync_body<{vt}>(a, g, reinterpret_cast<{vt}*>(smem_raw), DispatchLooped_{name}{{}});",
              "}",
              f"const void* many_sync_kernel_{name}_address() {{",
              f"    return reinterpret_cast<const void*>(&many_sync_kernel_{name});",
              "}",
              "}  // namespace offt"]
    return _write(os.path.join(outdir, f"many_sync_{name}.hip"), lines)


def emit_many(outdir):
    os.makedirs(outdir, exist_ok=True)
    files = []
    for prec, vt, dcode in PRECISIONS:
        for ex, which, persistent in EXECUTORS:
            cases = many_cases(prec, which, rules_only=True)
            files.append(_executor_file(outdir, ex, persistent, prec, vt, dcode, cases))
            if persistent:
                # in a file of its own: its looped tile code and register
                # budget would otherwise change the code of the level kernels
                files.append(_sync_file(outdir, ex, prec, vt, cases))
    inc = [f"extern const ManyExecutor g_many_{ex}_{prec};" for prec, _, _ in PRECISIONS for ex, _, _ in EXECUTORS]
    inc.append("#define OFFT_MANY_EXECUTORS_F64 " + ", ".join(f"&g_many_{ex}_f64" for ex, _, _ in EXECUTORS))
    inc.append("#define OFFT_MANY_EXECUTORS_F32 " + ", ".join(f"&g_many_{ex}_f32" for ex, _, _ in EXECUTORS))
    # the level-synchronous kernels are looked up through these functions
    # (null for an executor without persistent forms)
    inc += [f"const void* many_sync_kernel_{ex}_{prec}_address();"
            for prec, _, _ in PRECISIONS for ex, _, persistent in EXECUTORS if persistent]
    inc.append("inline const void* many_sync_kernel(const ManyExecutor* e) {")
    for prec, _, _ in PRECISIONS:
        for ex, _, persistent in EXECUTORS:
            if persistent:
                inc.append(f"    if (e == &g_many_{ex}_{prec}) return many_sync_kernel_{ex}_{prec}_address();")
    inc += ["    return nullptr;", "}"]
    _write(os.path.join(outdir, "many_executors.inc"), inc)
    return files


if __name__ == "__main__":
    outdir = sys.argv[1] if len(sys.argv) > 1 else os.path.join(os.path.dirname(__file__), "_gen")
    files = emit_many(outdir)
    print(len(files), "files;", [(ex, len(many_cases("f32", which))) for ex, which, _ in EXECUTORS],
          "cases per executor (f32)")
