"""Build the HIP library libsos.so in-tree for gfx950 with hipcc.

The sources compile to objects in parallel (the fused CG kernel once per
number of x-y columns per thread, 1 to 4, its on-chip form once per set of
variants) and are linked into one shared
library next to this file.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsos.so")
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
ARCH = "gfx950"
# (source, extra defines, object name)
UNITS = [("sos_kernels.hip", [], "sos_kernels.o"),
         ("sos_api.hip", [], "sos_api.o"),
         ("sos_cmaes.cpp", [], "sos_cmaes.o")] + \
        [("sos_fused.hip", [f"-DSOS_FUSED_CPT={c}", "-DSOS_CHIP_APART"], f"sos_fused_c{c}.o") for c in (1, 2, 3, 4)] + \
        [("sos_chip.hip", [f"-DSOS_CHIP_SET={k}"], f"sos_chip_{k}.o") for k in (0, 1, 2, 3, 4, 5)]


def hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _flags():
    return [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
            # packed FP32 instructions are kept out of the generated code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include")]


def masked_spills(asm: str) -> list[tuple[str, str]]:
    """Vector instructions that the compiler put between the head of a block
    where lanes come together again (the target of s_cbranch_execz, the exit of a
    loop that lanes leave one by one) and that block's restore of the lane mask,
    as (kernel, instruction). A register spill
    or copy there moves only the lanes that took the branch, none after a loop
    that every lane left, and the others read garbage later on."""
    joins = set(re.findall(r"s_cbranch_execz (\.LBB\w+)", asm))
    found, kernel, join, seen, loop_end = [], "", False, [], False
    for line in asm.split("\n"):
        label = re.match(r"(_Z\w+|\.LBB\w+):", line)
        if label:
            if label[1].startswith("_Z"):
                kernel = label[1]
            join, seen = label[1] in joins, []
            continue
        text = line.split(";")[0].strip()
        if text.startswith("s_cbranch_execnz"):  # falls through with no lane left
            join, seen = True, []
        elif line.startswith("; %bb."):
            join = join and loop_end
        elif not join or not text or text.startswith("."):
            continue
        elif text.startswith("s_or_b64 exec, exec"):
            found += [(kernel, t) for t in seen]
            join = False
        elif "exec" in text or text.startswith(("s_branch", "s_cbranch", "s_barrier")):
            join = False
        elif not text.startswith(("s_", "v_writelane", "v_readlane", "v_readfirstlane")):
            seen.append(text)
        loop_end = text.startswith("s_cbranch_execnz") or (loop_end and not text)
    return found


def _compile(unit, verbose):
    src, defs, obj = unit
    out = os.path.join(OBJDIR, obj)
    cmd = [hipcc(), *_flags(), *defs, "-c", os.path.join(CSRC, src), "-o", out]
    device = src.endswith(".hip")
    if device:  # keep the kernels' assembly, in a folder of the unit's own
        tmp = out + ".tmp"
        shutil.rmtree(tmp, ignore_errors=True)
        os.makedirs(tmp)
        cmd[-1] = os.path.join(tmp, "unit.o")
        cmd.append("-save-temps=obj")
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if device and res.returncode == 0:
        bad = []
        asm = [name for name in os.listdir(tmp) if ARCH in name and name.endswith(".s")]
        if not asm:
            raise RuntimeError("no assembly of " + src)
        for name in asm:
            with open(os.path.join(tmp, name)) as f:
                bad += masked_spills(f.read())
        if bad:
            res.returncode = 1
            res.stderr += "vector registers moved under a partial lane mask:\n" + "".join(f"  {k}: {t}\n" for k, t in bad)
        else:
            os.replace(os.path.join(tmp, "unit.o"), out)
        shutil.rmtree(tmp, ignore_errors=True)
    return cmd, res


def build(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every source and link libsos.so (always rebuilds)."""
    os.makedirs(OBJDIR, exist_ok=True)
    jobs = jobs or min(len(UNITS), max(1, os.cpu_count() or 1))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(lambda u: _compile(u, verbose), UNITS))
    for cmd, res in results:
        if res.returncode != 0:
            sys.stderr.write(" ".join(cmd) + "\n" + res.stdout + res.stderr)
            raise RuntimeError("hipcc failed building libsos.so")
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *[os.path.join(OBJDIR, u[2]) for u in UNITS],
           # roctx ranges around the outer iterations (rocprofv3 --marker-trace)
           "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx", "-Wl,-rpath,/opt/rocm/lib", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed linking libsos.so")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
