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


# instructions that only move a register: a spill, or a copy between registers
MOVES = ("scratch_store", "buffer_store", "v_accvgpr", "v_mov")


def masked_spills(asm: str) -> list[tuple[str, str]]:
    """Vector instructions that the compiler put between the head of a block
    where lanes come together again and that block's restore of the lane mask, as
    (kernel, instruction). A register spill or copy there moves only the lanes
    that were on, none after a loop that every lane left, and the others read
    garbage later on.

    Where the block is known to be such a join (the target of s_cbranch_execz, the
    exit of a loop that lanes leave one by one) every vector instruction counts. A
    block that only might be one (the branch round it was left out, the head of an
    else, a mask restored by a move) also holds code of its own before the mask
    changes: of it the spills count, which belong to every lane."""
    joins = set(re.findall(r"s_cbranch_execz (\.LBB\w+)", asm))
    found, kernel, join, seen, loop_end = [], "", False, [], False
    spills, here = [], set()  # spills of the block so far (None: its mask has changed), masks computed in it
    for line in asm.split("\n"):
        label = re.match(r"(_Z\w+|\.LBB\w+):", line)
        if label:
            if label[1].startswith("_Z"):
                kernel = label[1]
            join, seen = label[1] in joins, []
            spills, here = [], set()
            continue
        text = line.split(";")[0].strip()
        op, _, args = text.partition(" ")
        if spills is not None and text and not text.startswith("."):
            if "Folded Spill" in line:
                spills.append(text)
            elif "saveexec" in op or args.startswith("exec,"):
                source = args.rsplit(",", 1)[-1].strip()
                widens = op.startswith(("s_or", "s_xor", "s_andn2_saveexec")) or (op == "s_mov_b64" and source not in here)
                if widens and not (join and op == "s_or_b64"):  # (that one is looked at below)
                    found += [(kernel, t) for t in spills]
                spills = None
            elif op.startswith("s_"):
                here.add(args.split(",")[0])
        if text.startswith("s_cbranch_execnz"):  # falls through with no lane left
            join, seen = True, []
        elif line.startswith("; %bb."):
            join = join and loop_end
            spills, here = [], set()
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
        moves = [b for b in bad if b[1].startswith(MOVES)]
        for k, t in bad:
            if (k, t) not in moves:  # (computed in lanes that may need it: to be looked at, not certain)
                sys.stderr.write(f"warning: under a partial lane mask in {k}: {t}\n")
        if moves:
            res.returncode = 1
            res.stderr += "vector registers moved under a partial lane mask:\n" + "".join(f"  {k}: {t}\n" for k, t in moves)
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
