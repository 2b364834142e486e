"""Build the HIP library libmpath.so for gfx950 (in-tree).

    python -m paper_2111_08744_amd.build

All device code is compiled with packed-FP32 instructions disabled, and the
assembly of every kernel is searched for misplaced_spills: a build that holds
one fails.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmpath.so")
SOURCES = ["mpath_host.cpp", "grid.hip", "cast.hip", "adjoint.hip", "lensing.hip", "finder.hip", "probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"


def flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")]


# Instructions that switch lanes on (a branch's end, the way to its other side),
# and those that leave fewer.
_WIDEN = re.compile(r"s_or_b64 exec,|s_or_saveexec_b64|s_orn2_saveexec_b64|s_andn2_saveexec_b64|s_mov_b64 exec,|"
                    r"s_xnor_b64 exec,|s_not_b64 exec,|s_wqm_b64 exec,|s_cselect_b64 exec,")
_NARROW = re.compile(r"s_and_saveexec_b64|s_andn1_saveexec_b64|s_and_b64 exec,|s_andn2_b64 exec,|s_xor_b64 exec,|"
                     r"v_cmpx_")


def _registers(text):
    found = set()
    for m in re.finditer(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])(?![\w\[])", text):
        lo = int(m[2] or m[3])
        found.update(m[1] + str(k) for k in range(lo, int(m[4] or lo) + 1))
    return found


class _Region:
    """The instructions since lanes were last switched on or off in a block."""

    def __init__(self):
        self.written, self.spills, self.reloads = set(), {}, {}

    def add(self, ins):
        op, _, args = ins.partition(" ")
        first, _, rest = args.partition(",")
        if op.startswith(("v_accvgpr_write", "scratch_store")):
            # to an accumulation register, or to the stack at an offset
            to_acc = op.startswith("v_acc")
            value = _registers(rest) if to_acc else _registers(rest.split(",")[0])
            if value and not value <= self.written:
                self.spills[first if to_acc else rest.partition(",")[2].strip()] = ins
            if to_acc:
                self.written |= _registers(first)
            return
        if op.startswith(("v_accvgpr_read", "scratch_load")):
            slot = rest.strip()
            self.spills.pop(slot if op.startswith("v_acc") else slot.partition(",")[2].strip() or slot, None)
            self.reloads[first] = (_registers(first), ins)
            self.written |= _registers(first)
            return
        if op.startswith(("v_", "ds_", "global_", "flat_", "buffer_")):
            stores = "store" in op or "write" in op
            used = _registers(args if stores else rest)
            self.reloads = {k: v for k, v in self.reloads.items() if not v[0] & used}
            if not stores:
                self.written |= _registers(first)


def misplaced_spills(text):
    """(function, block, instruction) of the vector spills and reloads in an
    assembly listing that come before their block switches lanes on and are not
    the business of the lanes then running: a spill of a register that the block
    has not written and does not reload before, a reload that nothing reads
    before.  The lanes switched on afterwards would miss them.  (ROCm 7.2's
    compiler once put a pointer's spill there; the other lanes then read from
    wherever their register pointed.)"""
    found, fn, block, regions, scalar = [], None, None, [_Region()], {}
    for line in text.splitlines():
        label = re.match(r"([A-Za-z_]\w*|\.L\w+):|; (%bb\.\d+):", line)
        if label:
            name = label[1] or label[2]
            if not name.startswith((".L", "%")):
                fn = name
            block, regions, scalar = name, [_Region()], {}
            continue
        ins = " ".join(line.split(";")[0].split())
        if not ins or ins.startswith("."):
            continue
        op, _, args = ins.partition(" ")
        # exec = a register just made by an AND (with the lanes running) leaves fewer
        m = re.match(r"s_mov_b64 exec, (\S+)", ins)
        if _NARROW.match(ins) or (m and scalar.get(m[1]) == "s_and_b64"):
            regions.append(_Region())
        elif _WIDEN.match(ins):
            r = regions[-1]
            found += [(fn, block, i) for i in r.spills.values()]
            found += [(fn, block, i) for _, i in r.reloads.values()]
            if len(regions) > 1:
                regions.pop()
                regions[-1].written |= r.written
            else:
                r.spills, r.reloads = {}, {}
            if op.startswith("s_andn2_saveexec"):
                regions.append(_Region())
        else:
            regions[-1].add(ins)
        if op.startswith("s_"):
            scalar[args.partition(",")[0]] = op
    return found


def _compile(src, extra, verbose):
    """Object file of one source; its kernels' assembly is searched."""
    stem = os.path.splitext(src)[0]
    obj = os.path.join(HERE, "_build", stem + ".o")
    tmp = os.path.join(HERE, "_build", stem + ".tmp")     # a fixed name, which the object may hold
    shutil.rmtree(tmp, ignore_errors=True)
    os.mkdir(tmp)
    try:
        out = os.path.join(tmp, stem + ".o")
        cmd = [HIPCC, "-x", "hip", *flags(), *extra, "-save-temps=obj", "-c", os.path.join(CSRC, src), "-o", out]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        listings = [f for f in os.listdir(tmp) if f.endswith(f"{ARCH}.s")]
        if not listings:
            raise RuntimeError(f"{src}: the compiler left no assembly to search")
        for name in listings:
            with open(os.path.join(tmp, name)) as f:
                bad = misplaced_spills(f.read())
            if bad:
                raise RuntimeError(f"{src}: spills before their lanes are switched on: {bad[:5]}")
        os.replace(out, obj)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return obj


def build(verbose: bool = False, extra=()) -> str:
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            continue
        objs.append(_compile(src, extra, verbose))
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", OUT + ".tmp", *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
