"""The kernels' assembly: where lanes that branched off join the others again,
no register is spilled before the others are switched on.  The compiler once
put a pointer's spill there (to an accumulation register, in the reverse sweep
with four lanes a ray); the other lanes then read from wherever their register
happened to point."""
import os
import re
import subprocess

import pytest

from paper_2111_08744_amd import build

SPILL = ("v_accvgpr_write", "scratch_store")


def early_spills(text):
    """(function, block, instruction) of spills between the start of a block
    and the instruction that switches its lanes on, with nothing else but
    spills and reloads before it."""
    found, fn, block, head = [], None, None, None
    for line in text.splitlines():
        line = line.split(";")[0].rstrip()
        label = re.match(r"^(_Z\S+|\.LBB\S+):", line)
        if label:
            if label[1].startswith("_Z"):
                fn, head = label[1], None
            else:
                block, head = label[1], []
            continue
        op = line.strip()
        if head is None or not op or op.startswith("."):
            continue
        if op.startswith("s_or_b64 exec, exec"):
            found += [(fn, block, h) for h in head]
            head = None
        elif op.startswith(SPILL):
            head.append(op)
        elif not op.startswith(("v_accvgpr_read", "scratch_load", "v_readlane", "v_writelane", "s_nop", "s_waitcnt")):
            head = None
    return found


def test_scan_finds_an_early_spill():
    bad = "_Zk:\n.LBB0_1:\n\tv_accvgpr_write_b32 a8, v156\n\ts_or_b64 exec, exec, s[2:3]\n"
    assert early_spills(bad) == [("_Zk", ".LBB0_1", "v_accvgpr_write_b32 a8, v156")]
    assert early_spills(bad.replace("\tv_acc", "\tv_mul_f32 v1, v2, v3\n\tv_acc")) == []
    good = "_Zk:\n.LBB0_1:\n\ts_or_b64 exec, exec, s[2:3]\n\tv_accvgpr_write_b32 a8, v156\n"
    assert early_spills(good) == []


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not found")
def test_no_spill_before_the_lanes_join(tmp_path):
    jobs = []
    for src in (s for s in build.SOURCES if s.endswith(".hip")):
        out = str(tmp_path / (src + ".s"))
        jobs.append((src, out, subprocess.Popen(
            [build.HIPCC, "-x", "hip", *build.flags(), "-S", "--cuda-device-only", os.path.join(build.CSRC, src),
             "-o", out], stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)))
    for src, out, job in jobs:
        assert job.wait() == 0, src
        with open(out) as f:
            assert early_spills(f.read()) == [], src
