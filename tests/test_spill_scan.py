"""build.misplaced_spills on short listings: joins of every form, with and
without instructions between the start of the block and the spill, and the
spills that belong to the lanes running; and the build, which fails on one."""
import os

import pytest

from paper_2111_08744_amd import build

JOINS = ["s_or_b64 exec, exec, s[2:3]", "s_or_saveexec_b64 s[4:5], s[2:3]", "s_andn2_saveexec_b64 s[2:3], s[2:3]",
         "s_mov_b64 exec, s[2:3]"]
MISPLACED = ["v_accvgpr_write_b32 a8, v156", "scratch_store_dword off, v156, off offset:4",
             "scratch_store_dwordx2 off, v[156:157], off", "v_accvgpr_read_b32 v156, a8",
             "scratch_load_dword v156, off, off offset:4"]


def _listing(start, *ins):
    return "_Zk:\n\tv_mov_b32_e32 v156, v0\n" + start + "\n" + "".join(f"\t{i}\n" for i in ins) + ".Lfunc_end0:\n"


@pytest.mark.parametrize("start", [".LBB0_1:                                ; %if.end", "; %bb.7:                 ; join"])
@pytest.mark.parametrize("join", JOINS)
@pytest.mark.parametrize("spill", MISPLACED)
@pytest.mark.parametrize("before", [[], ["s_mov_b32 s9, 0"], ["v_mov_b32_e32 v7, v8"], ["s_waitcnt vmcnt(0)"],
                                    ["s_and_saveexec_b64 s[6:7], vcc", "v_mov_b32_e32 v7, v8",
                                     "s_or_b64 exec, exec, s[6:7]"]])
def test_misplaced(start, join, spill, before):
    found = build.misplaced_spills(_listing(start, *before, spill, join))
    assert [f[2] for f in found] == [spill] and found[0][0] == "_Zk"


@pytest.mark.parametrize("ins", [
    ["s_or_b64 exec, exec, s[2:3]", "v_accvgpr_write_b32 a8, v156"],                    # after the join
    ["v_add_u32_e32 v156, 1, v3", "v_accvgpr_write_b32 a8, v156", JOINS[0]],            # the block's own value
    ["v_accvgpr_write_b32 a8, v156", "v_mov_b32_e32 v156, v2", "v_accvgpr_read_b32 v156, a8",
     "v_add_u32_e32 v1, v156, v1", JOINS[0]],                                           # back before the join
    ["scratch_load_dword v9, off, off", "v_add_u32_e32 v1, v9, v1", JOINS[0]],          # read before it
    ["scratch_load_dword v9, off, off", "global_store_dword v[2:3], v9, off", JOINS[0]],
    ["s_and_b64 s[2:3], s[4:5], vcc", "v_accvgpr_write_b32 a8, v156", "s_mov_b64 exec, s[2:3]"],   # fewer lanes
    ["v_accvgpr_write_b32 a8, v156", "s_and_saveexec_b64 s[6:7], vcc", "v_mov_b32_e32 v7, v8",
     "s_or_b64 exec, exec, s[6:7]"],                                                    # before the branch
    ["s_or_saveexec_b64 s[4:5], s[2:3]", "v_accvgpr_write_b32 a8, v156", "s_xor_b64 exec, exec, s[4:5]"],
])
def test_in_place(ins):
    assert build.misplaced_spills(_listing(".LBB0_1:", *ins)) == []


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not found")
def test_build_fails_on_a_misplaced_spill(tmp_path, monkeypatch):
    csrc = tmp_path / "csrc"
    csrc.mkdir()
    (tmp_path / "_build").mkdir()
    (csrc / "k.hip").write_text("#include <hip/hip_runtime.h>\n__global__ void k(float* p) { *p = 1.0f; }\n")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CSRC", str(csrc))
    obj = build._compile("k.hip", (), False)
    assert os.path.getsize(obj) > 0 and os.listdir(tmp_path / "_build") == ["k.o"]
    os.remove(obj)
    seen = []
    monkeypatch.setattr(build, "misplaced_spills", lambda text: seen.append(text) or [("k", ".LBB0_1", "spill")])
    with pytest.raises(RuntimeError, match="before their lanes"):
        build._compile("k.hip", (), False)
    assert "_Z1kPf:" in seen[0] and not os.path.exists(obj)
