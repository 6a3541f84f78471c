"""Register spills under a partial lane mask: the forms in which a block can restore
or widen the mask, and those that only narrow it (CPU)."""
import pytest

from paper_2112_03851_amd.build import MOVES, masked_spills

SPILL = "scratch_store_dword off, v38, off offset:24"
LINE = f"\t{SPILL} ; 4-byte Folded Spill\n"
OWN = "\tscratch_store_dword off, v38, off offset:24\n"  # (a store of the program's own)


def _asm(head, body):
    return f"\n_Z3foo:\n; %bb.0:\n\ts_mov_b64 s[2:3], exec\n\ts_cbranch_vccnz .LBB0_9\n{head}\n{body}\ts_endpgm\n"


@pytest.mark.parametrize("head", [".LBB0_3:", "; %bb.3:"])
@pytest.mark.parametrize("restore", [
    "s_or_b64 exec, exec, s[2:3]",           # a join whose branch was left out
    "s_or_saveexec_b64 s[4:5], s[4:5]",      # the head of an else
    "s_andn2_saveexec_b64 s[4:5], s[4:5]",   # the same, shorter
    "s_xor_b64 exec, exec, s[4:5]",
    "s_mov_b64 exec, s[2:3]"])               # a mask saved in another block
def test_spill_before_the_mask_widens_is_found(head, restore):
    assert masked_spills(_asm(head, LINE + f"\t{restore}\n")) == [("_Z3foo", SPILL)]
    assert masked_spills(_asm(head, f"\t{restore}\n" + LINE)) == []
    assert masked_spills(_asm(head, OWN + "\tv_add_u32_e32 v1, v2, v3\n" + f"\t{restore}\n")) == []


@pytest.mark.parametrize("narrow", [
    "s_and_saveexec_b64 s[4:5], vcc",
    "s_and_b64 exec, exec, s[4:5]",
    "s_andn2_b64 exec, exec, s[4:5]",
    "s_and_b64 s[6:7], s[2:3], vcc\n\ts_mov_b64 exec, s[6:7]"])
def test_spill_before_the_mask_narrows_is_none(narrow):
    assert masked_spills(_asm(".LBB0_3:", LINE + f"\t{narrow}\n")) == []
    # and what follows in the narrowed region is that region's own
    assert masked_spills(_asm(".LBB0_3:", f"\t{narrow}\n" + LINE + "\ts_or_b64 exec, exec, s[4:5]\n")) == []


def test_a_join_is_reported_once_and_a_copy_stops_the_build():
    join = "\ts_cbranch_execz .LBB0_4\n.LBB0_4:\n" + LINE + "\tv_mov_b32_e32 v1, v2\n\tv_add_u32_e32 v1, v2, v3\n" + \
        "\ts_or_b64 exec, exec, s[2:3]\n"
    found = masked_spills(_asm("; %bb.3:", join))
    assert [t for _, t in found] == [SPILL, "v_mov_b32_e32 v1, v2", "v_add_u32_e32 v1, v2, v3"]
    assert [t.startswith(MOVES) for _, t in found] == [True, True, False]
