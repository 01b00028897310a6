"""The build's check of the kernels' assembly: no vector write under a branch's
lane mask after the branch has been left."""
import pytest

from paper_2006_15122_amd.build_lib import masked_join_writes

JOIN = """
_Z4passv:                               ; @_Z4passv
; %bb.0:
	v_cmp_gt_u32_e32 vcc, 4, v0
	s_and_saveexec_b64 s[76:77], vcc
	s_cbranch_execz .LBB0_2
; %bb.1:
	v_add_f64 v[90:91], v[100:101], v[116:117]
	ds_write_b128 v98, v[90:93]
.LBB0_2:                                ; %Flow
{copies}	s_or_b64 exec, exec, s[76:77]
	v_accvgpr_read_b32 v189, a3
	s_endpgm
.Lfunc_end0:
"""

OUT_OF_LINE = """
_Z4passv:
; %bb.0:
	s_and_saveexec_b64 s[0:1], vcc
	s_cbranch_execnz .LBB0_3
{join}
{copies}	s_or_b64 exec, exec, s[0:1]
	s_endpgm
.LBB0_3:
	v_add_u32_e32 v1, 1, v1
	s_branch .LBB0_1
.Lfunc_end0:
"""


@pytest.mark.parametrize("copy", ["v_accvgpr_write_b32 a3, v189", "v_mov_b32_e32 v119, v188",
                                  "v_mov_b32_e32 v239, 0x3ff00000",
                                  "v_cmp_lt_u32_e64 s[8:9], 33, v0", "ds_read_b64 v[2:3], v1"])
def test_a_copy_ahead_of_the_restored_mask_is_found(copy):
    got = masked_join_writes(JOIN.format(copies=f"\t{copy}\n"))
    assert got == [("_Z4passv", ".LBB0_2", [copy])]
    for join in (".LBB0_1:", "; %bb.1:"):
        got = masked_join_writes(OUT_OF_LINE.format(join=join, copies=f"\t{copy}\n"))
        assert [(k, c) for k, _, c in got] == [("_Z4passv", [copy])]


@pytest.mark.parametrize("ahead", ["", "\ts_mov_b32 s0, 4\n", "\tv_readlane_b32 s4, v255, 4\n",
                                   "\tv_writelane_b32 v255, s4, 4\n", "\ts_waitcnt lgkmcnt(0)\n"])
def test_a_mask_restored_first_passes(ahead):
    assert masked_join_writes(JOIN.format(copies=ahead)) == []
    assert masked_join_writes(OUT_OF_LINE.format(join=".LBB0_1:", copies=ahead)) == []


@pytest.mark.parametrize("turn", ["s_andn2_saveexec_b64 s[76:77], s[76:77]", "s_or_saveexec_b64 s[76:77], s[76:77]"])
def test_a_copy_ahead_of_an_else_is_found(turn):
    copy = "v_mov_b32_e32 v119, v188"
    asm = JOIN.replace("s_or_b64 exec, exec, s[76:77]", turn)
    assert masked_join_writes(asm.format(copies=f"\t{copy}\n")) == [("_Z4passv", ".LBB0_2", [copy])]
    assert masked_join_writes(asm.format(copies="")) == []


def test_a_body_that_ends_in_its_own_join_passes():
    # an if's body, entered with lanes: its writes are under the mask by right
    asm = JOIN.format(copies="\tv_mov_b32_e32 v119, v188\n")
    assert masked_join_writes(asm.replace("s_cbranch_execz .LBB0_2", "s_cbranch_execz .LBB0_9")) == []
