"""The build's check of the distances around MFMAs written as inline asm."""
import pytest

from paper_2311_02103_amd.build import check_mfma_listing, mfma_hazards

MFMA = "v_mfma_f32_16x16x32_f16 a[0:3], v[8:11], v[20:23], a[0:3]"


def hazards(*lines):
    return len(mfma_hazards("\n".join("\t" + l for l in lines)))


def test_an_operand_needs_two_slots():
    assert hazards("v_mov_b32_e32 v9, v0", MFMA) == 1
    assert hazards("v_mov_b32_e32 v9, v0", "s_add_u32 s0, s0, s1", MFMA) == 1
    assert hazards("v_mov_b32_e32 v9, v0", "s_nop 1", MFMA) == 0
    assert hazards("v_mov_b32_e32 v9, v0", "ds_read_b128 v[40:43], v44", "s_add_u32 s0, s0, s1", MFMA) == 0
    assert hazards("v_accvgpr_write_b32 a2, 0", MFMA) == 1
    assert hazards("v_mov_b32_e32 v12, v0", MFMA) == 0


def test_a_result_needs_the_pipe_to_drain():
    assert hazards(MFMA, "v_accvgpr_read_b32 v0, a3") == 1
    assert hazards(MFMA, "s_nop 15", "v_accvgpr_read_b32 v0, a3") == 1
    assert hazards(MFMA, "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v0, a3") == 0
    assert hazards(MFMA, MFMA) == 0
    assert hazards(MFMA, "v_accvgpr_read_b32 v0, a4") == 0


def test_modifiers_hide_no_register():
    assert hazards(MFMA, "ds_write_b128 v60, a[0:3] offset:16") == 1
    assert hazards("v_pk_mul_f16 v9, v0, v1 op_sel_hi:[1,0]", MFMA) == 1
    assert hazards("v_mov_b32_e32 v9, v0", "v_mfma_f32_16x16x32_f16 a[0:3], v[8:11], v[20:23], a[0:3] cbsz:1") == 1


def test_every_path_counts():
    loop = ["s_nop 15", "s_nop 15", ".LBB0_1:", MFMA, "s_nop 15", "s_nop 15", "%s", "s_cbranch_scc0 .LBB0_1", "s_endpgm"]
    assert hazards(*[l % "v_mov_b32_e32 v9, v0" if "%" in l else l for l in loop]) == 1            # the loop's end, then its first MFMA
    assert hazards(*[l % "v_mov_b32_e32 v40, v0" if "%" in l else l for l in loop]) == 0
    assert hazards(MFMA, "s_cbranch_scc1 .LBB0_2", "s_nop 15", "s_nop 15", ".LBB0_2:", "v_accvgpr_read_b32 v0, a3") == 1
    assert hazards(MFMA, "s_endpgm", "v_accvgpr_read_b32 v0, a3") == 0                             # the next kernel of the listing
    assert hazards(MFMA, "s_branch .LBB0_3", "v_accvgpr_read_b32 v0, a3", ".LBB0_3:", "s_nop 15", "s_nop 15") == 0


def test_a_listing_is_refused():
    clean = "\n".join(["\ts_nop 15", ".LBB0_1:", "\t" + MFMA, "\ts_nop 15", "\ts_cbranch_scc0 .LBB0_1"])
    check_mfma_listing("x.hip", clean + "\n\tscratch_load_dword v0, off, off")                     # behind the loop
    with pytest.raises(RuntimeError, match="no MFMA"):
        check_mfma_listing("x.hip", "\ts_nop 0")
    with pytest.raises(RuntimeError, match="too close"):
        check_mfma_listing("x.hip", clean + "\n\tv_accvgpr_read_b32 v0, a3")
    with pytest.raises(RuntimeError, match="scratch"):
        check_mfma_listing("x.hip", clean.replace("\ts_cbranch", "\tscratch_load_dword v60, off, off offset:4\n\ts_cbranch"))
