"""The build's check of the distances around MFMAs written as inline asm."""
from paper_2311_02103_amd.build import mfma_hazards

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
