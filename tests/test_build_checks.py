"""The build's check of the wait states around inline matrix and DPP instructions, on small pieces of assembly."""
import pytest

from paper_2604_24971_amd import build

MFMA = "v_mfma_f32_32x32x16_f16 v[0:15], v[20:23], a[0:3], 0"
FMAC = "v_fmac_f32_dpp v40, v30, v70 row_newbcast:1 row_mask:0xf bank_mask:0xf"


def _check(tmp_path, *lines):
    path = tmp_path / "kernel.s"
    path.write_text("\n".join(["\t.text", "_Z6kernelv:", *("%s%s" % ("" if l.endswith(":") else "\t", l) for l in lines),
                               "\ts_endpgm", ""]))
    return build._check_wait_states(str(path))


def test_distances_that_are_kept(tmp_path):
    assert _check(tmp_path, "v_mov_b32_e32 v20, v50", "s_nop 1", MFMA, "s_nop 11", "v_add_f32_e32 v60, v0, v1") == 1
    assert _check(tmp_path, "v_mov_b32_e32 v30, v50", "s_nop 1", FMAC, MFMA) == 1
    # a loop whose end is far enough from its head, and code behind an unconditional branch
    assert _check(tmp_path, ".LBB0_1:", MFMA, "s_nop 15", "v_mov_b32_e32 v20, v50", "s_nop 0", "s_cbranch_scc1 .LBB0_1") == 1
    assert _check(tmp_path, MFMA, "s_branch .LBB0_2", "v_add_f32_e32 v60, v0, v1", ".LBB0_2:", "s_nop 12", "v_add_f32_e32 v60, v0, v1") == 1


@pytest.mark.parametrize("lines,what", [
    (("v_mov_b32_e32 v21, v50", "s_nop 0", MFMA), "operand written"),
    ((MFMA, "s_nop 10", "v_add_f32_e32 v60, v0, v1"), "accessed too early"),
    ((MFMA, "s_nop 3", "v_mfma_f32_32x32x16_f16 a[16:31], v[0:3], a[0:3], 0"), "read too early"),
    ((MFMA, "v_mov_b32_e32 v30, v50", "s_nop 0", FMAC), "DPP source"),
    ((MFMA, "v_mov_b32_e32 v30, v50", FMAC), "DPP source"),
    # across a branch back to the head of a loop, one forward, and one behind another
    ((".LBB0_1:", MFMA, "s_nop 15", "v_mov_b32_e32 v20, v50", "s_cbranch_scc1 .LBB0_1"), "operand written"),
    ((".LBB0_1:", FMAC, MFMA, "s_nop 15", "v_mov_b32_e32 v30, v50", "s_cbranch_vccnz .LBB0_1"), "DPP source"),
    ((MFMA, "s_cbranch_scc0 .LBB0_3", "s_nop 15", ".LBB0_3:", "v_add_f32_e32 v60, v0, v1"), "accessed too early"),
    ((MFMA, "s_branch .LBB0_3", ".LBB0_4:", "v_add_f32_e32 v60, v0, v1", ".LBB0_3:", "s_branch .LBB0_4"), "accessed too early"),
    (("v_add_f32_e32 v60, v0, v1",), "no matrix instruction"),
])
def test_distances_that_are_too_short(tmp_path, lines, what):
    with pytest.raises(RuntimeError, match=what):
        _check(tmp_path, *lines)
