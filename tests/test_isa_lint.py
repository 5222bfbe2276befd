"""The compiled kernels hold no matrix instruction inside an execution-mask region that the compiler left
without a skip branch (MFMA ignores EXEC: such an instruction runs although its source-level condition is
false).  This is the cause of a wrong result the streaming GEMM once gave for one launch shape: the MFMAs of
register slots past a wavefront's K share ran with an empty mask and added the last weight tile again."""
import pytest

from paper_2603_25702_amd import isa_lint

BAD = """
_Z6kernelv:
	v_cmp_lt_i32_e32 vcc, v18, v66
	s_and_saveexec_b64 s[20:21], vcc
; %bb.12:
	v_mfma_f32_16x16x32_bf16 v[54:57], v[6:9], v[46:49], v[54:57]
	s_or_b64 exec, exec, s[20:21]
	v_mfma_f32_16x16x32_bf16 v[54:57], v[6:9], v[46:49], v[54:57]
	s_endpgm
"""
GOOD = """
_Z6kernelv:
	v_cmp_lt_i32_e32 vcc, v18, v66
	s_and_saveexec_b64 s[20:21], vcc
	s_cbranch_execz .LBB0_2
; %bb.12:
	v_mfma_f32_16x16x32_bf16 v[54:57], v[6:9], v[46:49], v[54:57]
.LBB0_2:
	s_or_b64 exec, exec, s[20:21]
	s_cmp_ge_i32 s14, s12
	s_cbranch_scc1 .LBB0_3
	v_mfma_f32_16x16x32_bf16 v[54:57], v[6:9], v[46:49], v[54:57]
.LBB0_3:
	s_endpgm
"""


def test_scanner_flags_an_mfma_in_a_mask_region_without_a_skip_branch():
    found = isa_lint.scan_asm(BAD)
    assert [(k, no) for k, no, _ in found] == [("_Z6kernelv", 6)]
    assert isa_lint.scan_asm(GOOD) == []


EARLY = """
_Z6kernelv:
	;;#ASMSTART
	v_mfma_f32_16x16x32_f16 a[4:7], v[6:9], v[46:49], a[4:7]
	v_mfma_f32_16x16x32_f16 a[8:11], v[6:9], v[46:49], a[8:11]
	;;#ASMEND
	s_nop 7
	v_accvgpr_read_b32 v0, a4
	v_accvgpr_read_b32 v1, a9
	s_nop 7
	v_accvgpr_read_b32 v1, a9
	s_endpgm
"""


def test_scanner_flags_a_result_that_is_read_before_it_is_there():
    found = isa_lint.scan_agpr_reads(EARLY)
    assert [no for _, no, _ in found] == [8, 9]   # 9 and 9 wait states


@pytest.mark.parametrize("touch,found", [
    ("global_store_dwordx4 v[0:1], a[4:7], off", 1),
    ("buffer_store_dword a7, v1, s[0:3], 0 offen", 1),
    ("scratch_store_dword off, a6, off offset:16", 1),          # a spill
    ("ds_write2_b64 v2, a[6:7], a[10:11] offset1:8", 1),        # two of one range
    ("v_accvgpr_write_b32 a5, 0", 1),                           # another value
    ("v_mfma_f32_16x16x32_f16 a[12:15], a[4:7], v[2:5], a[12:15]", 1),
    ("v_mfma_f32_16x16x32_f16 a[4:7], v[6:9], v[46:49], a[4:7]", 0),
    ("global_store_dwordx4 v[0:1], a[8:11], off", 0),
    ("s_nop 10\n\tglobal_store_dwordx4 v[0:1], a[4:7], off", 0),
    ("s_nop 9\n\tglobal_store_dwordx4 v[0:1], a[4:7], off", 1),
])
def test_scanner_knows_what_touches_an_accumulator(touch, found):
    text = f"_Z6kernelv:\n\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_f16 a[4:7], v[6:9], v[46:49], a[4:7]\n\t;;#ASMEND\n\t{touch}\n\ts_endpgm\n"
    assert len(isa_lint.scan_agpr_reads(text)) == found


LOOP = """
_Z6kernelv:
	s_mov_b32 s0, 4
.LBB0_1:
	v_accvgpr_read_b32 v0, a4
	s_nop 7
	;;#ASMSTART
	v_mfma_f32_16x16x32_f16 a[4:7], v[6:9], v[46:49], a[4:7]
	;;#ASMEND
	s_sub_u32 s0, s0, 1
	s_cbranch_scc0 .LBB0_1
	s_branch .LBB0_3
.LBB0_2:
	v_accvgpr_read_b32 v0, a4
.LBB0_3:
	v_accvgpr_read_b32 v0, a5
	s_endpgm
"""


def test_scanner_follows_branches():
    found = isa_lint.scan_agpr_reads(LOOP)
    assert [no for _, no, _ in found] == [5, 16]   # over the loop's back edge, over the jump; nothing jumps to the block between


def test_compiled_kernels_have_no_mfma_under_a_narrowed_execution_mask_and_read_no_result_early():
    found = isa_lint.lint_sources()
    assert not found, "\n".join(f"{s}: {k}: line {no}: {ins}" for s, k, no, ins in found[:20])
