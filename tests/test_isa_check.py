"""The compiled matrix-core kernels are scanned for results of matrix instructions that are read
too early on the far side of a branch (a case the compiler's own padding has missed; see
tests/isa_check.py).  CPU only: hipcc cross-compiles to assembly."""
from tests import isa_check

PLANTED = """
.LBB0_1:
	v_mfma_f32_32x32x16_bf16 a[64:79], v[72:75], v[112:115], a[64:79]
	s_cbranch_vccnz .LBB0_3
	v_add_u32_e32 v68, s57, v162
	v_ashrrev_i32_e32 v69, 31, v68
	v_and_b32_e32 v69, s16, v69
	v_add_u32_e32 v68, v68, v69
	v_cmp_ge_i32_e64 s[6:7], s21, v68
	v_mov_b32_e32 v1, 0
	v_mov_b32_e32 v2, 0
	v_mov_b32_e32 v3, 0
	v_mov_b32_e32 v4, 0
.LBB0_3:
	s_nop 1
	v_accvgpr_read_b32 v83, a79
	s_endpgm
"""

STRAIGHT = """
	v_mfma_f32_32x32x16_bf16 a[64:79], v[72:75], v[112:115], a[64:79]
	s_nop 11
	v_accvgpr_read_b32 v83, a79
	v_mfma_f32_32x32x16_bf16 a[0:15], v[72:75], v[112:115], a[0:15]
	v_mfma_f32_32x32x16_bf16 a[0:15], v[76:79], v[116:119], a[0:15]
	s_cbranch_scc1 .LBB0_9
	s_nop 15
.LBB0_9:
	s_nop 15
	v_accvgpr_read_b32 v1, a0
	s_endpgm
"""


def test_scanner_finds_a_result_read_too_early_across_a_branch():
    hits = isa_check.scan(PLANTED)
    assert len(hits) == 1
    mfma, reader, wait_states = hits[0]
    assert reader.startswith("v_accvgpr_read_b32 v83, a79") and wait_states == 3


INLINE_ASM = """
	v_mfma_f32_32x32x16_bf16 v[210:225], v[14:17], v[226:229], 0
	v_fma_f32 v16, s3, v210, v0
	s_endpgm
"""


def test_scanner_checks_vgpr_results_on_straight_paths_too():
    """A result tile in VGPRs comes from the kernels' inline assembly, which the compiler never pads."""
    hits = isa_check.scan(INLINE_ASM)
    assert len(hits) == 1 and hits[0][2] == 0


SRC_C = """
	v_mfma_f32_32x32x16_bf16 v[210:225], v[14:17], v[226:229], 0
	v_mfma_f32_32x32x16_bf16 v[100:115], v[14:17], v[226:229], v[210:225]
	s_endpgm
"""

RESTART = """
	v_mfma_f32_32x32x16_bf16 v[210:225], v[14:17], v[226:229], 0
	v_mfma_f32_32x32x16_bf16 v[210:225], v[18:21], v[230:233], 0
	s_endpgm
"""

DEEP = "\n\tv_mfma_f32_32x32x16_bf16 v[210:225], v[14:17], v[226:229], 0\n" + "".join(
    f"\ts_cbranch_scc1 .LBB0_{i}\n.LBB0_{i}:\n" for i in range(1, 9)) + "\tv_mov_b32_e32 v1, v210\n\ts_endpgm\n"


def test_scanner_counts_srcc_and_overlapping_destinations_of_other_matrix_instructions():
    """Another matrix instruction reads the tile as SrcC into a different destination, or restarts the
    same destination from zero: neither is the interlocked accumulation form."""
    assert len(isa_check.scan(SRC_C)) == 1
    assert len(isa_check.scan(RESTART)) == 1


def test_scanner_reports_the_branch_depth_limit():
    """Eight nested branches inside the hazard window: the walk gives up at depth 6 and must say so."""
    hits = isa_check.scan(DEEP)
    assert len(hits) == 1 and hits[0][1] == isa_check.DEPTH_LIMIT and hits[0][2] < isa_check.WAIT_STATES


def test_scanner_accepts_padded_code_and_accumulation_chains():
    assert isa_check.scan(STRAIGHT) == []


def test_compiled_kernels_are_clean():
    for src, hits in isa_check.check_all().items():
        assert not hits, (src, hits)


LOOPS = """
_Z6kernelv:
	scratch_store_dword off, v2, off
.LBB0_1:                                ; =>This Loop Header: Depth=1
                                        ;     Child Loop BB0_2 Depth 2
	scratch_load_dword v2, off, off
.LBB0_2:                                ;   Parent Loop BB0_1 Depth=1
                                        ; =>  This Inner Loop Header: Depth=2
	v_mfma_f32_16x16x4_f32 v[0:3], v4, v5, v[0:3]
	s_cbranch_vccnz .LBB0_4
; %bb.3:                                ;   in Loop: Header=BB0_2 Depth=2
	scratch_load_dword v6, off, off
.LBB0_4:                                ;   in Loop: Header=BB0_2 Depth=2
	s_cbranch_scc1 .LBB0_2
; %bb.5:                                ;   in Loop: Header=BB0_1 Depth=1
	scratch_load_dword v7, off, off
	s_endpgm
"""


def test_spills_are_counted_in_the_innermost_matrix_loop_only():
    assert isa_check.loop_spills(LOOPS) == {("_Z6kernelv", "BB0_2"): 1}


def test_fp32_matrix_loops_hold_no_spills():
    """The D = 128 dK/dV kernel once fetched four addresses from scratch on every row tile, behind its loads."""
    found = isa_check.loop_spills(isa_check.assembly("attn_fp32.hip"))
    assert len(found) >= 10      # forward and dQ in two tile widths, dK/dV, both head sizes
    assert not any(found.values()), found


FP32 = """
	v_mfma_f32_16x16x4_f32 v[8:11], v4, v5, v[8:11]
	v_mov_b32_e32 v1, 0
	s_cbranch_vccnz .LBB0_2
	s_nop 15
.LBB0_2:
	s_nop %d
	v_mul_f32_e32 v2, v3, v9
	s_endpgm
"""


def test_scanner_knows_the_fp32_instruction():
    """Two instructions and the branch, then 7 or 6 of s_nop: 10 wait states are enough, 9 are not; what the compiler
    schedules on a straight path is left to it where there is no inline assembly."""
    assert isa_check.scan(FP32 % 7, inline_asm=False) == []
    hits = isa_check.scan(FP32 % 6, inline_asm=False)
    assert len(hits) == 1 and hits[0][2] == 9
    straight = "\n\tv_mfma_f32_16x16x4_f32 v[8:11], v4, v5, v[8:11]\n\tv_mul_f32_e32 v2, v3, v9\n\ts_endpgm\n"
    assert isa_check.scan(straight, inline_asm=False) == [] and len(isa_check.scan(straight)) == 1


def test_every_source_with_matrix_instructions_is_scanned():
    import os
    import re
    for f in os.listdir(isa_check.CSRC):
        if f.endswith(".hip") and re.search(r"mfma32\w*\(|__builtin_amdgcn_mfma", open(os.path.join(isa_check.CSRC, f)).read()):
            assert f in isa_check.KERNEL_SOURCES, f
