"""The static check that build() runs on the generated gfx950 code: its logic on small hand-written listings, and
the package's own device sources (compiled to ISA text here: no GPU is needed)."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2408_01803_amd import build as stb_build
from paper_2408_01803_amd import isa_check

CLOSE = """
kernel:
\tv_readlane_b32 s5, v203, 3
\tv_add_u32_e32 v1, v2, v3
\tglobal_load_dword v4, v1, s[4:5]
\ts_endpgm
"""

PADDED = """
kernel:
\tv_readlane_b32 s5, v203, 3
\ts_nop 4
\tglobal_load_dword v4, v1, s[4:5]
\ts_endpgm
"""

OTHER_REGISTER = """
kernel:
\tv_readlane_b32 s7, v203, 3
\tglobal_load_dword v4, v1, s[4:5]
\ts_endpgm
"""

ACROSS_A_BRANCH = """
kernel:
\ts_cbranch_scc1 .LBB0_2
\tv_readfirstlane_b32 s4, v9
\ts_branch .LBB0_3
.LBB0_2:
\ts_nop 7
.LBB0_3:
\tglobal_load_dwordx2 v[4:5], v1, s[4:5] offset:512
\ts_endpgm
"""

SCALAR_ALU_WRITE = """
kernel:
\ts_add_u32 s4, s4, s8
\tglobal_load_dword v4, v1, s[4:5]
\ts_endpgm
"""

CARRY_OUT = """
kernel:
\tv_add_co_u32_e64 v1, s[4:5], v2, v3
\tv_mov_b32_e32 v7, 0
\tglobal_load_dword v4, v1, s[4:5]
\ts_endpgm
"""


def test_a_lane_read_right_in_front_of_the_load_is_found():
    found = isa_check.hazards(CLOSE)
    assert len(found) == 1 and found[0][1].startswith("v_readlane_b32 s5") and found[0][4] == 1


def test_five_wait_states_clear_it():
    assert isa_check.hazards(PADDED) == []


def test_a_write_of_another_scalar_is_no_finding():
    assert isa_check.hazards(OTHER_REGISTER) == []


def test_every_path_to_the_load_is_walked():
    found = isa_check.hazards(ACROSS_A_BRANCH)
    assert len(found) == 1 and found[0][1].startswith("v_readfirstlane_b32 s4")


def test_scalar_alu_writes_are_interlocked_and_not_reported():
    assert isa_check.hazards(SCALAR_ALU_WRITE) == []


def test_carry_outputs_count_as_vector_alu_writes():
    assert len(isa_check.hazards(CARRY_OUT)) == 1


SPILL_OF_A_LOAD_IN_FLIGHT = """
kernel:
\t;;#ASMSTART
\tglobal_load_dwordx2 v[10:11], v1, s[4:5]
\t;;#ASMEND
\tv_add_u32_e32 v2, v3, v4
\tscratch_store_dword off, v11, off offset:4 ; 4-byte Folded Spill
\t;;#ASMSTART
\ts_waitcnt vmcnt(0)
\t;;#ASMEND
\ts_endpgm
"""

SPILL_OF_A_COMPUTED_VALUE = """
kernel:
\t;;#ASMSTART
\tglobal_load_dwordx2 v[10:11], v1, s[4:5]
\t;;#ASMEND
\t;;#ASMSTART
\ts_waitcnt vmcnt(0)
\t;;#ASMEND
\tv_add_u32_e32 v11, v10, v11
\tscratch_store_dword off, v11, off offset:4 ; 4-byte Folded Spill
\ts_endpgm
"""


def test_a_spill_of_a_register_that_an_asm_load_has_just_written_is_found():
    assert isa_check.spilled_asm_kernels(SPILL_OF_A_LOAD_IN_FLIGHT) == [("kernel", [11])]


def test_a_spill_of_a_value_computed_after_the_wait_is_no_finding():
    assert isa_check.spilled_asm_kernels(SPILL_OF_A_COMPUTED_VALUE) == []


COPY_OF_A_LOAD_IN_FLIGHT = """
kernel:
\t;;#ASMSTART
\tglobal_load_dwordx2 v[10:11], v1, s[4:5]
\t;;#ASMEND
\tv_add_u32_e32 v2, v3, v4
\tv_mov_b32_e32 v20, v11
\t;;#ASMSTART
\ts_waitcnt vmcnt(0)
\t;;#ASMEND
\ts_endpgm
"""

COPIES_THAT_ARE_FINE = """
kernel:
\t;;#ASMSTART
\tglobal_load_dwordx2 v[10:11], v1, s[4:5]
\t;;#ASMEND
\tv_mov_b32_e32 v20, v12
\t;;#ASMSTART
\ts_waitcnt vmcnt(0)
\t;;#ASMEND
\tv_mov_b32_e32 v20, v11
\tglobal_load_dword v13, v1, s[4:5]
\ts_endpgm
other:
\tv_accvgpr_write_b32 a0, v13
\ts_endpgm
"""


def test_a_move_of_a_register_that_an_asm_load_still_writes_is_found():
    assert isa_check.copied_asm_kernels(COPY_OF_A_LOAD_IN_FLIGHT) == [("kernel", [11])]


def test_moves_of_other_registers_and_after_the_wait_are_no_finding():
    assert isa_check.copied_asm_kernels(COPIES_THAT_ARE_FINE) == []


def _asm(text):
    return f"\t;;#ASMSTART\n\t{text}\n\t;;#ASMEND\n"


MATRIX = _asm("v_smfmac_f32_16x16x64_f16 a[0:3], v[4:7], v[8:15], v16")


@pytest.mark.parametrize("before,found", [
    ("v_mov_b32_e32 v16, v20\n", True), ("v_mov_b32_e32 v16, v20\n\ts_nop 0\n", True), ("v_mov_b32_e32 v16, v20\n\ts_nop 1\n", False),
    ("v_add_u32_e32 v8, v1, v2\n", True), ("v_accvgpr_write_b32 a2, 0\n", True), ("v_add_u32_e32 v17, v4, v5\n", False),
    ("ds_read_b128 v[4:7], v1\n\ts_waitcnt lgkmcnt(0)\n", False),                         # (waited for, as the compiler does)
    ("s_cbranch_scc1 .LBB0_1\n\tv_mov_b32_e32 v4, 0\n.LBB0_1:\n", True)])
def test_vector_writes_right_ahead_of_a_matrix_instruction_in_an_asm_statement(before, found):
    got = isa_check.asm_matrix_hazards("kernel:\n\t" + before + MATRIX + "\ts_endpgm\n")
    assert len(got) == found, got
    # the compiler pads the matrix instructions that it sees
    assert isa_check.asm_matrix_hazards("kernel:\n\t" + before + MATRIX.split("\n")[1] + "\n\ts_endpgm\n") == []


@pytest.mark.parametrize("behind,found", [
    ("\tv_accvgpr_read_b32 v1, a3\n", True), ("\ts_nop 15\n\tv_accvgpr_read_b32 v1, a3\n", True), ("\ts_nop 15\n\ts_nop 15\n\tv_accvgpr_read_b32 v1, a3\n", False),
    ("\tv_accvgpr_read_b32 v1, a4\n", False), ("\tv_accvgpr_write_b32 a0, 0\n", True), ("\tglobal_store_dwordx4 v1, a[0:3], s[4:5]\n", True),
    (MATRIX, False),                                                                         # adds to the same registers again
    (_asm("v_smfmac_f32_16x16x64_f16 a[2:5], v[4:7], v[8:15], v16"), True), (_asm("v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]"), True),
    (_asm("v_smfmac_f32_16x16x64_f16 a[0:3], a[0:3], v[8:15], v16"), True)])
def test_results_of_a_matrix_instruction_in_an_asm_statement_that_are_touched_too_early(behind, found):
    got = isa_check.asm_matrix_hazards("kernel:\n" + MATRIX + behind + "\ts_endpgm\n")
    assert (len(got) > 0) == found, got


def test_a_loop_back_to_another_kind_of_matrix_instruction_is_followed():
    other = _asm("v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]")
    assert len(isa_check.asm_matrix_hazards("kernel:\n.LBB0_1:\n" + other + "\ts_nop 15\n\ts_nop 15\n" + MATRIX + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n")) == 1


@pytest.mark.parametrize("store,behind,found", [
    ("global_store_dwordx4 v[0:1], v[4:7], off sc1", "\tv_mov_b32_e32 v6, 0\n", True), ("global_store_dwordx4 v[0:1], v[4:7], off sc1", "\tv_mov_b32_e32 v0, 0\n", False),
    ("global_store_dwordx4 v[0:1], v[4:7], off sc1\n\ts_nop 1", "\tv_mov_b32_e32 v6, 0\n", False), ("global_store_dwordx2 v[0:1], v[4:5], off", "\tv_mov_b32_e32 v4, 0\n", False),
    ("buffer_store_dwordx4 v[4:7], v0, s[0:3], 0 offen", "\ts_nop 0\n\tv_add_u32_e32 v7, v1, v2\n", True)])
def test_data_of_a_wide_store_in_an_asm_statement_that_is_overwritten_right_behind_it(store, behind, found):
    assert len(isa_check.asm_matrix_hazards("kernel:\n" + _asm(store) + behind + "\ts_endpgm\n")) == found


def test_the_device_sources_of_the_package_are_clean(tmp_path):
    inc = ["-I" + os.path.join(stb_build.ROOT, "include"), "-I" + stb_build.CSRC]
    srcs = [os.path.join(stb_build.CSRC, s) for s in stb_build.DEVICE_SOURCES]
    with ThreadPoolExecutor(max_workers=len(srcs)) as pool:
        found = list(pool.map(lambda s: isa_check.check_source(s, str(tmp_path), stb_build.HIPCC, [*stb_build.DEVICE_FLAGS, *inc]), srcs))
    assert all(f == [] for f in found), [f[:3] for f in found if f]


def test_the_kernels_of_the_packer_keep_their_values_in_registers(tmp_path):
    """None of them has scratch memory: an occupancy bound that one ratio's assignment kernel does not fit shows here."""
    text = isa_check.compile_to_isa(os.path.join(stb_build.CSRC, "stb_pack.hip"), str(tmp_path / "pack.s"), stb_build.HIPCC,
                                    [*stb_build.DEVICE_FLAGS, "-I" + os.path.join(stb_build.ROOT, "include"), "-I" + stb_build.CSRC])
    sizes = {name: int(size) for name, size in re.findall(r"^\s*\.name:\s*(_Z\S*)\n\s*\.private_segment_fixed_size:\s*(\d+)", text, re.M)}
    assert any("k_assign" in name for name in sizes)
    assert {name: size for name, size in sizes.items() if size} == {}
