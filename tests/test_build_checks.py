"""The build's look through the kernels' assembly."""
import glob
import os

import pytest

from paper_2103_14949_amd import build

KERNEL = """
_Zkern: ; @_Zkern
\tv_lshl_add_u64 v[2:3], v[30:31], 3, s[12:13]
.LBB0_2:
\t{shift}
\ts_endpgm
\t.amdhsa_kernel _Zkern
\t\t.amdhsa_next_free_vgpr {registers}
\t.end_amdhsa_kernel
"""


@pytest.mark.parametrize("shift,registers,refused", [
    ("v_ashrrev_i64 v[16:17], v31, v[16:17]", 32, True),
    ("v_lshlrev_b64 v[4:5], v215, v[132:133]", 209, True),      # registers come in blocks of eight
    ("v_lshrrev_b64_e64 v[4:5], v31, s[2:3]", 25, True),
    ("v_ashrrev_i64 v[16:17], v31, v[16:17]", 33, False),       # another block follows
    ("v_ashrrev_i64 v[16:17], v30, v[30:31]", 32, False),
    ("v_ashrrev_i64 v[30:31], s31, v[30:31]", 32, False),
    ("v_lshlrev_b32_e32 v16, v31, v16", 32, False),
])
def test_shift_amounts_in_the_last_register_are_found(shift, registers, refused):
    found = build.check_shift_amounts(KERNEL.format(shift=shift, registers=registers))
    assert bool(found) == refused
    if refused:
        assert "_Zkern" in found[0] and shift in found[0]


@pytest.mark.parametrize("lines,refused", [
    ("s_mov_b32 m0, s4|buffer_load_dwordx4 v1, s[8:11], 0 offen lds", True),
    ("s_add_u32 m0, m0, s4|; a comment|buffer_load_dword v1, s[8:11], s2 offen offset:16 lds", True),
    ("s_mov_b32 m0, s4|s_nop 0|buffer_load_dwordx4 v1, s[8:11], 0 offen lds", False),
    ("s_mov_b32 m0, s4|v_xor_b32 v1, s4, v1|buffer_load_dwordx4 v1, s[8:11], 0 offen lds", False),
    ("s_mov_b32 m0, s4|buffer_load_dwordx4 v[4:7], v1, s[8:11], 0 offen", False),
    ("s_mov_b32 s3, s4|buffer_load_dwordx4 v1, s[8:11], 0 offen lds", False),
])
def test_lds_loads_directly_after_m0_are_found(lines, refused):
    assembly = "_Zkern:\n" + "".join(f"\t{x}\n" for x in lines.split("|"))
    assert bool(build.check_lds_loads(assembly)) == refused
    assert bool(build.check_assembly(assembly)) == refused


@pytest.mark.parametrize("lines,refused", [
    ("global_store_dwordx4 v[4:5], v[0:3], off sc1", True),
    ("global_store_dwordx4 v[4:5], v[0:3], off sc1|s_nop 0", True),
    ("buffer_store_dwordx3 v[0:2], v4, s[0:3], 0 offen|v_mov_b32 v0, 0", True),
    ("global_store_dwordx4 v[4:5], v[0:3], off sc1|s_nop 1", False),
    ("global_store_dwordx2 v[4:5], v[0:1], off sc1", False),
])
def test_wide_stores_without_wait_states_behind_them_are_found(lines, refused):
    body = "".join(f"\t{x}\n" for x in lines.split("|"))
    assert bool(build.check_wide_stores(f"_Zkern:\n\t;;#ASMSTART\n{body}\t;;#ASMEND\n\tv_mov_b32 v0, 1\n")) == refused
    assert not build.check_wide_stores(f"_Zkern:\n{body}")  # (the compiler's own)


@pytest.mark.parametrize("lines,refused", [
    ("v_permlane16_swap_b32 v1, v2", True),
    ("v_permlane32_swap_b32 v2, v1", True),
    ("s_nop 0|v_permlane16_swap_b32 v1, v2", True),
    ("s_nop 1|v_permlane16_swap_b32 v1, v2", False),
    ("v_xor_b32_e32 v1, v1, v9|v_permlane16_swap_b32 v7, v2|v_permlane16_swap_b32 v1, v2", False),
    ("v_permlane16_swap_b32 v3, v2", False),
    ("v_mov_b32_dpp v3, v1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1", True),
    ("v_add_u32_dpp v3, v[0:1], v4 row_shr:1 row_mask:0xf bank_mask:0xf", True),
    ("v_mov_b32_dpp v1, v3 row_half_mirror row_mask:0xf bank_mask:0xf", False),
    ("s_branch .LBB0_9|v_mov_b32_e32 v3, v4|.LBB0_9:|v_permlane16_swap_b32 v1, v2", True),
    ("s_cbranch_scc1 .LBB0_9|s_nop 3|s_endpgm|.LBB0_9:|v_permlane16_swap_b32 v1, v2", True),
    ("s_branch .LBB0_9|v_permlane16_swap_b32 v1, v2|.LBB0_9:|v_mov_b32_e32 v3, v4", False),
])
def test_lane_exchanges_behind_inline_assembly_are_found(lines, refused):
    body = "".join(x + "\n" if x.endswith(":") else f"\t{x}\n" for x in lines.split("|"))
    written = "\tv_ashr_pk_i8_i32 v1, v4, v5, v6 op_sel:[0,0,0,1]\n"
    assert bool(build.check_lane_exchanges(f"_Zkern:\n\t;;#ASMSTART\n{written}\t;;#ASMEND\n{body}")) == refused
    assert not build.check_lane_exchanges(f"_Zkern:\n{written}{body}")  # (behind an instruction of the compiler's own it sees to them)


def test_no_kernel_as_built_has_one():
    directory = os.path.join(os.path.dirname(build.LIB), "_build")
    paths = glob.glob(os.path.join(directory, "**", "*gfx950.s"), recursive=True)
    if not paths:
        pytest.skip("no assembly here: the libraries were built elsewhere")
    for path in paths:
        with open(path) as f:
            assert build.check_assembly(f.read()) == [], path
