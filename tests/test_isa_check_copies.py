"""The build's checks of the two-group GEMM kernels' machine code: foreign vector-memory instructions among hand-counted
copies, and wide stores whose data the next instruction overwrites."""
from paper_2510_25590_amd import isa_check as ic

LOOP = """
	s_mov_b32 s0, 0
.LBB0_1:
	;;#ASMSTART
	global_load_lds_dwordx4 v1, s[2:3]
	;;#ASMEND
	v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[4:7]
	s_cbranch_scc1 .LBB0_1
	buffer_store_dwordx4 v[4:7], v20, s[8:11], 0 offen
	s_nop 0
	v_add_u32_e32 v4, 0x7000, v21
	s_endpgm
"""


def test_loop_of_copies_passes():
    lines = LOOP.strip().splitlines()
    assert ic.check_copies("clean", lines) == [] and ic.check_wide_stores("clean", lines) == []


def test_foreign_load_in_the_loop_is_found():
    errs = ic.check_copies("foreign", LOOP.replace("\tv_mfma", "\tglobal_load_dword v30, v[2:3], off\n\tv_mfma").strip().splitlines())
    assert errs and "global_load_dword v30" in errs[0]


def test_overwritten_store_data_is_found():
    errs = ic.check_wide_stores("store", LOOP.replace("\ts_nop 0\n", "").strip().splitlines())
    assert errs and "v_add_u32_e32 v4" in errs[0]
