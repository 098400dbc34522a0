"""The build's checks of the two-group kernels' machine code: foreign vector-memory instructions among hand-counted
copies, wide stores whose data the next instruction overwrites, and what a full round of the attention may hold."""
import pytest

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


ROUND = (".LBB0_1:\n\tglobal_load_dword v30, v[2:3], off\n" + "\tv_mfma_f32_32x32x16_bf16 v[4:19], v[20:23], v[24:27], v[4:19]\n" * 16
         + "\t;;#ASMSTART\n\tglobal_load_lds_dwordx4 v1, s[2:3]\n\t;;#ASMEND\n" * 4 + "\ts_waitcnt vmcnt(4)\n"
         + "\tv_mfma_f32_32x32x16_bf16 v[4:19], v[20:23], v[24:27], v[4:19]\n" * 16 + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n")


def test_full_round_passes():
    assert ic.check_rounds("round", ROUND.splitlines()) == []


@pytest.mark.parametrize("was,now,found", [
    ("\ts_waitcnt vmcnt(4)\n", "\tscratch_load_dword v40, off, s32\n\ts_waitcnt vmcnt(4)\n", "scratch_load_dword"),
    ("\ts_waitcnt vmcnt(4)\n", "\tglobal_store_dwordx4 v[2:3], v[4:7], off\n\ts_waitcnt vmcnt(4)\n", "global_store_dwordx4"),
    ("vmcnt(4)", "vmcnt(5)", "leave [5]"),
    ("\ts_waitcnt vmcnt(4)\n", "", "leave []"),
    ("global_load_lds_dwordx4", "ds_nop", "no full round"),
])
def test_faults_of_a_full_round_are_found(was, now, found):
    errs = ic.check_rounds("round", ROUND.replace(was, now).splitlines())
    assert len(errs) == 1 and found in errs[0]
