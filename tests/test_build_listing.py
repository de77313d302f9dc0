"""What the build looks for in the assembly listing of the device code: vector instructions that no lane executes."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
spec = importlib.util.spec_from_file_location("_clt_build_listing", os.path.join(ROOT, "paper_2603_21014_amd", "build.py"))
B = importlib.util.module_from_spec(spec)
spec.loader.exec_module(B)

LOOP = """
row_kernel:
	s_mov_b64 s[72:73], exec
.LBB21_28:                              ;   Parent Loop
	v_readfirstlane_b32 s56, v0
	v_cmp_eq_u64_e32 vcc, s[56:57], v[0:1]
	s_and_saveexec_b64 s[2:3], s[2:3]
	buffer_load_dwordx4 v[10:13], v62, s[56:59], 0 offen nt
                                        ; implicit-def: $vgpr0_vgpr1
	s_xor_b64 exec, exec, s[2:3]
	s_cbranch_execnz .LBB21_28
; %bb.29:
"""
RESTORE = "	s_mov_b64 exec, s[72:73]\n"


@pytest.mark.parametrize("behind,lost", [
    # a spill store and a copy before the lanes are back
    ("	s_waitcnt vmcnt(1)\n	scratch_store_dwordx4 off, v[4:7], off offset:4 ; 16-byte Folded Spill\n	s_cmp_lg_u32 s60, 0\n" + RESTORE,
     [("row_kernel", "scratch_store_dwordx4 off, v[4:7], off offset:4")]),
    ("	v_mov_b32_e32 v53, v22\n" + RESTORE, [("row_kernel", "v_mov_b32_e32 v53, v22")]),
    # after them; single lanes; scalar work
    (RESTORE + "	scratch_store_dwordx4 off, v[4:7], off offset:4 ; 16-byte Folded Spill\n", []),
    ("	v_readlane_b32 s2, v71, 17\n	v_writelane_b32 v71, s2, 25\n	s_cmp_lg_u32 s60, 0\n" + RESTORE + "	v_mov_b32_e32 v0, 0\n", []),
    # an ordinary loop with lanes that leave early
    ("	s_or_b64 exec, exec, s[2:3]\n	v_mov_b32_e32 v0, 0\n", []),
    # a block that other paths reach as well
    (".LBB21_30:\n	v_mov_b32_e32 v0, 0\n" + RESTORE, [("row_kernel", "v_mov_b32_e32 v0, 0")]),
])
def test_vector_work_without_lanes(behind, lost):
    assert B.vector_work_without_lanes(LOOP + behind + "	s_endpgm\n") == lost
