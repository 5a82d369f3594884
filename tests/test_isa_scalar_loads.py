"""The scanners for hand-placed scalar loads and for wait states around asm statements, and the
code-generation checks of the build.

A scalar load written as inline asm is invisible to the compiler between its issue and the
s_waitcnt that follows: nothing scheduled there may touch its destination SGPRs.  The kernels
use compiler-tracked constant-address-space loads instead; the scanner guards against a
hand-placed load coming back.  It is first shown to catch a planted violation in a small
listing, then run over the real device code of every source (where it must find nothing).
"""
import os
import shutil

import pytest

from paper_1705_09864_amd import build as hip_build
from paper_1705_09864_amd import isa_check

GOOD = """
_Z4kernv:
	s_load_dwordx2 s[4:5], s[0:1], 0x0
	s_waitcnt lgkmcnt(0)
	;;#ASMSTART
	s_load_dwordx16 s[36:51], s[4:5], 0x0
	;;#ASMEND
	v_xor_b32_e32 v1, s8, v2
	s_add_u32 s6, s6, s7
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	v_xor_b32_e32 v1, s36, v2
	s_endpgm
"""

# the compiler reloads a kernel argument into s[48:51] on the loop exit path while the
# inline-asm load of s[36:51] may still be in flight
BAD_WRITE = GOOD.replace("s_add_u32 s6, s6, s7", "s_cbranch_scc1 .LBB0_9").replace(
    "s_endpgm", "s_endpgm\n.LBB0_9:\n\ts_load_dwordx4 s[48:51], s[0:1], 0x78\n\ts_waitcnt lgkmcnt(0)\n\ts_endpgm")
BAD_READ = GOOD.replace("v_xor_b32_e32 v1, s8, v2", "v_xor_b32_e32 v1, s40, v2")


def _scan_text(tmp_path, text):
    f = tmp_path / "k.s"
    f.write_text(text)
    return isa_check.scan(str(f))


def test_scanner_accepts_clean_listing(tmp_path):
    assert _scan_text(tmp_path, GOOD) == []


def test_scanner_flags_write_on_branch_target(tmp_path):
    bad = _scan_text(tmp_path, BAD_WRITE)
    assert len(bad) == 1 and bad[0][3] == "writes" and bad[0][4] == (48, 49, 50, 51)


def test_scanner_flags_early_read(tmp_path):
    bad = _scan_text(tmp_path, BAD_READ)
    assert len(bad) == 1 and bad[0][3] == "reads" and bad[0][4] == (40,)


@pytest.mark.skipif(shutil.which(hip_build.HIPCC) is None and not os.path.exists(hip_build.HIPCC),
                    reason="hipcc not available")
def test_compiled_kernels_have_no_inflight_hazard():
    hip_build.check_scalar_loads()   # raises with the offending lines


@pytest.mark.skipif(shutil.which(hip_build.HIPCC) is None and not os.path.exists(hip_build.HIPCC),
                    reason="hipcc not available")
def test_compiled_kernels_keep_registers_and_wide_lds_reads():
    """No vector-register spills, no scratch memory, in the short-K convolution kernel one 16-byte LDS read
    per MFMA filter operand, one set of result stores for blocks inside the result and one for its edge, and no
    scalar-register spills, in the 64 x 64 per wave product kernel two sets of loads and packed words made by
    v_writelane_b32, and no calls (see build.check_codegen)."""
    hip_build.check_scalar_loads()   # makes sure the device listings exist
    hip_build.check_codegen()
    stats = isa_check.kernel_stats(hip_build.device_asm("conv_mfma.hip"))
    assert any("conv_mfma_ws_kernelILi9ELi1E" in k for k in stats)


def test_kernel_stats_count_behind_an_early_exit(tmp_path):
    f = tmp_path / "k.s"
    f.write_text("_Z4kernv:\n\ts_cbranch_scc1 .LBB0_2\n\ts_endpgm\n.LBB0_2:\n\tv_mov_b32_e32 v0, 0\n\ts_endpgm\n.Lfunc_end0:\n"
                 "\tv_mov_b32_e32 v0, 0\n    .name:           _Z4kernv\n    .vgpr_spill_count: 0\n")
    assert isa_check.kernel_stats(str(f))["_Z4kernv"] == (0, {"s_cbranch_scc1": 1, "s_endpgm": 2, "v_mov_b32_e32": 1})


# a compare writes a mask and an asm statement reads it at the join behind a branch around the
# compiler's own use of it: one wait state (the branch) on the short way, two are needed
HAZARD = """
_Z4kernv:
	v_cmp_le_f32_e64 s[0:1], 0, v11
	s_cbranch_scc1 .LBB0_1
	s_and_b64 s[0:1], s[0:1], s[40:41]
.LBB0_1:
	;;#ASMSTART
	v_writelane_b32 v10, s1, 3
	;;#ASMEND
	s_endpgm
"""
# an operand of a matrix-core instruction made by an asm statement
HAZARD_OPERAND = """
_Z4kernv:
	;;#ASMSTART
	v_and_or_b32 v23, v30, s4, v31
	;;#ASMEND
	v_mfma_i32_32x32x32_i8 v[0:15], v[20:23], v[24:27], v[0:15]
	s_endpgm
"""
# a wide store as asm, and the compiler's next use of a register that it sends
HAZARD_STORE = """
_Z4kernv:
	;;#ASMSTART
	global_store_dwordx4 v9, v[10:13], s[0:1] nt
	;;#ASMEND
	v_mov_b32_e32 v13, 0
	s_endpgm
"""
# (text, wait states there, wait states needed), None where nothing is to be reported
HAZARDS = [
    (HAZARD, (1, 2)),
    (HAZARD.replace("v_writelane_b32", "s_nop 0\n\tv_writelane_b32"), None),
    (HAZARD.replace("v_writelane_b32 v10, s1, 3", "s_nop 1\n\tv_writelane_b32 v10, s1, 3"), None),
    (HAZARD.replace(";;#ASMSTART", "").replace(";;#ASMEND", ""), None),  # the compiler's own pair
    (HAZARD.replace("v_cmp_le_f32_e64 s[0:1], 0, v11", "s_mov_b64 s[0:1], 0"), None),  # scalar results interlock
    (HAZARD.replace("v_writelane_b32 v10, s1, 3", "global_store_dword v3, v4, s[0:1] nt"), (1, 5)),
    (HAZARD.replace("v_cmp_le_f32_e64 s[0:1], 0, v11", "v_readlane_b32 s0, v9, 4"), None),  # (s1 is read, not s0)
    (HAZARD.replace("v_writelane_b32 v10, s1, 3", "v_add_u32_e32 v10, v11, v12").replace(
        "s_endpgm", "v_mov_b32_dpp v1, v10 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\ts_endpgm"), (0, 2)),
    (HAZARD.replace("v_cmp_le_f32_e64 s[0:1], 0, v11", "v_mfma_i32_32x32x32_i8 v[0:15], v[20:23], v[24:27], v[0:15]").replace(
        "v_writelane_b32 v10, s1, 3", "v_bcnt_u32_b32 v30, v15, v30"), (1, 20)),
    (HAZARD_OPERAND, (0, 2)),
    (HAZARD_OPERAND.replace(";;#ASMEND", ";;#ASMEND\n\tv_mov_b32_e32 v40, 0"), (1, 2)),
    (HAZARD_OPERAND.replace(";;#ASMEND", "s_nop 1\n\t;;#ASMEND"), None),
    (HAZARD_OPERAND.replace(";;#ASMSTART", "").replace(";;#ASMEND", ""), None),
    (HAZARD_STORE, (0, 2)),
    (HAZARD_STORE.replace(";;#ASMEND", "s_nop 0\n\t;;#ASMEND"), (1, 2)),
    (HAZARD_STORE.replace(";;#ASMEND", "s_nop 1\n\t;;#ASMEND"), None),
    (HAZARD_STORE.replace("v_mov_b32_e32 v13", "v_mov_b32_e32 v14"), None),  # (v14 is not sent)
    (HAZARD_STORE.replace("dwordx4", "dwordx2").replace("v[10:13]", "v[12:13]"), None),
]


@pytest.mark.parametrize("text,expected", HAZARDS)
def test_asm_wait_states(tmp_path, text, expected):
    f = tmp_path / "k.s"
    f.write_text(text)
    bad = isa_check.asm_hazards(str(f))
    assert [e[4:] for e in bad] == ([expected] if expected else [])


@pytest.mark.skipif(shutil.which(hip_build.HIPCC) is None and not os.path.exists(hip_build.HIPCC),
                    reason="hipcc not available")
def test_compiled_kernels_leave_asm_its_wait_states():
    hip_build.check_asm_hazards()   # raises with the offending lines
