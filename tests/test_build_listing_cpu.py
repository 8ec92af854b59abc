"""The build's search for spills of lanes that a block has not got back yet."""
from paper_2602_21237_amd.build import lost_lanes

KERNEL = """
_ZN2tj8k_kernelEv:                      ; @k_kernel
; %%bb.0:
\ts_load_dwordx2 s[0:1], s[4:5], 0x0
.LBB0_1:                                ; =>This Inner Loop Header: Depth=1
\tv_add_u32_e32 v1, 1, v1
\ts_cbranch_execnz .LBB0_1
; %%bb.2:                                ; in the loop's exit
%s
\ts_endpgm
.Lfunc_end0:
"""
SPILL = "\tscratch_store_dword off, v38, off offset:4 ; 4-byte Folded Spill"
BACK = "\ts_or_b64 exec, exec, s[2:3]"


def test_a_spill_before_the_lanes_are_back_is_found():
    bad = lost_lanes(KERNEL % "\n".join([SPILL, "\tv_mov_b32_e32 v38, 0", BACK]))
    assert len(bad) == 1 and bad[0].startswith("_ZN2tj8k_kernelEv: scratch_store_dword")


def test_spills_with_all_lanes_are_not():
    assert lost_lanes(KERNEL % "\n".join([BACK, SPILL])) == []
    assert lost_lanes(KERNEL % "\n".join([SPILL, ".LBB0_3:", BACK])) == []
    assert lost_lanes(KERNEL % "\n".join(["\tscratch_store_dword off, v38, off offset:4", BACK])) == []  # a program's own
