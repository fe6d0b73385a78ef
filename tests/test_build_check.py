"""The build's look at the persistent sweep's assembly: a register copy placed
before the lanes of a divergent branch come back is found, ordinary code and
other functions are not."""
from paper_2205_04295_amd import build

CLEAN = """
_ZN5mrpie10member_jobE:
\tv_mov_b32_e32 v1, v2
\ts_and_saveexec_b64 s[2:3], vcc
\ts_cbranch_execz .LBB0_2
; %bb.1:
\tglobal_atomic_or v0, v1, s[4:5]
.LBB0_2:
\ts_or_b64 exec, exec, s[2:3]
\tv_accvgpr_write_b32 a3, v218
"""
BAD = CLEAN.replace("\ts_or_b64 exec, exec, s[2:3]\n\tv_accvgpr_write_b32 a3, v218",
                    "\tv_accvgpr_write_b32 a3, v218\n\ts_or_b64 exec, exec, s[2:3]")


def test_copy_before_lanes_return_is_found():
    assert build.lost_copies(CLEAN, "member_job") == []
    assert build.lost_copies(BAD, "member_job") == [("_ZN5mrpie10member_jobE", ".LBB0_2:",
                                                     "v_accvgpr_write_b32 a3, v218")]
    assert build.lost_copies(BAD, "k_team") == []
