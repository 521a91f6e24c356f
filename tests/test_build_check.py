"""The build's check of the compiled kernels: lane-wise code at the join of a
divergent branch must not stand ahead of the exec mask's restore."""
import glob
import os

import pytest

from paper_2109_01928_amd import build as B

BRANCH = """_Z6kernelv: ; @_Z6kernelv
; %bb.0:
	v_mov_b64_e32 v[92:93], v[8:9]
	s_and_saveexec_b64 s[12:13], s[4:5]
	s_cbranch_execz .LBB0_2
; %bb.1:
	v_add_f64 v[4:5], v[4:5], -v[158:159]
.LBB0_2:                                ; %join
@JOIN@	s_endpgm
.Lfunc_end0:
"""
RESTORE = "\ts_or_b64 exec, exec, s[12:13]\n"


def _kernel(join):
    return BRANCH.replace("@JOIN@", join).splitlines()


@pytest.mark.parametrize("code", ["\tv_mov_b64_e32 v[92:93], v[62:63]\n",
                                  "\tscratch_store_dwordx2 off, v[70:71], off offset:328 ; 8-byte Folded Spill\n",
                                  "\tscratch_load_dwordx2 v[6:7], off, off offset:344 ; 8-byte Folded Reload\n"])
def test_lane_wise_code_ahead_of_the_restore_is_found(code):
    found = B.masked_join_code(_kernel("\ts_mov_b32 s76, s92\n" + code + RESTORE))
    assert [(f, i) for _, f, i in found] == [("_Z6kernelv", code.split(";")[0].strip())]


def test_code_of_the_sides_and_scalar_spills_are_not():
    ok = ("\tv_writelane_b32 v255, s43, 4\n\tv_readlane_b32 s0, v255, 4\n\ts_mov_b32 s76, s92\n" + RESTORE +
          "\tv_mov_b64_e32 v[92:93], v[62:63]\n")
    assert B.masked_join_code(_kernel(ok)) == []
    # a block that opens the next branch: its own mask, then the join's
    nested = "\tv_mov_b64_e32 v[0:1], 0\n\ts_and_saveexec_b64 s[0:1], s[2:3]\n\ts_cbranch_execz .LBB0_3\n"
    assert B.masked_join_code(_kernel(nested)) == []


def test_built_kernels_hold_none():
    files = glob.glob(os.path.join(os.path.dirname(B.LIB), "_build", "*-amdhsa-*.s"))
    if not files:
        pytest.skip("the library was built elsewhere")
    for path in files:
        with open(path) as f:
            assert B.masked_join_code(f) == [], path
