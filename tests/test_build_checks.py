"""The build's look at the compiled device code (paper_2603_29942_amd/build.py)."""
import pytest

from paper_2603_29942_amd.build import check, outside_registers, vgpr_spills

REMARKS = """a.hip:1:1: remark: Function Name: enum_a [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     VGPRs: 200 [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:2:1: remark: Function Name: mlp_b [-Rpass-analysis=kernel-resource-usage]
a.hip:2:1: remark:     VGPRs Spill: {n} [-Rpass-analysis=kernel-resource-usage]
"""
LISTING = """enum_a:                                ; @enum_a
; %bb.0:
	v_mov_b32_e32 v0, 0
	global_load_dwordx4 v[0:3], v[4:5], off
{a}
	s_endpgm
helper:                                ; @helper
	v_add_u32_e32 v0, v0, v1
{b}
	s_setpc_b64 s[30:31]
"""


def test_clean_code_passes():
    assert vgpr_spills(REMARKS.format(n=0)) == {"enum_a": 0, "mlp_b": 0}
    check(REMARKS.format(n=0), LISTING.format(a="", b=""))


@pytest.mark.parametrize("remarks,listing", [
    (REMARKS.format(n=4), LISTING.format(a="", b="")),  # any kernel, not only the enumeration's
    ("", LISTING.format(a="", b="")),
    (REMARKS.format(n=0), ""),
    (REMARKS.format(n=0), LISTING.format(a="\ts_swappc_b64 s[30:31], s[16:17]", b="")),
    (REMARKS.format(n=0), LISTING.format(a="", b="\tscratch_store_dword off, v40, s33 ; 4-byte Folded Spill")),
    (REMARKS.format(n=0), LISTING.format(a="", b="\tscratch_load_dwordx2 v[2:3], off, s32")),
])
def test_spills_calls_and_scratch_are_refused(remarks, listing):
    with pytest.raises(RuntimeError):
        check(remarks, listing)


def test_the_function_is_named():
    assert list(outside_registers(LISTING.format(a="", b="\tscratch_store_dword off, v40, s33"))) == ["helper"]
