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


def test_autotuner_picks_no_noise():
    """Flat times and small groups keep the default size; a real gain is taken,
    at the nearest size that has it."""
    from paper_2603_29942_amd.autotune import DEFAULT_OPS, pick_ops
    flat = {1500: 0.430, 12000: 0.457, DEFAULT_OPS: 0.455, 192000: 0.429}
    assert pick_ops(flat, 36.0) == DEFAULT_OPS  # 6% of 0.4 ms in a sample of 36 ms
    assert pick_ops(flat, 0.43) == 192000  # the group is the sample; 1500 is further off: a factor of 12, not 10.7
    assert pick_ops({6000: 7.7, DEFAULT_OPS: 6.9, 24000: 6.85, 96000: 6.84}, 7.0) == DEFAULT_OPS
    assert pick_ops({6000: 7.7, DEFAULT_OPS: 6.9, 48000: 6.3, 96000: 6.28, 192000: 6.27}, 7.0) == 48000
