"""CPU: the register counts that the launch shapes rely on, beside the budgets of the fused passes'
own test: every 512-thread depositing pass without the thermostat, with a bond length or without,
and the force pass of the separate-call step keep 4 waves per SIMD (at most 128 VGPRs)."""
import re

from test_kernel_resources import kernel_metadata


def test_forms_that_need_four_waves_per_simd(tmp_path):
    md = kernel_metadata(tmp_path)
    deposit = {k: v for k, v in md.items() if re.search(r"k_advance_scatterILb[01]ELi512ELb[01]ELb0E", k)}
    force = {k: v for k, v in md.items() if "k_force_kickI" in k}
    assert {re.search(r"ILb([01])E", k).group(1) for k in deposit} == {"0", "1"}
    assert len(force) == 8
    for k, v in {**deposit, **force}.items():
        assert v["vgpr_count"] <= 128, (k, v)
