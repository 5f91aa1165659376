"""The build's check for register spills, on remarks as the compiler prints them,
and that it is on for the kernels it is meant for."""
import pytest

from paper_2104_01196_amd import build

REMARKS = """
resident.hip:743:1: remark: Function Name: _ZN3gs210k_residentIffLi0ELi1024EEEvNS_7ResArgsE [-Rpass-analysis=kernel-resource-usage]
resident.hip:743:1: remark:     TotalSGPRs: 106 [-Rpass-analysis=kernel-resource-usage]
resident.hip:743:1: remark:     VGPRs: 128 [-Rpass-analysis=kernel-resource-usage]
resident.hip:743:1: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis=kernel-resource-usage]
resident.hip:743:1: remark:     SGPRs Spill: 139 [-Rpass-analysis=kernel-resource-usage]
resident.hip:743:1: remark:     VGPRs Spill: {spill} [-Rpass-analysis=kernel-resource-usage]
resident.hip:1:1: remark: Function Name: _ZN3gs25otherEv [-Rpass-analysis=kernel-resource-usage]
resident.hip:1:1: remark:     ScratchSize [bytes/lane]: 64 [-Rpass-analysis=kernel-resource-usage]
resident.hip:1:1: remark:     VGPRs Spill: 9 [-Rpass-analysis=kernel-resource-usage]
"""


def test_spills_and_scratch_fail():
    assert build.check_spills(REMARKS.format(scratch=0, spill=0), "k_resident") == 1
    for scratch, spill in ((220, 55), (36, 0), (0, 1)):
        with pytest.raises(RuntimeError, match="must be 0"):
            build.check_spills(REMARKS.format(scratch=scratch, spill=spill), "k_resident")
    with pytest.raises(RuntimeError, match="no resource remarks"):
        build.check_spills(REMARKS.format(scratch=0, spill=0), "k_small_apply")


def test_on_for_the_kernels_that_wait():
    assert build.NO_SPILLS == {"resident.hip": "k_resident", "small.hip": "k_small_apply"}
