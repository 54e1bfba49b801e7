"""The build refuses persistent kernels that outgrow the registers of four waves per SIMD: the parser
of hipcc's resource-usage remarks finds them (CPU only, no compilation)."""
from paper_2511_15028_amd import _build as B

REMARKS = """\
x.hip:10:1: remark: Function Name: _Z15k_trace_persistPf [-Rpass-analysis=kernel-resource-usage]
x.hip:10:1: remark:     TotalSGPRs: 106 [-Rpass-analysis=kernel-resource-usage]
x.hip:10:1: remark:     VGPRs: 137 [-Rpass-analysis=kernel-resource-usage]
x.hip:10:1: remark:     VGPRs Spill: 500 [-Rpass-analysis=kernel-resource-usage]
x.hip:20:1: remark: Function Name: _Z13k_batch_tracePf [-Rpass-analysis=kernel-resource-usage]
x.hip:20:1: remark:     VGPRs: 128 [-Rpass-analysis=kernel-resource-usage]
x.hip:30:1: remark: Function Name: _Z7k_otherPf [-Rpass-analysis=kernel-resource-usage]
x.hip:30:1: remark:     VGPRs: 200 [-Rpass-analysis=kernel-resource-usage]
"""


def test_large_persistent_kernels_are_found():
    assert B._large_kernels(REMARKS) == [("_Z15k_trace_persistPf", 137)]

