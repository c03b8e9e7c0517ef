"""The build's check that kernels with assembler reads of LDS stay out of scratch memory, on remarks as the compiler prints them."""
from paper_2001_04206_amd import build

REMARK = """csrc/dn_gemm.hip:1094:0: remark: Function Name: _ZN2dn11gemm_kernelINS_%s [-Rpass-analysis=kernel-resource-usage]
csrc/dn_gemm.hip:1094:0: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
csrc/dn_gemm.hip:1094:0: remark:     ScratchSize [bytes/lane]: %d [-Rpass-analysis=kernel-resource-usage]
"""


def test_scratch_in_a_slice_kernel_is_found():
    text = REMARK % ("9SliceTileILi64", 0) + REMARK % ("4TileILi128", 36) + REMARK % ("9SliceTileILi32", 20) + REMARK % ("18corr3_split_kernelILi1", 4)
    spilled, seen = build.kernels_with_scratch(text)
    assert seen == 3 and len(spilled) == 2 and "SliceTileILi32" in spilled[0] and "corr3" in spilled[1]


def test_no_scratch_passes():
    assert build.kernels_with_scratch(REMARK % ("9SliceTileILi64", 0)) == ([], 1)
    assert build.kernels_with_scratch("") == ([], 0)   # the build treats this as a failure: the check saw nothing
