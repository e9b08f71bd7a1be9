"""The build refuses scratch in every kernel that loads operands into accumulation registers from assembly: a spill right
after such a load would save the register before its data has arrived, and give wrong results without an error."""
import pytest

from paper_2401_09149_amd import build

REMARKS = """attn.hip:1:1: remark: Function Name: {} [-Rpass-analysis=kernel-resource-usage]
attn.hip:1:1: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
attn.hip:1:1: remark:     ScratchSize [bytes/lane]: {} [-Rpass-analysis=kernel-resource-usage]
"""


@pytest.mark.parametrize("name", [
    "_ZN2ie20attn_fwd_wide_kernelILb0EEEvNS_10AttnParamsE",
    "_ZN2ie20attn_bwd_dkdv_kernelILi64ELb0ELb0EEEvNS_10AttnParamsE",
    "_ZN2ie20attn_bwd_dkdv_kernelILi128ELb1ELb0EEEvNS_10AttnParamsE",
    "_ZN2ie20attn_bwd_both_kernelILi64ELb1ELb0EEEvNS_10AttnParamsES1_",
    "_ZN2ie20attn_bwd_both_kernelILi64ELb0ELb1EEEvNS_10AttnParamsES1_",
    "_ZN2ie20attn_bwd_both_kernelILi128ELb0ELb1EEEvNS_10AttnParamsES1_",
])
def test_scratch_is_refused(name):
    build._check_scratch("attn.hip", REMARKS.format(name, 0))
    with pytest.raises(RuntimeError, match="spills to scratch"):
        build._check_scratch("attn.hip", REMARKS.format(name, 8))
