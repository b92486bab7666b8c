"""tl_kernel_info without a shape answers for the default members given as one."""
import pytest

from gpu_util import need_gpu
from paper_1804_10120_amd import _abi, tl_kernel_info

pytestmark = pytest.mark.gpu

BLOCK = {"dtg_chain_batched": 128, "dtg_chain_bwd_batched": 128}


@pytest.mark.parametrize("kernel", ["sym_inverse", "christoffel", "cov_deriv", "dtg", "dtg_chain",
                                    "dtg_chain_bwd", "dtg_chain_fwd_bwd", *BLOCK, *_abi.EXPRS])
def test_no_shape_is_the_default_members(kernel):
    need_gpu()
    a = tl_kernel_info(kernel)
    assert a == tl_kernel_info(kernel, tune=dict(nt=True))
    assert a["block"] == BLOCK.get(kernel, 256) and a["ppt"] == 1, a
    assert a["flags"] == _abi.TL_TUNE_NT and a["scratch_bytes"] == 0, a
