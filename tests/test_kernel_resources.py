"""The kernels that a call without a launch shape runs, in the compiler's resource report: nothing
spills, and the registers leave room for the waves that the launch counts on."""
import os

import pytest

from paper_1804_10120_amd import build

REPORT = os.path.join(build.BUILD, "resource_usage.txt")
KERNELS = ("k_small", "k_staged", "k_batched_staged", "k_batched_args")


@pytest.mark.skipif(not os.path.exists(REPORT), reason="the library was not built here")
@pytest.mark.parametrize("kernel", KERNELS)
def test_default_kernels_do_not_spill(kernel):
    with open(REPORT) as f:
        table = build.resource_table(f.read())
    rows = {k: v for k, v in table.items() if f"{len(kernel)}{kernel}I" in k}
    assert rows, f"no {kernel} in the report"
    for name, (sgprs, vgprs, agprs, scratch, waves) in rows.items():
        assert scratch == 0, f"{name}: {scratch} bytes of scratch a lane"
        # two waves a SIMD: two blocks of 256 a compute unit, or eight of 64
        assert agprs == 0 and vgprs <= 256 and waves >= 2, f"{name}: {vgprs} + {agprs} registers"
