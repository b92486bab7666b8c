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


@pytest.mark.skipif(not os.path.exists(REPORT), reason="the library was not built here")
def test_launch_shapes_keep_their_registers():
    """The covariant derivative at two points a lane keeps four waves a SIMD in every block size,
    and the adjoint at two points in blocks of 1024, which cannot but spill, stays at two cache lines
    a lane with buffer addressing (a product rounded on its own for the three gradients it goes
    into needed 188 bytes)."""
    with open(REPORT) as f:
        table = build.resource_table(f.read())

    def rows(op, block, ppt, form=""):
        want = f"k_pointsINS_{len(op)}{op}ELi{block}ELi{ppt}E{form}"
        return [v for k, v in table.items() if want in k.replace("2tl", "")]
    for block in (64, 128, 256, 512, 1024):
        found = rows("OpCovDeriv", block, 2)
        assert len(found) == 3
        for sgprs, vgprs, agprs, scratch, waves in found:
            assert waves >= 4 and scratch == 0, (block, vgprs, scratch, waves)
    (buffered,) = rows("OpChainBwd", 1024, 2, "Lb1ELb1E")
    assert buffered[3] <= 128, buffered


@pytest.mark.skipif(not os.path.exists(REPORT), reason="the library was not built here")
def test_no_policy_is_compiled_that_no_call_reaches():
    """Load policy 0 or 2 and store policy 16 or 2: inputs kept, outputs kept, neither, never both;
    a grid that is loaded first keeps no outputs, a forward batch no inputs."""
    with open(REPORT) as f:
        table = build.resource_table(f.read())
    both = [k for k in table if "ELi0ELi16E" in k]
    assert not both, both[:3]
    assert not [k for k in table if "k_small" in k and "ELi16ELb1E" in k]
    assert sum("k_batched_args" in k for k in table) == 2
    assert sum("16k_batched_stagedINS_7OpChainE" in k for k in table) == 2
    assert sum("16k_batched_stagedINS_10OpChainBwdE" in k for k in table) == 3
