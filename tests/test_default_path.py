"""Which kernel a call without a launch shape runs, where a measured loss decides it."""
import pytest

import default_path_probe

P16, P18, P20 = 1 << 16, 1 << 18, 1 << 20


@pytest.fixture(scope="module")
def rule():
    return default_path_probe.load()


@pytest.mark.parametrize("comps", [(90, 81), (81, 81)], ids=["contract1", "assign4"])
def test_alternating_bodies_keep_the_launch_shape(rule, comps):
    """A wide body with about one load for each store, over aligned points beyond the sizes at
    which 64-thread blocks gain."""
    for n in (62 ** 3, P18, 67 ** 3, 72 ** 3, 88 ** 3, 100 ** 3, P20 - 1):
        assert rule("Generic", n, comps=comps)[0] == "shape", n
    for n in (17 ** 3, 40 ** 3, 50 ** 3, 59 ** 3):
        assert rule("Generic", n, comps=comps)[0] == "small", n
    assert rule("Generic", P20 + 16, comps=comps)[0] == "staged"
    for n in (63 ** 3, 75 ** 3):
        assert rule("Generic", n, align=1, comps=comps)[0] == "staged", n


@pytest.mark.parametrize("comps", [(99, 81), (108, 81), (12, 81)],
                         ids=["contract2", "contract3", "mult3"])
def test_other_wide_bodies_do_not(rule, comps):
    for n in (62 ** 3, 67 ** 3, 76 ** 3):
        assert rule("Generic", n, comps=comps)[0] == "small", n
