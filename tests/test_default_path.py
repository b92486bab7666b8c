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


def test_last_blocks_of_a_turn(rule):
    """Where blocks of 1024 points come to one or two for each compute unit, two points a lane: the
    inverse, the adjoint and the one-pass kernel over ragged fields on 16 bytes, and on aligned ones
    the kernels of few streams and the one-pass kernel."""
    for cus in (256, 128):
        one = cus * 1024
        for kernel in ("SymInverse", "ChainBwd", "ChainFwdBwd"):
            for n in (one * 13 // 16 + 8, one * 7 // 8 + 8, one - 8, one * 13 // 8 + 24,
                      2 * one - 8):
                assert rule(kernel, n, align=2, cus=cus)[0] == "shape", (kernel, n)
                assert rule(kernel, n, align=1, cus=cus)[0] != "shape", (kernel, n)
                if kernel != "SymInverse":      # left-out outputs: only read what is needed
                    assert rule(kernel, n, align=2, partial=True, cus=cus)[0] != "shape"
            for n in (one * 13 // 16 - 8, one + 8, one * 13 // 8 - 24, 2 * one + 8):
                assert rule(kernel, n, align=2, cus=cus)[0] != "shape", (kernel, n)
        for kernel in ("Christoffel", "CovDeriv", "Dtg", "Chain"):
            assert rule(kernel, one - 8, align=2, cus=cus)[0] != "shape"
        for kernel in ("SymInverse", "ChainFwdBwd"):
            assert rule(kernel, one, cus=cus)[0] == "shape"
            assert rule(kernel, one * 7 // 8, cus=cus)[0] == "small"
        assert rule("ChainBwd", one, cus=cus)[0] == "small"


def test_few_streams_are_staged_late(rule):
    """Below 12 streams never, below 20 from 2^17 ragged points, or from 2^20 where every component
    starts on 16 bytes."""
    for comps in ((3, 3), (6, 3)):                      # assign1, add1
        assert rule("Generic", 67 ** 3, align=2, comps=comps)[0] == "small", comps
        for n, align in ((65 ** 3, 1), (111 ** 3, 1), (112 ** 3, 16), (159 ** 3, 16)):
            assert rule("Generic", n, align=align, comps=comps)[0] == "shape", (comps, n)
    for kernel, comps in (("SymInverse", None), ("Generic", (9, 9)), ("Generic", (10, 6))):
        for n, align, path in ((47 ** 3, 1, "small"), (49 ** 3, 1, "small"), (51 ** 3, 1, "staged"),
                               (50 ** 3, 2, "small"), (54 ** 3, 2, "small"), (66 ** 3, 2, "small"),
                               (102 ** 3, 2, "staged"), (112 ** 3, 16, "staged")):
            assert rule(kernel, n, align=align, comps=comps)[0] == path, (kernel, n, align)
    for kernel in ("Christoffel", "CovDeriv", "Dtg", "ChainBwd", "ChainFwdBwd"):
        for align in (1, 2):
            assert rule(kernel, 47 ** 3, align=align)[0] == "staged"
    # a batch is staged from 2^18 points in all, whatever its outputs
    assert rule("ChainBwdBatched", P18, align=1, comps=(13, 1), partial=True)[0] == "staged"


def test_every_compiled_policy_is_reached(rule):
    """What a kernel may keep in the caches is what it is compiled for: a grid that is loaded first
    keeps no outputs, a forward batch no inputs; and every other combination occurs."""
    seen = set()
    bodies = [(k, None) for k in default_path_probe.COMPS]
    bodies += [("Generic", c) for c in ((3, 3), (9, 9), (10, 6), (27, 27), (9, 27), (12, 81),
                                        (90, 81), (99, 81), (108, 81))]
    bodies += [("ChainBwdBatched", (40, 1)), ("ChainBwdBatched", (40, 21))]
    sizes = [int(2 ** (9 + e / 8)) for e in range(0, 8 * 14)]
    for kernel, comps in bodies:
        for n in sizes:
            for align in (1, 2, 16):
                for m in (n, n // 16 * 16):
                    path, _, preload, kept = rule(kernel, m, align=align, comps=comps,
                                                  partial=comps in ((40, 1), (40, 21)))
                    if path == "shape":
                        assert kept == "nothing"
                        continue
                    group = kernel if "Batched" in kernel else path
                    seen.add((group, preload and kernel == "Generic", kept))
    loaded_first = {k for _, first, k in seen if first}
    assert loaded_first == {"nothing", "inputs"}, loaded_first
    for group, kept in (("small", {"nothing", "inputs", "outputs"}),
                        ("staged", {"nothing", "inputs", "outputs"}),
                        ("ChainBatched", {"nothing", "outputs"}),
                        ("ChainBatchedOnce", {"nothing", "outputs"}),
                        ("ChainBwdBatched", {"nothing", "inputs", "outputs"})):
        assert {k for g, _, k in seen if g == group} == kept, group
