"""The two forms of the batch without a plan: descriptors in the kernel arguments, 46 subgrids a
launch (no launch shape), and tables that kernels write to the library's array (a launch shape).
Both from the native marshalling, which takes a list of dicts without empty subgrids, and from the
Python one."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import CANARY, assert_close, need_gpu
from paper_1804_10120_amd import BatchPlan, _abi, tl_batch_run_noalloc
from paper_1804_10120_amd.synth import make_fields

pytestmark = pytest.mark.gpu

KEYS = ("g", "dg", "beta", "dbeta", "K", "alpha")
SHAPE = dict(block=64, ppt=1, nt=True)
TUNES = {"arguments": None, "tables": SHAPE}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def field(host, pad):
    """A device copy with its own leading dimension; pad: doubles beyond n, None for whole lines."""
    c, n = host.shape
    ld = n + pad if pad is not None else -(-n // 16) * 16
    buf = torch.full((c, max(ld, 1)), CANARY, dtype=torch.float64, device="cuda")
    buf[:, :n] = torch.from_numpy(np.ascontiguousarray(host))
    return buf[:, :n]


def subgrids(sizes, seed):
    """Subgrids whose layouts differ (contiguous, padded, whole lines), each with an output."""
    hosts = [make_fields(int(n), seed=seed * 1000 + d) for d, n in enumerate(sizes)]
    doms = []
    for d, f in enumerate(hosts):
        pad = (0, 1, 5, None)[d % 4]
        doms.append(dict({k: field(f[k], pad) for k in KEYS},
                         dtg=field(np.full((6, f["g"].shape[1]), CANARY), (3, None, 0)[d % 3])))
    return hosts, doms


def clear(doms):
    for d in doms:
        d["dtg"].fill_(float("nan"))


def check(hosts, outs, what):
    for i, (f, o) in enumerate(zip(hosts, outs)):
        if f["g"].shape[1]:
            assert_close(o, oracle.dtg_chain(*[f[k] for k in KEYS]), what=f"{what}: subgrid {i}")


@pytest.mark.parametrize("count", [2, 45, 46, 47, 92, 93])
def test_native_marshalling_of_many_subgrids(count):
    """Sizes and layouts of their own for every subgrid, none empty: the extension takes the call."""
    hosts, doms = subgrids([1 + (i * 337) % 900 for i in range(count)], seed=51)
    got = _abi.bind().noalloc(doms)
    torch.cuda.synchronize()
    assert got is not None and all(a is d["dtg"] for a, d in zip(got, doms))
    check(hosts, got, "native")
    first = [o.clone() for o in got]
    clear(doms)
    again = tl_batch_run_noalloc(tuple(doms))       # a tuple is marshalled in Python
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(first, again))


@pytest.mark.parametrize("form", list(TUNES))
def test_limit_of_subgrids(form):
    """1024 subgrids, empty ones among them: 23 launches of 46, or 34 that write the tables."""
    rng = np.random.default_rng(61)
    sizes = [int(x) for x in rng.integers(0, 40, size=_abi.TL_NOALLOC_MAX_DOMAINS)]
    hosts, doms = subgrids(sizes, seed=52)
    got = tl_batch_run_noalloc(doms, tune=TUNES[form])
    torch.cuda.synchronize()
    check(hosts, got, form)


@pytest.mark.parametrize("form", list(TUNES))
def test_side_stream_and_fewer_subgrids_afterwards(form):
    """On a stream of its own, repeated, then fewer and smaller subgrids on the same stream."""
    hosts, doms = subgrids([9 ** 3, 40, 30 ** 3, 1] + [77] * 60, seed=53)
    small_hosts, small = subgrids([5, 700, 2], seed=54)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        first = [o.clone() for o in tl_batch_run_noalloc(doms, tune=TUNES[form])]
        clear(doms)
        again = tl_batch_run_noalloc(doms, tune=TUNES[form])
        last = tl_batch_run_noalloc(small, tune=TUNES[form])
    s.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    check(hosts, again, form)
    check(small_hosts, last, form + ", fewer")


@pytest.mark.parametrize("form", list(TUNES))
def test_captured_in_a_graph(form):
    """Replayed several times with another batch, of the same form, between the replays."""
    hosts, doms = subgrids([20 ** 3, 7, 33 ** 3] + [50] * 46, seed=55)
    _, other = subgrids([300, 20], seed=56)
    eager = [o.clone() for o in tl_batch_run_noalloc(doms, tune=TUNES[form])]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tl_batch_run_noalloc(doms, tune=TUNES[form])
    for rep in range(3):
        clear(doms)
        tl_batch_run_noalloc(other, tune=TUNES[form])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, d["dtg"]) for a, d in zip(eager, doms)), f"replay {rep}"
    check(hosts, [d["dtg"] for d in doms], form)


# ---- the staged kernel of a plan with outputs left out

GRADS = ("g", "dg", "beta", "dbeta", "K", "alpha")
NCOMP = (6, 18, 3, 9, 6, 1)


@pytest.mark.parametrize("want", [(0, 1, 0, 0, 1, 1), (1, 0, 0, 0, 0, 0), (0, 0, 0, 1, 0, 0),
                                  (0, 0, 1, 1, 0, 1)],
                         ids=["dg_K_alpha", "g", "dbeta", "gauge"])
def test_staged_plan_with_outputs_left_out(want):
    """From 2^18 points in all a plan is staged; the subgrids differ in the outputs they have too."""
    sizes = [70000, 1, 255, 65536, 0, 257, 90001, 40000]
    assert sum(sizes) >= 2 ** 18
    hosts = [make_fields(n, seed=57000 + d) for d, n in enumerate(sizes)]
    got = []
    for tune in (None, dict(block=128, ppt=1, nt=True)):
        doms, bufs = [], []
        for d, f in enumerate(hosts):
            pad = (0, 1, None)[d % 3]
            dom = {k: field(f[k], pad) for k in ("g", "dg", "beta", "K", "alpha", "W")}
            for i, (k, c) in enumerate(zip(GRADS, NCOMP)):
                if want[i] or (d == 3 and i == 2):      # one subgrid has an output more
                    dom[k + "_bar"] = field(np.full((c, sizes[d]), CANARY), pad)
                    bufs.append(dom[k + "_bar"])
            doms.append(dom)
        plan = BatchPlan(doms, kind="bwd", want=want, tune=tune)
        plan.run()
        torch.cuda.synchronize()
        got.append((bufs, plan.outputs))
        plan.close()
    for a, b in zip(got[0][0], got[1][0]):
        assert torch.equal(a._base, b._base)        # the padding around the fields included
    for f, outs in zip(hosts, got[0][1]):
        if f["g"].shape[1] == 0:
            continue
        ref = oracle.dtg_chain_vjp(tuple(f[k] for k in KEYS), f["W"])
        for k, w, o in zip(GRADS, want, outs):
            if w:
                assert_close(o, ref[k], what=f"{k}_bar n={f['g'].shape[1]}")
