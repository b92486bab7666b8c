"""A batch plan's launch captured into a caller's HIP graph: the graph holds the
work, so a replay writes the outputs."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_close, dev, need_gpu
from paper_1804_10120_amd import BatchPlan
from paper_1804_10120_amd.synth import make_fields

pytestmark = pytest.mark.gpu

KEYS = ("g", "dg", "beta", "dbeta", "K", "alpha")
# the kernel of a launch shape (below 2^18 points in all) and the staged one
SIZES = {"small": [500, 0, 1, 2048, 77], "staged": [2 ** 18 - 1000, 0, 1, 999]}


@pytest.mark.parametrize("run", ["run", "run_direct"])
@pytest.mark.parametrize("sizes", list(SIZES))
@pytest.mark.parametrize("kind", ["fwd", "bwd"])
def test_captured_plan_replays(kind, sizes, run):
    """Several replays, each over outputs filled with NaN, with eager work and
    synchronisation in between; new inputs before the last."""
    need_gpu()
    hosts = [make_fields(n, seed=700 + d) for d, n in enumerate(SIZES[sizes])]
    names = KEYS if kind == "fwd" else ("g", "dg", "beta", "K", "alpha", "W")
    devs = [{k: dev(f[k]) for k in names} for f in hosts]
    plan = BatchPlan(devs, kind=kind)
    outs = plan.outputs if kind == "fwd" else [o for d in plan.outputs for o in d]
    plan.run()
    torch.cuda.synchronize()
    eager = [o.clone() for o in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        getattr(plan, run)()
    for rep in range(3):
        for o in outs:
            o.fill_(np.nan)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(eager, outs)):
            assert torch.equal(a, b), f"replay {rep}: output {i} differs from the eager run"
    for f, d in zip(hosts, devs):
        f["K"] = 2.0 * f["K"]
        d["K"].mul_(2.0)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    for f, o in zip(hosts, plan.outputs):
        if f["g"].shape[1] == 0:
            continue
        if kind == "fwd":
            assert_close(o, oracle.dtg_chain(*[f[k] for k in KEYS]), what="replay on new inputs")
        else:
            ref = oracle.dtg_chain_vjp(tuple(f[k] for k in KEYS), f["W"])
            for k, x in zip(KEYS, o):
                assert_close(x, ref[k], what=f"replay on new inputs, {k}_bar")
    plan.close()
