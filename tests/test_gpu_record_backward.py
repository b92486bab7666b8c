"""A backward pass inside ``record``: recorded where it runs on the recording
thread, launched where the autograd engine runs it on a thread of its own."""
import pytest
import torch

from gpu_util import need_gpu
from paper_1804_10120_amd import dtg_chain
from paper_1804_10120_amd.ops import record

pytestmark = pytest.mark.gpu

NCOMP = {"g": 6, "dg": 18, "beta": 3, "dbeta": 9, "K": 6, "alpha": 1}


@pytest.mark.parametrize("threads", [False, True], ids=["calling_thread", "engine_thread"])
def test_backward_while_recording(threads):
    need_gpu()
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = [torch.rand(c, 200, dtype=torch.float64, device="cuda", generator=gen)
         for c in NCOMP.values()]
    x[0][[0, 3, 5]] += 3.0
    x = [t.requires_grad_() for t in x]
    w = torch.rand(6, 200, dtype=torch.float64, device="cuda", generator=gen)
    want = torch.autograd.grad(dtg_chain(*x), x, w)
    out = dtg_chain(*x)
    torch.cuda.synchronize()
    with torch.autograd.set_multithreading_enabled(threads), record() as calls:
        got = torch.autograd.grad(out, x, w)
    assert len(calls) == (0 if threads else 1)
    for c in calls:
        for t in got:
            t.fill_(float("nan"))
        c()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    # recording has ended: the next backward pass runs
    with torch.autograd.set_multithreading_enabled(threads):
        again = torch.autograd.grad(dtg_chain(*x), x, w)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, again))
