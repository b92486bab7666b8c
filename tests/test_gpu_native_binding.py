"""The native marshalling of plain calls and the native autograd node against the
Python code they stand in for: the same results bit for bit, the same shapes,
strides and objects, and the same exceptions where a call is refused or a
transform does not apply.  Each scenario runs once through the extension and
once with it answering None to everything."""
import types

import pytest
import torch

from gpu_util import need_gpu
from paper_1804_10120_amd import (BatchPlan, _abi, dtg_chain, generated, ops, tl_batch_run_noalloc,
                                  tl_christoffel, tl_cov_deriv, tl_dtg, tl_dtg_chain,
                                  tl_dtg_chain_bwd, tl_dtg_chain_fwd_bwd, tl_expr, tl_sym_inverse)

pytestmark = pytest.mark.gpu

NCOMP = {"g": 6, "dg": 18, "beta": 3, "dbeta": 9, "K": 6, "alpha": 1, "w": 6}
CHAIN = ("g", "dg", "beta", "dbeta", "K", "alpha")
BWD = ("g", "dg", "beta", "K", "alpha", "w")


def fields(n=333, flat_alpha=False, pad=0, seed=0):
    need_gpu()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    f = {k: (torch.rand(c, n + pad, dtype=torch.float64, device="cuda", generator=gen) - 0.5)[:, :n]
         for k, c in NCOMP.items()}
    f["g"][[0, 3, 5]] += 3.0
    if flat_alpha:
        f["alpha"] = f["alpha"][0]
    return f


def outcome(fn):
    """What a call gives, as something to compare."""
    try:
        r = fn()
    except Exception as e:      # noqa: BLE001 - the exception is the result
        return type(e).__name__, str(e).splitlines()[0] if str(e) else ""
    torch.cuda.synchronize()

    def plain(x):
        if isinstance(x, torch.Tensor):
            return tuple(x.shape), x.stride(), x.requires_grad, x.detach().cpu().numpy().tobytes()
        if isinstance(x, (list, tuple)):
            return type(x).__name__, [plain(v) for v in x]
        return x
    return plain(r)


def both(monkeypatch, make):
    """The outcomes of make()'s call through the extension and through Python."""
    nothing = types.SimpleNamespace(**{k: lambda *a: None for k in
                                       ("call", "fields", "noalloc", "plan_launch", "dtg_chain")})
    _abi.bind()
    got = []
    for module in (_abi._bind, nothing):
        monkeypatch.setattr(_abi, "_bind", module)
        got.append(outcome(make()))
    return got


def ones(c, n=333):
    return torch.ones(c, n, dtype=torch.float64, device="cuda")


CALLS = {
    "inverse": lambda f: tl_sym_inverse(f["g"]),
    "christoffel": lambda f: tl_christoffel(f["g"], f["dg"]),
    "cov_deriv": lambda f: tl_cov_deriv(f["dg"], f["beta"], f["dbeta"]),
    "dtg": lambda f: tl_dtg(f["alpha"], f["K"], f["dbeta"]),
    "chain": lambda f: tl_dtg_chain(*[f[k] for k in CHAIN]),
    "chain_out": lambda f: (lambda o: [tl_dtg_chain(*[f[k] for k in CHAIN], o) is o, o])(ones(6)),
    "bwd": lambda f: tl_dtg_chain_bwd(*[f[k] for k in BWD]),
    "bwd_some": lambda f: tl_dtg_chain_bwd(*[f[k] for k in BWD], want=(0, 1, 0, 1, 0, 1)),
    "bwd_out_and_want": lambda f: tl_dtg_chain_bwd(*[f[k] for k in BWD], K_bar=ones(6),
                                                   want=(0, 0, 1, 0, 0, 0)),
    "bwd_none": lambda f: tl_dtg_chain_bwd(*[f[k] for k in BWD], want=(0,) * 6),
    "bwd_short_want": lambda f: tl_dtg_chain_bwd(*[f[k] for k in BWD], want=(1, 1)),
    "fwd_bwd": lambda f: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], f["w"]),
    "fwd_bwd_some": lambda f: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], f["w"],
                                                   want=(1, 0, 0, 1, 0, 0, 0)),
    "expr": lambda f: tl_expr("kij", f["alpha"], f["g"], f["beta"]),
    "expr_few": lambda f: tl_expr("kij", f["alpha"], f["g"]),
    "generated": lambda f: generated.call("dtg", f["alpha"], f["K"], f["dbeta"]),
    "generated_out": lambda f: generated.call("kij", f["alpha"], f["g"], f["beta"], outs=[ones(6)]),
    "generated_few": lambda f: generated.call("kij", f["alpha"], f["g"]),
    "noalloc": lambda f: tl_batch_run_noalloc([dict(f, dtg=ones(6))] * 1),
    "noalloc_no_out": lambda f: tl_batch_run_noalloc([dict(f)]),
    "overlap": lambda f: tl_dtg_chain(*[f[k] for k in CHAIN], f["K"]),
    "float32": lambda f: tl_sym_inverse(f["g"].float()),
    "host": lambda f: tl_sym_inverse(f["g"].cpu()),
    "shape": lambda f: tl_sym_inverse(f["dg"]),
    "points": lambda f: tl_christoffel(f["g"], f["dg"][:, :5]),
    "stride": lambda f: tl_sym_inverse(f["g"].T.contiguous().T),
    "not_a_tensor": lambda f: tl_sym_inverse([1.0]),
    "no_points": lambda f: tl_sym_inverse(f["g"][:, :0]),
    "one_point": lambda f: tl_sym_inverse(f["g"][:, :1]),
    "neg_view": lambda f: tl_sym_inverse(torch._neg_view(f["g"])),
    "requires_grad": lambda f: tl_sym_inverse(f["g"].clone().requires_grad_()),
}


@pytest.mark.parametrize("flat_alpha", [False, True], ids=["alpha1n", "alphan"])
@pytest.mark.parametrize("name", list(CALLS))
def test_calls(monkeypatch, name, flat_alpha):
    a, b = both(monkeypatch, lambda: lambda: CALLS[name](fields(flat_alpha=flat_alpha, pad=3)))
    assert a == b


def leaves(f, wrt=CHAIN):
    return [f[k].clone().requires_grad_(k in wrt) for k in CHAIN]


def grad(x, w, wrt=None, **kw):
    return list(torch.autograd.grad(dtg_chain(*x), [t for t in x if t.requires_grad] if wrt is None
                                    else wrt, w, **kw))


def _second(f):
    x = leaves(f)
    w = f["w"].clone().requires_grad_()
    g = grad(x, w, create_graph=True)
    return torch.autograd.grad(g[0].sum(), x[0])


def _twice(f):
    x = leaves(f)
    out = dtg_chain(*x)
    a = torch.autograd.grad(out, x, f["w"], retain_graph=True)
    b = torch.autograd.grad(out, x, f["w"])
    assert all(torch.equal(p, q) for p, q in zip(a, b))
    return torch.autograd.grad(out, x, f["w"])       # the graph is freed


def _hooks(f, unpack):
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(t.shape) or t, unpack):
        out = dtg_chain(*leaves(f))
    x = [out]
    out.backward(f["w"])
    return [len(seen)] + x


def _inplace(f):
    x = leaves(f, ("g",))
    out = dtg_chain(*x)
    x[1].add_(1.0)
    return torch.autograd.grad(out, x[0], f["w"])


def _stream(f):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        r = grad(leaves(f), f["w"])
    torch.cuda.current_stream().wait_stream(s)
    return r


def _checkpoint(f):
    from torch.utils.checkpoint import checkpoint
    x = leaves(f)
    checkpoint(dtg_chain, *x, use_reentrant=False).backward(f["w"])
    return [t.grad for t in x]


def _forward_ad(f):
    import torch.autograd.forward_ad as fa
    with fa.dual_level():
        x = [fa.make_dual(f[k].clone(), torch.ones_like(f[k])) for k in CHAIN]
        return dtg_chain(*x)


class _Sub(torch.Tensor):
    pass


AUTOGRAD = {
    "all": lambda f: grad(leaves(f), f["w"]),
    "some": lambda f: grad(leaves(f, ("beta", "alpha")), f["w"]),
    "subset_asked": lambda f: (lambda x: grad(x, f["w"], wrt=[x[4]]))(leaves(f)),
    "none": lambda f: dtg_chain(*[f[k] for k in CHAIN]),
    "no_grad": lambda f: torch.no_grad()(lambda: dtg_chain(*leaves(f)))(),
    "backward": lambda f: (lambda x: [dtg_chain(*x).backward(f["w"]), [t.grad for t in x]])(
        leaves(f)),
    "strided_cotangent": lambda f: grad(leaves(f), f["w"].T.contiguous().T),
    "expanded_cotangent": lambda f: (lambda x: [dtg_chain(*x).sum().backward(),
                                                [t.grad for t in x]])(leaves(f)),
    "second_derivative": _second,
    "create_graph_constant_w": lambda f: grad(leaves(f), f["w"], create_graph=True),
    "twice": _twice,
    "hooks": lambda f: _hooks(f, lambda t: t.clone()),
    "hooks_to_host": lambda f: _hooks(f, lambda t: t.cpu()),
    "in_place": _inplace,
    "side_stream": _stream,
    "checkpoint": _checkpoint,
    "batched_grads": lambda f: (lambda x: torch.autograd.grad(
        dtg_chain(*x), x, torch.stack([f["w"], f["w"]]), is_grads_batched=True))(leaves(f)),
    "forward_ad": _forward_ad,
    "func_grad": lambda f: torch.func.grad(lambda g: dtg_chain(g, *[f[k] for k in CHAIN[1:]]).sum())(
        f["g"]),
    "vmap": lambda f: torch.func.vmap(lambda g: dtg_chain(g, *[f[k] for k in CHAIN[1:]]))(
        torch.stack([f["g"], f["g"]])),
    "subclass": lambda f: dtg_chain(f["g"].as_subclass(_Sub), *[f[k] for k in CHAIN[1:]]
                                    ).as_subclass(torch.Tensor),
    "wrong_shape": lambda f: dtg_chain(f["dg"], *[f[k] for k in CHAIN[1:]]),
    "inference": lambda f: torch.inference_mode()(lambda: dtg_chain(*[f[k] for k in CHAIN]))(),
}


@pytest.mark.parametrize("flat_alpha", [False, True], ids=["alpha1n", "alphan"])
@pytest.mark.parametrize("name", list(AUTOGRAD))
def test_autograd(monkeypatch, name, flat_alpha):
    a, b = both(monkeypatch, lambda: lambda: AUTOGRAD[name](fields(flat_alpha=flat_alpha)))
    assert a == b


def test_plan_and_record(monkeypatch):
    """A plan runs through the extension; a call being recorded does not."""
    f = fields()

    def run():
        plan = BatchPlan([dict(f)])
        plan.run()
        torch.cuda.synchronize()
        out = plan.outputs[0].clone()
        plan.close()
        with ops.record() as calls:
            o = tl_dtg_chain(*[f[k] for k in CHAIN])
        assert len(calls) == 1
        calls[0]()
        return [out, o]
    a, b = both(monkeypatch, lambda: run)
    assert a == b


def test_large_grid_gradients_from_threads():
    """Backward passes of several threads at once, each with its own leaves."""
    import threading
    f = fields(n=70001)
    want = grad(leaves(f), f["w"])
    torch.cuda.synchronize()
    bad = []

    def work():
        for _ in range(10):
            got = grad(leaves(f), f["w"])
            torch.cuda.synchronize()
            if not all(torch.equal(a, b) for a, b in zip(got, want)):
                bad.append(1)
    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not bad and not any(t.is_alive() for t in threads)
