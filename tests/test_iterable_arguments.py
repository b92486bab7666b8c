"""``want``, ``grads`` and ``outs`` may be any iterable: a generator, the values of a
dict, an array.  On the CPU the calls get as far as refusing host tensors."""
import numpy as np
import pytest
import torch

from paper_1804_10120_amd import generated, tl_dtg_chain_bwd, tl_dtg_chain_fwd_bwd

NCOMP = {"g": 6, "dg": 18, "beta": 3, "dbeta": 9, "K": 6, "alpha": 1, "w": 6}
CHAIN = ("g", "dg", "beta", "dbeta", "K", "alpha", "w")
BWD = ("g", "dg", "beta", "K", "alpha", "w")
FORMS = {"tuple": tuple, "list": list, "generator": lambda v: (x for x in v), "iterator": iter,
         "map": lambda v: map(lambda x: x, v), "dict_values": lambda v: dict(enumerate(v)).values()}


def fields(device):
    gen = torch.Generator(device=device).manual_seed(5)
    f = {k: torch.rand(c, 70, dtype=torch.float64, device=device, generator=gen)
         for k, c in NCOMP.items()}
    f["g"][[0, 3, 5]] += 3.0
    return f


def calls(form, device):
    f = fields(device)
    w = (1, 0, 1, 0, 0, 1)

    def outs(sizes):
        return [torch.zeros(c, 70, dtype=torch.float64, device=device) for c in sizes]
    yield lambda: tl_dtg_chain_bwd(*[f[k] for k in BWD], want=form(w))
    yield lambda: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], want=form((1,) + w))
    yield lambda: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN],
                                       grads=form(outs((6, 18, 3, 9, 6, 1))))
    yield lambda: generated.call("kij", f["alpha"], f["g"], f["beta"], outs=form(outs((6,))))


def flat(r):
    return [x for v in r for x in (flat(v) if isinstance(v, tuple) else [v])]


@pytest.mark.parametrize("form", list(FORMS))
def test_host_tensors_are_refused(form):
    for call in calls(FORMS[form], "cpu"):
        with pytest.raises(ValueError, match="expected a HIP device tensor"):
            call()


def test_wrong_counts_are_refused():
    f = fields("cpu")
    with pytest.raises(ValueError):
        tl_dtg_chain_bwd(*[f[k] for k in BWD], want=(x for x in (1, 1)))
    with pytest.raises(TypeError, match="not iterable"):
        tl_dtg_chain_bwd(*[f[k] for k in BWD], want=3)


@pytest.mark.gpu
@pytest.mark.parametrize("form", list(FORMS) + ["array"])
def test_results(form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # an array of tensors is no field list: only want is given as one
    makers = calls((lambda v: np.array(v)) if form == "array" else FORMS[form], "cuda")
    for k, (call, ref) in enumerate(zip(makers, calls(tuple, "cuda"))):
        if form == "array" and k >= 2:
            break
        got, want = flat(call()), flat(ref())
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert (a is None and b is None) or torch.equal(a, b)
