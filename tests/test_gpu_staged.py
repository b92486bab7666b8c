"""The kernels a call without a launch shape runs -- outputs staged through LDS on
large and on ragged grids, else one point per lane in blocks of 64, each with
the cache policies of its size -- against the kernels of a given shape, which
the parity tests hold to the oracle: the same bodies, so bitwise the same
buffers, everything around the fields included.  Sizes and layouts at the edges
of the rule and of the staged tiles (256 points, lines of 16 doubles)."""
import pytest
import torch

from gpu_util import CANARY, need_gpu
from paper_1804_10120_amd import (BatchPlan, generated, tl_batch_run_noalloc, tl_christoffel, tl_cov_deriv, tl_dtg,
                                  tl_dtg_chain, tl_dtg_chain_bwd, tl_dtg_chain_fwd_bwd, tl_expr,
                                  tl_sym_inverse)

pytestmark = pytest.mark.gpu

DIRECT = dict(block=256, ppt=1, nt=True)
NCOMP = {"g": 6, "dg": 18, "beta": 3, "dbeta": 9, "K": 6, "alpha": 1, "w": 6}
CHAIN = ("g", "dg", "beta", "dbeta", "K", "alpha")
BWD = ("g", "dg", "beta", "K", "alpha", "w")
# (n, leading-dimension padding or None for whole lines, offset of the field in its buffer)
LAYOUTS = [(2 ** 16, 1, 0), (2 ** 16 + 1, 0, 3), (2 ** 16 + 255, 13, 15), (2 ** 16 + 256, 8, 0),
           (2 ** 19 - 1, 0, 0), (2 ** 19, None, 0), (2 ** 19 + 17, None, 0), (2 ** 19 + 241, 7, 1),
           (2 ** 20, None, 0), (2 ** 20 + 1, None, 0), (2 ** 20 + 243, 1, 0),
           (98303, 0, 0), (98304, 1, 3), (163840, 1, 0), (2 ** 18, None, 0), (2 ** 18 + 1, None, 0)]
IDS = [f"n{n}pad{p}off{o}" for n, p, o in LAYOUTS]


def field(ncomp, lay, gen=None):
    """A [ncomp, n] view and the canary-filled buffer around it (inputs: uniform on [-1, 1])."""
    n, pad, off = lay
    ld = n + pad if pad is not None else -(-n // 16) * 16
    buf = torch.full((off + ncomp * ld + 64,), CANARY, dtype=torch.float64, device="cuda")
    view = buf[off:off + ncomp * ld].view(ncomp, ld)[:, :n]
    if gen is not None:
        view.copy_(torch.rand(ncomp, n, dtype=torch.float64, device="cuda", generator=gen) * 2 - 1)
    return view, buf


def inputs(names, lay, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    f = {k: field(NCOMP[k], lay, gen)[0] for k in names}
    if "g" in f:
        f["g"][[0, 3, 5]] += 4.0
    return f


def same(call, ncomps, lay):
    """Runs call(outputs, tune) with the default and from registers; compares the buffers."""
    got = []
    for tune in (None, DIRECT):
        outs = [field(c, lay) if c else (None, None) for c in ncomps]
        call([v for v, _ in outs], tune)
        got.append([b for _, b in outs if b is not None])
    torch.cuda.synchronize()
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), f"output {k}: {int((a != b).sum())} of {a.numel()} differ"


@pytest.mark.parametrize("lay", LAYOUTS, ids=IDS)
def test_steps(lay):
    need_gpu()
    f = inputs(("g", "dg", "beta", "dbeta", "K", "alpha"), lay)
    same(lambda o, t: tl_sym_inverse(f["g"], o[0], tune=t), [6], lay)
    same(lambda o, t: tl_christoffel(f["g"], f["dg"], o[0], tune=t), [18], lay)
    same(lambda o, t: tl_cov_deriv(f["dg"], f["beta"], f["dbeta"], o[0], tune=t), [9], lay)
    same(lambda o, t: tl_dtg(f["alpha"], f["K"], f["dbeta"], o[0], tune=t), [6], lay)


@pytest.mark.parametrize("want", [(1,) * 7, (0, 0, 1, 0, 0, 0, 1), (1, 1, 0, 1, 1, 1, 0)],
                         ids=["all", "dg_alpha", "some"])
@pytest.mark.parametrize("lay", LAYOUTS, ids=IDS)
def test_chain_and_gradients(lay, want):
    need_gpu()
    f = inputs(CHAIN + ("w",), lay, seed=1)
    if want[0]:
        same(lambda o, t: tl_dtg_chain(*[f[k] for k in CHAIN], o[0], tune=t), [6], lay)
    ncomps = [c if w else 0 for c, w in zip((6, 6, 18, 3, 9, 6, 1), want)]
    same(lambda o, t: tl_dtg_chain_bwd(*[f[k] for k in BWD], *o, want=want[1:], tune=t),
         ncomps[1:], lay)
    same(lambda o, t: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], f["w"], o[0], o[1:], want=want,
                                           tune=t), ncomps, lay)


@pytest.mark.parametrize("lay", [(777, 0, 1), (2 ** 16 + 9, 3, 0)], ids=["small", "staged"])
def test_every_subset_of_outputs(lay):
    """The inputs read for each subset of the outputs are all that it depends on."""
    need_gpu()
    f = inputs(CHAIN + ("w",), lay, seed=4)
    for bits in range(1, 128):
        want = [bits >> k & 1 for k in range(7)]
        ncomps = [c if w else 0 for c, w in zip((6, 6, 18, 3, 9, 6, 1), want)]
        same(lambda o, t: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], f["w"], o[0], o[1:],
                                               want=want, tune=t), ncomps, lay)
        if any(want[1:]):
            same(lambda o, t: tl_dtg_chain_bwd(*[f[k] for k in BWD], *o, want=want[1:], tune=t),
                 ncomps[1:], lay)


@pytest.mark.parametrize("name", ["assign1", "add3", "mult2", "mult3", "contract1", "contract2",
                                  "contract3", "kij"])
@pytest.mark.parametrize("lay", [LAYOUTS[1], LAYOUTS[2], LAYOUTS[6]], ids=[IDS[1], IDS[2], IDS[6]])
def test_expressions(name, lay):
    need_gpu()
    ins = {p: [t["ncomp"] for t in generated.programs()[p]["inputs"]] for p in generated.programs()}
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = [field(c, lay, gen)[0] for c in ins[name]]
    nout = generated.programs()[name]["outputs"][0]["ncomp"]
    same(lambda o, t: tl_expr(name, *x, out=o[0], tune=t), [nout], lay)
    same(lambda o, t: generated.call(name, *x, outs=o, tune=t), [nout], lay)


@pytest.mark.parametrize("name", ["mult3", "contract1", "contract2", "contract3"])
@pytest.mark.parametrize("lay", [(1, 0, 0), (65, 0, 3), (2 ** 15, 1, 0), (2 ** 15 + 1, 0, 0), (2 ** 16, None, 0),
                                 (2 ** 16 + 1, None, 0), (2 ** 16 - 1, 0, 0), (98304, None, 0),
                                 (98305, None, 0)],
                         ids=["n1", "n65", "n32768pad1", "n32769", "n65536lines", "n65537lines",
                              "n65535", "n98304lines", "n98305lines"])
def test_small_expressions(name, lay):
    """Up to 3/2 2^16 points a streaming body loads all its inputs before its first store."""
    test_expressions(name, lay)


@pytest.mark.parametrize("name", ["spacetime_split", "lst_fixed_offset", "dtg_chain_invg"])
def test_generated_several_fields(name):
    """Two output fields, an output with components that are never written, and many inputs."""
    need_gpu()
    lay, p = LAYOUTS[2], generated.programs()[name]
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = [field(t["ncomp"], lay, gen)[0] for t in p["inputs"]]
    same(lambda o, t: generated.call(name, *x, outs=o, tune=t), [t["ncomp"] for t in p["outputs"]],
         lay)


@pytest.mark.parametrize("kind", ["fwd", "bwd"])
@pytest.mark.parametrize("pad", [0, 1, None], ids=["contiguous", "pad1", "lines"])
def test_batch(kind, pad):
    """Subgrids of every remainder, an empty one, one of a single point, and one large enough
    for the rule's upper range, against a plan that stores from registers."""
    need_gpu()
    sizes = [0, 1, 15, 16, 17, 255, 256, 257, 1331, 65537, 2 ** 19 - 70000, 4097]
    names = CHAIN if kind == "fwd" else BWD
    outs = {"dtg": 6} if kind == "fwd" else {k + "_bar": NCOMP[k] for k in CHAIN}
    doms = [inputs(names, (n, pad, i % 3 if pad is not None else 0), seed=10 + i)
            for i, n in enumerate(sizes)]
    got = []
    for tune in (None, dict(block=128, ppt=1, nt=True)):
        made = [{k: field(c, (n, pad, 0)) for k, c in outs.items()} for n in sizes]
        plan = BatchPlan([dict(d, **{k: v for k, (v, _) in m.items()},
                               **({"W": d["w"]} if kind == "bwd" else {}))
                          for d, m in zip(doms, made)], tune=tune, kind=kind)
        plan.run()
        torch.cuda.synchronize()
        plan.close()
        got.append([b for m in made for _, b in m.values()])
    for k, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), f"field {k}: {int((a != b).sum())} of {a.numel()} differ"


@pytest.mark.parametrize("count", [1, 45, 46, 47, 93])
@pytest.mark.parametrize("pad", [0, None], ids=["contiguous", "lines"])
def test_batch_without_plan(count, pad):
    """Descriptors in the kernel arguments, 46 subgrids a launch, empty subgrids between them."""
    need_gpu()
    sizes = [0 if i % 5 == 3 else 1 + (i * 337) % 900 for i in range(count)]
    doms = [inputs(CHAIN, (n, pad, 0), seed=40 + i) for i, n in enumerate(sizes)]
    got = []
    for tune in (None, dict(block=128, ppt=1, nt=True)):
        made = [field(6, (n, pad, 0)) for n in sizes]
        tl_batch_run_noalloc([dict(d, dtg=v) for d, (v, _) in zip(doms, made)], tune=tune)
        torch.cuda.synchronize()
        got.append([b for _, b in made])
    assert all(torch.equal(a, b) for a, b in zip(*got))
