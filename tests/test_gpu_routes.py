"""Sizes and alignments at the edges of the ranges in which a call without a launch shape runs one
kernel or another (default_path of tl_abi.cpp), against the kernel that stores from registers:
bitwise the same buffers, everything around the fields included."""
import pytest
import torch

from gpu_util import need_gpu
from paper_1804_10120_amd import generated, tl_dtg_chain_bwd, tl_dtg_chain_fwd_bwd, tl_expr
from test_gpu_staged import BWD, CHAIN, field, inputs, same, test_steps as steps

pytestmark = pytest.mark.gpu

# (n, leading-dimension padding or None for whole lines, offset): components on 16 bytes where n, the
# padding and the offset are even, the last blocks of a turn of 256 compute units among them
LAYOUTS = [(2 ** 18 - 8, 0, 0), (212992 + 8, 0, 2), (212992 - 8, 2, 0), (2 ** 19 - 8, 0, 4),
           (425984 + 8, 0, 0), (2 ** 17 - 1, 0, 1), (2 ** 17 + 1, 0, 0), (2 ** 17 + 2, 0, 0),
           (2 ** 20 + 8, 0, 0)]
IDS = [f"n{n}pad{p}off{o}" for n, p, o in LAYOUTS]


@pytest.mark.parametrize("lay", LAYOUTS, ids=IDS)
def test_steps(lay):
    steps(lay)


@pytest.mark.parametrize("want", [(1,) * 7, (0, 0, 0, 1, 0, 0, 1)], ids=["all", "some"])
@pytest.mark.parametrize("lay", LAYOUTS, ids=IDS)
def test_gradients(lay, want):
    need_gpu()
    f = inputs(CHAIN + ("w",), lay, seed=6)
    ncomps = [c if w else 0 for c, w in zip((6, 6, 18, 3, 9, 6, 1), want)]
    same(lambda o, t: tl_dtg_chain_bwd(*[f[k] for k in BWD], *o, want=want[1:], tune=t),
         ncomps[1:], lay)
    same(lambda o, t: tl_dtg_chain_fwd_bwd(*[f[k] for k in CHAIN], f["w"], o[0], o[1:], want=want,
                                           tune=t), ncomps, lay)


@pytest.mark.parametrize("name", ["assign1", "add1", "assign2", "kij", "contract1"])
@pytest.mark.parametrize("lay", LAYOUTS + [(7 * 2 ** 15, None, 0), (7 * 2 ** 15 + 16, None, 0),
                                           (2 ** 20 - 16, None, 0)],
                         ids=IDS + ["n229376lines", "n229392lines", "n1048560lines"])
def test_expressions(name, lay):
    need_gpu()
    gen = torch.Generator(device="cuda").manual_seed(7)
    p = generated.programs()[name]
    x = [field(t["ncomp"], lay, gen)[0] for t in p["inputs"]]
    nout = p["outputs"][0]["ncomp"]
    same(lambda o, t: tl_expr(name, *x, out=o[0], tune=t), [nout], lay)
    same(lambda o, t: generated.call(name, *x, outs=o, tune=t), [nout], lay)
