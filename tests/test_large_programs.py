"""Generated programs with fields of more than 255 components: the table of stores holds their
component numbers, and the call goes through the Python marshalling."""
import os
import re
import shutil
import subprocess

import pytest
import torch

from paper_1804_10120_amd import build, generated
from paper_1804_10120_amd.codegen import Program, Sum, Tensor, indices
from paper_1804_10120_amd.codegen.emit import _Emitter


@pytest.mark.parametrize("rank", [3, 4, 5])
def test_store_table_compiles(tmp_path, rank):
    """Rank-``rank`` tensors over four indices: 64, 256 and 1024 components."""
    idx = indices("a b c d e", 4)[:rank]
    A, B = Tensor("A", (4,) * rank), Tensor("B", (4,) * rank)
    p = Program("copy", "a copy").let(A[tuple(idx)], B[tuple(idx)])
    text = _Emitter(p).struct()
    tables = re.findall(r"  static constexpr int store_[fc]\(int k\) \{.*?\n  \}", text, re.S)
    assert len(tables) == 2
    n = 4 ** rank
    src = tmp_path / "t.cpp"
    src.write_text("struct T {\n" + "\n".join(tables) + "\n};\n"
                   f"static_assert(T::store_f({n - 1}) == 0 && T::store_c({n - 1}) == {n - 1}, "
                   "\"\");\n")
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", str(src)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[:500]


def test_call_reaches_the_argument_checks(monkeypatch):
    """A 256-component field is refused for its device, not for its size."""
    prog = {"big": {"inputs": [{"name": "B", "ncomp": 256}],
                    "outputs": [{"name": "A", "ncomp": 256}]}}
    monkeypatch.setattr(generated, "_programs", prog)
    monkeypatch.setattr(generated, "_plain", {})
    monkeypatch.setattr(generated, "_fns", {"big": generated._fn("kij")})
    with pytest.raises(ValueError, match="expected a HIP device tensor"):
        generated.call("big", torch.zeros(256, 3, dtype=torch.float64))


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no compiler")
def test_inputs_that_do_not_fit_registers_are_not_loaded_first(tmp_path):
    """A contraction of a rank-4 tensor over four indices reads 272 components; the library's own
    three contractions, 108, are loaded before the first store."""
    a, b, c, d, m = indices("a b c d m", 4)
    A, B, E = Tensor("A", (4,) * 4), Tensor("B", (4, 4)), Tensor("E", (4,) * 4)
    p = Program("big", "a contraction").let(A[a, b, c, d], Sum(m, B[a, m] * E[m, b, c, d]))
    src = tmp_path / "t.hip"
    src.write_text("#include <hip/hip_runtime.h>\n"
                   + "".join(f'#include "{os.path.join(build.CSRC, h)}"\n'
                             for h in ("tl_internal.hpp", "tl_expr_ops.hpp", "tl_stream.hpp"))
                   + "namespace tl {\n" + _Emitter(p).struct()
                   + 'static_assert(Gen_big::NIN == 272 && !preloads<Gen_big>(), "");\n'
                     'static_assert(preloads<OpContract<3>>() && !preloads<OpChain>(), "");\n}\n')
    r = subprocess.run([build.HIPCC, *build.COMMON, "-fsyntax-only", str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[:800]
