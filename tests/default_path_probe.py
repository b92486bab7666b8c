"""The launch rule of calls without a shape (default_path of tl_abi.cpp) on the host: compiled
from the library's source into a library of its own, whose launches stay unresolved."""
import ctypes
import os
import shutil
import subprocess
import tempfile

import pytest

from paper_1804_10120_amd import build

KERNELS = ("SymInverse", "Christoffel", "CovDeriv", "Dtg", "Chain", "ChainBwd", "ChainBatched",
           "ChainFwdBwd", "ChainBwdBatched", "ChainBatchedOnce", "Generic")
# components read and written
COMPS = {"SymInverse": (6, 6), "Christoffel": (24, 18), "CovDeriv": (30, 9), "Dtg": (16, 6),
         "Chain": (43, 6), "ChainBwd": (40, 43), "ChainFwdBwd": (49, 49),
         "ChainBatched": (43, 6), "ChainBwdBatched": (40, 43), "ChainBatchedOnce": (43, 6)}
PATHS = ("shape", "small", "staged")
KEEP = ("nothing", "inputs", "outputs")

SOURCE = """
#include "%s"
extern "C" void probe(int k, int64_t n, int align, int partial, int64_t in, int64_t out, int cus,
                      int* res) {
  Layout lay;
  lay.vec_ok = align >= 2;
  lay.line_ok = align >= 16;
  lay.partial = partial != 0;
  lay.in_bytes = in * 8 * n;
  lay.out_bytes = out * 8 * n;
  const tl::KernelId id = static_cast<tl::KernelId>(k);
  tl::Resolved r = defaults(id, n);
  r.num_cu = cus;
  default_path(id, lay, n, &r);
  res[0] = static_cast<int>(r.path);
  res[1] = r.block;
  res[2] = r.preload;
  res[3] = static_cast<int>(r.keep);
}
"""


class Rule:
    def __init__(self, lib):
        self.lib = lib

    def __call__(self, kernel, n, align=16, comps=None, partial=False, cus=256):
        """(path, block, preload, kept) of a call over n points; align: doubles that components
        are aligned to."""
        i, o = comps or COMPS[kernel]
        res = (ctypes.c_int * 4)()
        self.lib.probe(KERNELS.index(kernel), ctypes.c_int64(n), align, int(partial),
                       ctypes.c_int64(i), ctypes.c_int64(o), cus, res)
        return PATHS[res[0]], res[1], bool(res[2]), KEEP[res[3]]


def load():
    if shutil.which(build.HIPCC) is None:
        pytest.skip("no compiler")
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "probe.cpp"), os.path.join(d, "probe.so")
        with open(src, "w") as f:
            f.write(SOURCE % os.path.join(build.CSRC, "tl_abi.cpp"))
        r = subprocess.run([build.HIPCC, *build.COMMON, "-x", "hip", "-shared", src, "-o", so],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return Rule(ctypes.CDLL(so, mode=os.RTLD_LAZY | os.RTLD_LOCAL))
