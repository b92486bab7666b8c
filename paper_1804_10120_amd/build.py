"""Builds ``libtl.so`` (the C-ABI library of HIP kernels) for gfx950 in-tree, and
``_bind.so``, the torch binding's extension.

    python -m paper_1804_10120_amd.build

The library is compiled with hipcc for gfx950 only.  Packed FP32 instructions
are disabled (all arithmetic here is FP64 anyway).  The compiler's per-kernel
resource report (VGPRs, SGPRs, scratch, occupancy) is written beside the
objects in ``_build/resource_usage.txt``.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libtl.so")
BIND = os.path.join(PKG, "_bind.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["tl_kernels.hip", "tl_noalloc.hip", "tl_expr.hip", "generated/tlg_kernels.hip",
           "tl_abi.cpp"]
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.splitext(os.path.basename(src))[0] + ".o")
    cmd = [HIPCC, *COMMON, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".hip"):
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    return src, obj, r


def _rocm_include():
    """The HIP headers that belong to the compiler (HIPCC), else /opt/rocm's."""
    found = shutil.which(HIPCC)
    for root in ([os.path.dirname(os.path.dirname(p)) for p in (found, os.path.realpath(found))]
                 if found else []):
        inc = os.path.join(root, "include")
        if os.path.exists(os.path.join(inc, "hip", "hip_runtime_api.h")):
            return inc
    return "/opt/rocm/include"


def _compile_bind(verbose):
    """The torch binding's extension (csrc/py_bind.cpp): host code only."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    tmp = BIND + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", os.path.join(t, "include"),
           "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-isystem", _rocm_include(), "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "py_bind.cpp"), "-o", tmp, "-L", os.path.join(t, "lib"),
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("the torch binding's extension did not compile")
    os.replace(tmp, BIND)


_REMARK = re.compile(r"remark: +(Function Name|TotalSGPRs|VGPRs|AGPRs|ScratchSize \[bytes/lane\]|"
                     r"Occupancy \[waves/SIMD\]): (\S+)")
_FIELDS = ("TotalSGPRs", "VGPRs", "AGPRs", "ScratchSize [bytes/lane]", "Occupancy [waves/SIMD]")


def resource_table(report: str):
    """{mangled kernel name: (SGPRs, VGPRs, AGPRs, scratch bytes per lane, waves
    per SIMD)} from the compiler's kernel-resource-usage remarks."""
    table, name, cur = {}, None, {}
    for m in _REMARK.finditer(report):
        key, val = m.group(1), m.group(2)
        if key == "Function Name":
            name, cur = val, {}
        elif name is not None:
            cur[key] = int(val)
            if all(f in cur for f in _FIELDS):
                table[name] = tuple(cur[f] for f in _FIELDS)
                name = None
    return table


def _demangled(names):
    try:
        r = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                           check=True)
        out = r.stdout.split("\n")
        return out[:len(names)] if len(out) >= len(names) else [None] * len(names)
    except (OSError, subprocess.CalledProcessError):
        return [None] * len(names)


def write_resource_source(table, path):
    """A C++ translation unit holding the resource table, looked up by
    tl_kernel_info by the kernel's mangled (or demangled) name."""
    names = sorted(table)
    dem = _demangled(names)
    rows = []
    for n, d in zip(names, dem):
        for key in {n, d} - {None, ""}:
            rows.append((key, table[n]))
    rows.sort()
    with open(path, "w") as f:
        f.write("// Generated by build.py from the compiler's resource-usage report.\n"
                "#include <cstring>\n\n#include \"tl_internal.hpp\"\n\nnamespace tl {\n"
                "namespace {\nstruct Row {\n  const char* name;\n  KernelResources r;\n};\n"
                "const Row kRows[] = {\n")
        for key, v in rows:
            f.write(f'    {{"{key}", {{{v[0]}, {v[1]}, {v[2]}, {v[3]}, {v[4]}}}}},\n')
        f.write("};\n}  // namespace\n\n"
                "bool kernel_resources(const char* name, KernelResources* out) {\n"
                "  if (name == nullptr) return false;\n"
                "  size_t lo = 0, hi = sizeof(kRows) / sizeof(kRows[0]);\n"
                "  while (lo < hi) {\n"
                "    const size_t mid = (lo + hi) / 2;\n"
                "    const int c = std::strcmp(kRows[mid].name, name);\n"
                "    if (c == 0) {\n      *out = kRows[mid].r;\n      return true;\n    }\n"
                "    if (c < 0) lo = mid + 1;\n    else hi = mid;\n  }\n  return false;\n}\n\n"
                "}  // namespace tl\n")


def build(verbose: bool = False) -> str:
    """Regenerates the generated kernels from the registry, compiles every
    translation unit (in parallel), compiles the kernels' resource table from
    the compiler's report, and links libtl.so."""
    from .codegen.__main__ import main as codegen
    codegen([])
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as pool:
        bind = pool.submit(_compile_bind, verbose)
        results = list(pool.map(lambda s: _compile(s, verbose), SOURCES))
        bind.result()
    objs, report = [], []
    for src, obj, r in results:
        report.append(r.stderr)
        if r.returncode != 0:
            sys.stderr.write(r.stderr)
            raise RuntimeError(f"hipcc failed on {src}")
        objs.append(obj)
    res_src = os.path.join(BUILD, "tl_resources.cpp")
    write_resource_source(resource_table("".join(report)), res_src)
    res_obj = os.path.join(BUILD, "tl_resources.o")
    r = subprocess.run([HIPCC, *COMMON, "-x", "hip", "-c", res_src, "-o", res_obj],
                       capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("hipcc failed on the resource table")
    objs.append(res_obj)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    with open(os.path.join(BUILD, "resource_usage.txt"), "w") as f:
        f.write("".join(report))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
