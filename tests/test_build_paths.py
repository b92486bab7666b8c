"""The extension is compiled with the headers of the compiler that HIPCC names."""
import os

import pytest

from paper_1804_10120_amd import build


def tree(root):
    """A ROCm tree with a compiler and a HIP header."""
    (root / "bin").mkdir(parents=True)
    (root / "include" / "hip").mkdir(parents=True)
    (root / "include" / "hip" / "hip_runtime_api.h").write_text("")
    hipcc = root / "bin" / "hipcc"
    hipcc.write_text("#!/bin/sh\n")
    hipcc.chmod(0o755)
    return hipcc


class Stop(Exception):
    pass


def command(monkeypatch):
    """The extension's compile command."""
    seen = []

    def run(cmd, **kw):
        seen.append(cmd)
        raise Stop
    monkeypatch.setattr(build.subprocess, "run", run)
    with pytest.raises(Stop):
        build._compile_bind(False)
    return seen[0]


@pytest.mark.parametrize("form", ["path", "on_path", "symlink"])
def test_headers_follow_the_compiler(tmp_path, monkeypatch, form):
    hipcc = tree(tmp_path / "rocm-x")
    if form == "on_path":
        monkeypatch.setenv("PATH", str(hipcc.parent) + os.pathsep + os.environ["PATH"])
        hipcc = "hipcc"
    elif form == "symlink":
        link = tmp_path / "bin" / "hipcc"
        link.parent.mkdir()
        link.symlink_to(hipcc)
        hipcc = link
    monkeypatch.setattr(build, "HIPCC", str(hipcc))
    cmd = command(monkeypatch)
    assert cmd[cmd.index(str(tmp_path / "rocm-x" / "include")) - 1] == "-isystem"
    assert "/opt/rocm/include" not in cmd


def test_default(monkeypatch):
    monkeypatch.setattr(build, "HIPCC", "/nowhere/hipcc")
    assert "/opt/rocm/include" in command(monkeypatch)
