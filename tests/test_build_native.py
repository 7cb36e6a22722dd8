"""When and where the binding's native half is built (host only; the compiler is not run)."""
import importlib
import os
import subprocess

import pytest
import torch

from paper_2506_06266_amd import build as installed


@pytest.fixture
def build(tmp_path, monkeypatch):
    monkeypatch.setenv("CART_LIB_OUT", str(tmp_path / "out" / "libcartridge.so"))
    monkeypatch.setenv("CART_OBJ_DIR", str(tmp_path / "obj"))
    (tmp_path / "out").mkdir()
    (tmp_path / "obj").mkdir()
    b = importlib.reload(installed)
    b.runs = []

    def run(cmd, **kw):
        b.runs.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(b.subprocess, "run", run)
    yield b
    monkeypatch.undo()
    importlib.reload(installed)


def test_goes_beside_the_library(build, tmp_path):
    assert build._compile_pycall(True) == str(tmp_path / "out" / "_pycall.so") == build.runs[0][build.runs[0].index("-o") + 1]


def test_is_built_again_for_another_pytorch_or_command(build, monkeypatch):
    for _ in range(2):
        build._compile_pycall(False)
    assert len(build.runs) == 1             # (nothing changed)
    monkeypatch.setattr(torch, "__version__", "0.0.0+other")
    for _ in range(2):
        build._compile_pycall(False)
    assert len(build.runs) == 2
    monkeypatch.setattr(build.sysconfig, "get_config_var", lambda name: "cpython-999")
    for _ in range(2):
        build._compile_pycall(False)
    assert len(build.runs) == 3
    monkeypatch.setenv("CXX", "another-compiler")
    build._compile_pycall(False)
    assert len(build.runs) == 4
    os.utime(build.PYCALL, (0, 0))          # a newer source
    build._compile_pycall(False)
    assert len(build.runs) == 5


def test_its_own_warnings_are_shown(build):
    build._compile_pycall(True)
    assert "-w" not in build.runs[0] and "-Wall" in build.runs[0]
