"""What a build needs of a machine and what it builds (no compiler is run here): the C library needs neither PyTorch nor the headers
of Python, and a binding belongs to one Python and one PyTorch."""
import importlib.util
import os
import shutil
import subprocess
import sysconfig

import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F
from paper_2502_15804_amd import build as B


@pytest.fixture
def commands(monkeypatch):
    """The commands of a build, none of which is run."""
    ran = []

    def run(cmd, **_):
        ran.append(cmd)
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(B.subprocess, "run", run)
    return ran


def _no_torch(monkeypatch):
    find = importlib.util.find_spec
    monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find(name, *a))
    monkeypatch.setitem(__import__("sys").modules, "torch", None)


def _no_headers(monkeypatch):
    monkeypatch.setattr(sysconfig, "get_paths", lambda *a: {"include": "/nowhere"})


def _no_compiler(monkeypatch):
    monkeypatch.delenv("CXX", raising=False)
    monkeypatch.setenv("PATH", "/nowhere")
    monkeypatch.setenv("HIPCC", "/nowhere/hipcc")


@pytest.mark.parametrize("take", [_no_torch, _no_headers, _no_compiler])
def test_the_library_is_built_without_what_the_binding_needs(monkeypatch, commands, capsys, take):
    take(monkeypatch)
    assert B.build() == B.LIB
    assert len(commands) == 1 and B.LIB in commands[0]
    assert "the Python binding is not" in capsys.readouterr().err


def test_both_are_built_here(commands):
    B.build()
    assert [B.LIB in commands[0], B.BINDING in commands[-1], len(commands)] == [True, True, 2]


def test_the_binding_that_cannot_be_compiled_is_an_error(monkeypatch):
    def run(cmd, **_):
        return subprocess.CompletedProcess(cmd, int(B.BINDING in cmd), "", "no such type")

    monkeypatch.setattr(B.subprocess, "run", run)
    with pytest.raises(RuntimeError, match="no such type"):
        B.build()


@pytest.fixture
def own_binding(monkeypatch, tmp_path):
    """A copy of the built binding, so that the one in use stays."""
    copy = str(tmp_path / "_binding.so")
    shutil.copyfile(B.BINDING, copy)
    monkeypatch.setattr(B, "BINDING", copy)
    return copy


def test_a_binding_for_another_pytorch_or_python_is_stale_and_not_loaded(monkeypatch, own_binding):
    monkeypatch.setattr(F, "_native_module", None)
    assert not B.binding_is_stale() and F._native()
    monkeypatch.setattr(F, "_native_module", None)
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", torch.__version__[:-1])      # what the version of the other starts with
        assert B.binding_is_stale()
        with pytest.raises(ImportError, match="another Python or PyTorch"):
            F._native()
    with monkeypatch.context() as m:
        m.setattr(sysconfig, "get_config_var", lambda name: "cpython-399-x86_64-linux-gnu")
        assert B.binding_is_stale()
        with pytest.raises(ImportError, match="another Python or PyTorch"):
            F._native()


def test_only_what_is_stale_is_built(monkeypatch, commands, own_binding):
    monkeypatch.setattr(B, "library_is_stale", lambda: False)
    B.build(force=False)
    assert commands == []
    os.utime(own_binding, (0, 0))
    B.build(force=False)
    assert len(commands) == 1 and own_binding in commands[0]
