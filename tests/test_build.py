"""What the build needs of a machine (nothing is compiled here but the binding): the C library needs neither PyTorch nor the
headers of Python."""
import importlib.util
import subprocess
import sysconfig

import pytest

pytest.importorskip("torch")
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
