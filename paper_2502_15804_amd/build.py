"""Compile the HIP library in-tree for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfairkv.so")
BINDING = os.path.join(HERE, "_binding.so")
BINDING_SOURCE = os.path.join(CSRC, "binding.cpp")
SOURCES = [os.path.join(CSRC, "fairkv_api.hip"), os.path.join(CSRC, "fairkv_plan.cpp"),
           os.path.join(CSRC, "fairkv_place.cpp")]
HEADERS = [os.path.join(ROOT, "include", "fairkv.h"), os.path.join(ROOT, "include", "fairkv_measure.h")] + [os.path.join(CSRC, h) for h in ("common.h", "decode_f32.h", "decode_mfma.h", "decode_valu.h", "pack.h", "plan_check.h", "rows.h", "stream_probe.h")]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _older(out, inputs) -> bool:
    return not os.path.exists(out) or any(os.path.getmtime(f) > os.path.getmtime(out) for f in inputs)


def library_is_stale() -> bool:
    return _older(LIB, SOURCES + HEADERS)


def binding_is_stale() -> bool:
    return _older(BINDING, [BINDING_SOURCE] + HEADERS[:2]) or not binding_is_made_for_this()


def is_stale() -> bool:
    return library_is_stale() or (missing_for_binding() is None and binding_is_stale())


def _made_for() -> str:
    """The interpreter and the PyTorch whose objects the binding reads; numpy looks at its own version when it is loaded."""
    import torch
    return f"binding made for {sysconfig.get_config_var('SOABI')} and PyTorch {torch.__version__};"


def binding_is_made_for_this() -> bool:
    """Whether the binding that is built carries the versions of the running Python and PyTorch (its file is looked at, not loaded)."""
    with open(BINDING, "rb") as f:
        return _made_for().encode() in f.read()


def _compiler():
    """The host compiler of the binding: CXX, g++, or the one that comes with hipcc."""
    for name in (os.environ.get("CXX"), "g++", os.path.join(os.path.dirname(_hipcc()), "amdclang++")):
        if name and shutil.which(name):
            return name
    return None


def missing_for_binding():
    """What this machine lacks to build the native part of the Python binding, or None.  Callers of the C library need none of it."""
    if importlib.util.find_spec("torch") is None:
        return "PyTorch"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "the headers of Python"
    if _compiler() is None:
        return "a C++ compiler"
    return None


def build_binding() -> str:
    """The native part of the Python binding, against the PyTorch and numpy that import it."""
    import numpy
    import torch

    at = os.path.dirname(torch.__file__)
    cmd = [_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", f'-DMADE_FOR="{_made_for()}"', "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(at, "include"), "-isystem", numpy.get_include(), "-isystem", sysconfig.get_paths()["include"],
           BINDING_SOURCE, "-o", BINDING, "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("building the binding failed:\n" + res.stderr)
    return BINDING


def _build_library(verbose: bool) -> None:
    cmd = [_hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           # MFMA accumulators in ordinary vector registers: the softmax rescales them with vector
           # instructions, and the accumulation-register form costs a copy in and out per tile
           "-mllvm", "-amdgpu-mfma-vgpr-form=1",
           "-Wall", "-Wextra", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
           "-I", os.path.join(ROOT, "include"), "-x", "hip", *SOURCES, "-o", LIB]
    if verbose:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err:
        print(err)


def build(force: bool = True, verbose: bool = False) -> str:
    if force or library_is_stale():
        _build_library(verbose)
    missing = missing_for_binding()
    if missing is None:
        if force or binding_is_stale():
            build_binding()
    else:
        print(f"{LIB} is built, the Python binding is not: {missing} not found", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
