"""The native part of the binding refuses what the library cannot take, by the argument's name (no GPU: nothing gets as far as
a launch), and lets PyTorch's own errors through."""
import ctypes
import os
import subprocess
import sys
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F

Q, K = torch.zeros((1, 8, 128)), torch.zeros((4, 128))
ITEMS, SLOTS = np.zeros(1, F.ITEM_DTYPE), np.zeros(2, np.int32)


def decode(q=Q, k=K, v=K, items=K, workspace=K, out=Q, lse=None, **more):
    F.fairkv_decode_attn(q, k, v, items, ITEMS, SLOTS, 1, workspace, out, lse, 1.0, 1, **more)


@pytest.mark.parametrize("change,error,words", [
    (dict(q="q"), TypeError, "q must be a tensor"), (dict(workspace=3), TypeError, "workspace must be a tensor"),
    (dict(q=Q.double()), TypeError, "share bf16 or fp32"), (dict(v=K.bfloat16()), TypeError, "share bf16 or fp32"),
    (dict(out=Q.int()), TypeError, "out must be bf16 or fp32"), (dict(), ValueError, "q must be a contiguous device tensor"),
    (dict(stream=torch.cuda.Stream), ValueError, "q must be")])
def test_decode(change, error, words):
    with pytest.raises(error, match=words):
        decode(**change)


def test_the_others():
    byte, wide = K.to(torch.uint8), Q.bfloat16()
    for args, error, words in (((Q, byte, byte), TypeError, "q must be bf16"), ((wide, K, byte), TypeError, "k8/v8"),
                               ((wide, byte, byte), ValueError, "q must be a contiguous device tensor")):
        with pytest.raises(error, match=words):
            F.fairkv_decode_attn_kv8(*args, 1.0, [1.0], K, ITEMS, SLOTS, 1, K, Q, None, 1.0, 1)
    with pytest.raises(ValueError, match=r"k_new must be \[B, Hkv, D\]"):
        F.fairkv_append(K, K, K, K, K, K, K)
    with pytest.raises(ValueError, match="k_dense must be a contiguous device tensor"):
        F.fairkv_pack(Q[None], Q[None], K, K, K, K, K, K, K)
    with pytest.raises(TypeError, match="16 arguments"):
        F._native().decode(Q)


def test_a_program_keeps_its_own_module_of_that_name():
    program = ("import sys, types; sys.modules['_binding'] = mine = types.ModuleType('_binding'); import paper_2502_15804_amd as F; F._native(); "
               "assert sys.modules['_binding'] is mine")
    subprocess.run([sys.executable, "-c", program], cwd=os.path.dirname(os.path.dirname(F.__file__)), check=True)


@pytest.mark.parametrize("Hkv", [1.0, 1.7, "1", None, np.float32(1)])
def test_the_number_of_heads_is_an_integer(Hkv):
    byte, wide = K.to(torch.uint8), Q.bfloat16()
    with pytest.raises(TypeError, match="cannot be interpreted as an integer"):
        F.fairkv_decode_attn(Q, K, K, K, ITEMS, SLOTS, 1, K, Q, None, 1.0, Hkv)
    with pytest.raises(TypeError, match="cannot be interpreted as an integer"):
        F.fairkv_decode_attn_kv8(wide, byte, byte, 1.0, 1.0, K, ITEMS, SLOTS, 1, K, Q, None, 1.0, Hkv)


@pytest.mark.parametrize("Hkv", [1, True, np.int64(1), np.uint8(1), torch.tensor(1)])
def test_any_integer_is_a_number_of_heads(Hkv):
    with pytest.raises(ValueError, match="q must be a contiguous device tensor"):
        F.fairkv_decode_attn(Q, K, K, K, ITEMS, SLOTS, 1, K, Q, None, 1.0, Hkv)


@pytest.mark.gpu
@pytest.mark.parametrize("scale", ["0.5", np.array(0.5), torch.tensor(0.5), np.float32(0.5)])
@pytest.mark.parametrize("form", [int, ctypes.c_void_p, lambda s: None])
def test_what_a_scale_and_a_stream_may_be(scale, form):
    """A scale is whatever float() takes; a stream has a cuda_stream, which is a number, a pointer of ctypes or None."""
    from paper_2502_15804_amd.runtime import DecodeLayer
    from test_gpu_parity import make_case
    w, off, q, k, v = make_case(1, 4, 2, 64, "bf16", np.array([[33, 90]], np.int32), seed=1)
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, np.array([[33, 90]], np.int32), 0.5)
    want = [t.clone() for t in layer.run()]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    layer.scale = scale
    layer.out.zero_(), layer.lse.zero_()
    torch.cuda.synchronize()
    layer.run(stream=types.SimpleNamespace(cuda_stream=form(side.cuda_stream)))
    torch.cuda.synchronize()
    assert torch.equal(layer.out, want[0]) and torch.equal(layer.lse, want[1])
    with pytest.raises(AttributeError):
        layer.run(stream=types.SimpleNamespace(cuda_stream="7"))
    with pytest.raises(TypeError):
        layer.run(stream=types.SimpleNamespace(cuda_stream=ctypes.c_double(0.0)))
