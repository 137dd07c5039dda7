"""The binding asks PyTorch for the current stream by a name that is not public: without it the calls still check their
arguments, and still enqueue on the caller's current stream."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F


@pytest.fixture
def without_the_name(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(F, "_pt", None)


def test_a_host_tensor_is_refused_by_name(without_the_name):
    q, k = torch.zeros((1, 8, 128)), torch.zeros((4, 128))
    with pytest.raises(ValueError, match="q must be a contiguous device tensor"):
        F.fairkv_decode_attn(q, k, k, k, np.zeros(1, F.ITEM_DTYPE), np.zeros(2, np.int32), 1, k, q, None, 1.0, 1)
    with pytest.raises(ValueError, match="k_new must be a contiguous device tensor"):
        F.fairkv_append(k[None], k[None], k, k, k, k, k)


@pytest.mark.gpu
def test_the_current_stream_is_found(without_the_name):
    t = torch.zeros(1, device="cuda")
    F._torch()
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            assert F._stream(None, t) == stream.cuda_stream
        assert F._stream(stream, t) == stream.cuda_stream
