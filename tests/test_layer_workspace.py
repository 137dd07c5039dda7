"""A workspace of a given size that held a layer's plan holds it still, although DecodeLayer's present figures may cut more pieces."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F
from paper_2502_15804_amd import runtime as R

N_CU, D, G = 256, 128, 8
EARLIER = {"bf16": {}, "kv8": dict(tile=32, min_chunk=64, overhead_tokens=256, short_overhead_tokens=96),
           "f32": dict(overhead_tokens=80, short_overhead_tokens=32)}
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _layer(kind, lens, **more):
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])[:-1].reshape(lens.shape)
    q = torch.zeros((lens.shape[0], lens.shape[1] * G, D), dtype=DTYPE.get(kind, torch.bfloat16))
    k = torch.zeros((1, D), dtype=torch.uint8 if kind == "kv8" else q.dtype)      # planning reads no rows
    return R.DecodeLayer(q, k, k, off, lens, 1.0, **more)


def _need(plan, lens):
    return F.fairkv_workspace_bytes(plan.n_parts, lens.size, G, D)


def _earlier(kind, lens):
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])[:-1]
    return F.fairkv_plan(lens, off, *lens.shape, F.fairkv_default_params(N_CU, **EARLIER[kind]))


def _layers(kind):
    """Layers of which the present figures cut more pieces than the earlier ones did."""
    found = 0
    for seed in range(400):
        rng = np.random.default_rng(seed)
        shape = int(rng.integers(2, 120)), int(rng.choice([2, 4, 8]))
        lens = np.clip(np.rint(rng.integers(20, 400) * np.exp(0.6 * rng.standard_normal(shape))), 1, 8192).astype(np.int32)
        earlier = _earlier(kind, lens)
        if _layer(kind, lens).plan.n_parts > earlier.n_parts:
            found += 1
            yield lens, earlier
            if found == 3:
                return
    assert found, kind


@pytest.fixture(autouse=True)
def compute_units(monkeypatch):
    monkeypatch.setattr(R, "device_compute_units", lambda device=None: N_CU)


@pytest.mark.parametrize("kind", list(EARLIER))
def test_a_workspace_of_the_earlier_size(kind):
    for lens, earlier in _layers(kind):
        room = _need(earlier, lens)
        layer = _layer(kind, lens, workspace=torch.zeros(room, dtype=torch.uint8))
        assert np.array_equal(layer.plan.items, earlier.items)
        with pytest.raises(ValueError, match="too small"):
            _layer(kind, lens, workspace=torch.zeros(room - 1, dtype=torch.uint8))
        own = _layer(kind, lens)                                                  # its own workspace is as large as it needs
        assert own.plan.n_parts > earlier.n_parts and own.workspace.numel() == _need(own.plan, lens)


@pytest.mark.parametrize("B,mean", [(242, 60), (238, 100), (232, 200), (225, 500)])
def test_the_static_workspace(B, mean):
    """The earlier plan fits into the library's own workspace, the present one does not."""
    lens = np.clip(np.rint(mean * np.exp(0.6 * np.random.default_rng(B).standard_normal((B, 8)))), 1, 8192).astype(np.int32)
    earlier, room = _earlier("f32", lens), F.FAIRKV_STATIC_WORKSPACE_BYTES
    assert _need(earlier, lens) <= room < _need(_layer("f32", lens).plan, lens)
    assert np.array_equal(_layer("f32", lens, static_workspace=True).plan.items, earlier.items)


def test_given_parameters_are_kept():
    lens, earlier = next(_layers("f32"))
    p = F.fairkv_default_params(N_CU, overhead_tokens=64, short_overhead_tokens=32)
    with pytest.raises(ValueError, match="too small"):
        _layer("f32", lens, params=p, workspace=torch.zeros(_need(earlier, lens), dtype=torch.uint8))
