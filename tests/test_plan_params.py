"""Which figures DecodeLayer plans with at the edges of its rules, and that a workspace of the size before pieces became larger holds a plan."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F
from paper_2502_15804_amd import runtime as R

N_CU, D = 256, 128


def _lens(tokens, pairs):
    """`pairs` pairs of `tokens` tokens in all, and an empty one."""
    n = np.full(pairs, tokens // pairs)
    n[: tokens % pairs] += 1
    return np.append(n, 0).astype(np.int32).reshape(-1, 1)


@pytest.mark.parametrize("kv8,f32,cols,tokens,pairs,min_chunk", [
    (True, False, 8, 64 * N_CU, 100, 64), (True, False, 16, 384 * N_CU, 100, 64),
    (False, False, 16, 384 * N_CU - 1, 100, 128), (False, False, 16, 384 * N_CU, 100, 256), (False, False, 16, 1000, 3, 64),
    (False, False, 8, 384 * N_CU, 100, 128), (False, False, 8, 128 * N_CU - 1, 100, 64), (False, False, 8, 128 * N_CU, 100, 128),
    (False, True, 8, 600 * N_CU - 1, 4 * N_CU, 32), (False, True, 8, 600 * N_CU, 4 * N_CU, 64), (False, True, 8, 600 * N_CU, 4 * N_CU + 1, 32)])
def test_smallest_pieces_at_the_edges(kv8, f32, cols, tokens, pairs, min_chunk):
    lens = _lens(tokens, pairs)
    p = R._plan_params(N_CU, kv8, f32, D, lens, cols)
    assert p.min_chunk == min_chunk and p.min_chunk % p.tile == 0
    plan = F.fairkv_plan(lens, np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])[:-1], len(lens), 1, p)
    cut = plan.items["n_chunks"] > 1
    assert not cut.any() or plan.items["tok_count"][cut].min() >= min_chunk


def _f32_layers():
    """Layers of which the present figures cut more pieces than those before."""
    for seed in range(4000):
        rng = np.random.default_rng(seed)
        lens = np.clip(np.rint(rng.integers(400, 2500) * np.exp(0.6 * rng.standard_normal((int(rng.integers(40, 120)), 2)))), 1, 8192).astype(np.int32)
        off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])[:-1].reshape(lens.shape)
        present, before = (F.fairkv_plan(lens, off, *lens.shape, R._plan_params(N_CU, False, True, D, lens, larger_pieces=larger))
                           for larger in (True, False))
        if present.n_parts > before.n_parts:
            yield lens, off, before


def test_a_workspace_of_the_size_before(monkeypatch):
    monkeypatch.setattr(R, "device_compute_units", lambda device=None: N_CU)
    lens, off, before = next(_f32_layers())
    room = F.fairkv_workspace_bytes(before.n_parts, lens.size, 8, D)
    q = torch.zeros((len(lens), 16, D))
    layer = R.DecodeLayer(q, torch.zeros((1, D)), torch.zeros((1, D)), off, lens, 1.0, workspace=torch.zeros(room, dtype=torch.uint8))
    assert np.array_equal(layer.plan.items, before.items)
