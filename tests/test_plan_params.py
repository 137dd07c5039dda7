"""What DecodeLayer plans with: pieces no larger than were found to keep an output's error, and, where a workspace of a given size holds no such
plan, those that it was planned with at other times.  test_layer_workspace.py has the workspaces of still earlier plans."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F
import workloads as W
from oracle import attention as OA
from paper_2502_15804_amd import runtime as R

N_CU, D = 256, 128
# with larger pieces (256 tokens) an output's error is 0.2 to 2 % larger
LARGE = {"equal": np.full((24, 8), 700), "in the middle": np.full((40, 8), 450),
         "ragged": np.rint(np.clip(700 * np.exp(0.6 * np.random.default_rng(4).standard_normal((24, 8))), 1, 8192)),
         "some of them short": np.rint(np.clip(700 * np.exp(1.2 * np.random.default_rng(5).standard_normal((24, 8))), 1, 8192))}


@pytest.fixture(autouse=True)
def compute_units(monkeypatch):
    monkeypatch.setattr(R, "device_compute_units", lambda device=None: N_CU)


def _layer(kind, cols, lens, **more):
    off = W.packed_offsets(lens)[0]
    dt = torch.float32 if kind == "f32" else torch.bfloat16
    q = torch.zeros((lens.shape[0], cols // 8, 8 * lens.shape[1], D) if cols > 8 else (lens.shape[0], cols * lens.shape[1], D), dtype=dt)
    k = torch.zeros((1, D), dtype=dt)      # planning reads no rows
    return R.DecodeLayer(q, k, k, off, lens, 1.0, **more)


@pytest.mark.parametrize("kind,cols,tokens,min_chunk", [
    ("bf16", 8, 128 * N_CU - 1, 64), ("bf16", 8, 128 * N_CU, 128), ("bf16", 16, 128 * N_CU - 1, 64), ("bf16", 16, 128 * N_CU, 128),
    ("bf16", 16, 384 * N_CU, 128), ("bf16", 16, 2000 * N_CU, 128), ("f32", 8, 600 * N_CU, 32), ("f32", 8, 2000 * N_CU, 32)])
def test_smallest_pieces(kind, cols, tokens, min_chunk):
    lens = np.full((10, 10), tokens // 100, np.int32)
    lens.reshape(-1)[: tokens % 100] += 1
    items = _layer(kind, cols, lens).plan.items
    assert min_chunk <= items["tok_count"][items["n_chunks"] > 1].min() < 2 * min_chunk


def _larger(lens):
    """The plan with larger pieces and the bytes that it needs."""
    short = dict(short_overhead_tokens=96) if (lens <= F.FAIRKV_SHORT_PAIR_TOKENS).any() else {}
    plan = F.fairkv_plan(lens, W.packed_offsets(lens)[0], *lens.shape, F.fairkv_default_params(N_CU, overhead_tokens=96, min_chunk=256, **short))
    return plan, F.fairkv_workspace_bytes(plan.n_parts, lens.size, 16, D)


@pytest.mark.parametrize("name", list(LARGE))
def test_a_workspace_that_held_larger_pieces(name):
    lens = LARGE[name].astype(np.int32)
    larger, room = _larger(lens)
    own = _layer("bf16", 16, lens)
    assert own.workspace.numel() > room and own.plan.n_parts > larger.n_parts
    layer = _layer("bf16", 16, lens, workspace=torch.zeros(room, dtype=torch.uint8))
    assert np.array_equal(layer.plan.items, larger.items)
    with pytest.raises(ValueError, match="too small"):
        _layer("bf16", 16, lens, workspace=torch.zeros(room - 1, dtype=torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("name", ["in the middle", "some of them short"])
def test_layers_of_16_columns_match_the_oracle(name, small):
    """As a layer plans by itself, and with the larger pieces of a smaller workspace; two calls each."""
    lens = LARGE[name].astype(np.int32)
    off, total = W.packed_offsets(lens)
    gen = torch.Generator().manual_seed(6)
    q, k, v = (torch.randn(shape, generator=gen).to(torch.bfloat16) for shape in ((len(lens), 2, 64, D), (total, D), (total, D)))
    larger, room = _larger(lens)
    layer = R.DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, D ** -0.5,
                          workspace=torch.zeros(room, dtype=torch.uint8, device="cuda") if small else None)
    assert np.array_equal(layer.plan.items, larger.items) == small
    want = OA.attention_multi(W.to_numpy_bits(q), W.to_numpy_bits(k), W.to_numpy_bits(v), off, lens, D ** -0.5)
    for _ in range(2):
        layer.out.fill_(float("nan"))
        layer.run()
        for got, ref in zip((layer.out, layer.lse), want):
            assert np.abs(got.cpu().numpy() - ref).max() <= W.WORKLOADS["llama70b"].tol
