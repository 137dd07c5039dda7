"""A pair in few pieces, in as many as the two-level merge starts with (16), in whole groups of 8 and one more or less:
every element against the fp64 oracle, and the counters left at zero by every call."""
import numpy as np
import pytest

import workloads as W
from oracle import attention as OA
from test_gpu_parity import _kv8_case, _kv8_check, check, make_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 8), ("bf16", 64, 1), ("f32", 128, 4)])
@pytest.mark.parametrize("pieces", [8, 9, 15, 16, 17, 23, 24, 25, 33])
def test_pieces_around_the_groups(dtype, D, G, pieces):
    lens = np.full((1, 1), 48 * pieces, np.int32)
    w, off, q, k, v = make_case(1, G, 1, D, dtype, lens, seed=pieces)
    _, layer = check(w, q, k, v, off, lens, calls=3, n_slots=pieces, tile=16, min_chunk=16, overhead_tokens=0)
    assert layer.plan.items["n_chunks"].max() == pieces


@pytest.mark.parametrize("G,D,q_len", [(8, 128, 1), (8, 128, 2), (1, 64, 1)])
@pytest.mark.parametrize("pieces", [15, 16, 17, 24, 31])
def test_pieces_around_the_groups_of_an_8_bit_cache(G, D, q_len, pieces):
    lens = np.full((1, 1), 96 * pieces, np.int32)
    w, off, q, k8, v8, ks, vs = _kv8_case(1, 1, G, lens, seed=pieces, q_len=q_len, D=D)
    layer = _kv8_check(w, off, lens, q, k8, v8, ks, vs, n_slots=pieces, tile=32, min_chunk=32, overhead_tokens=0)
    assert layer.plan.items["n_chunks"].max() == pieces


@pytest.mark.parametrize("G,D,q_len", [(8, 128, 2), (4, 128, 4), (8, 64, 2)])
@pytest.mark.parametrize("pieces", [15, 16, 17, 24, 31])
def test_pieces_around_the_groups_with_16_columns(G, D, q_len, pieces):
    # D = 128: a thread merges two columns
    import paper_2502_15804_amd as F
    from paper_2502_15804_amd.runtime import DecodeLayer
    lens = np.full((1, 1), 48 * pieces, np.int32)
    w, off, _, k, v = make_case(1, G, 1, D, "bf16", lens, seed=pieces)
    q = torch.randn((1, q_len, G, D), generator=torch.Generator().manual_seed(pieces)).to(torch.bfloat16)
    want = OA.attention_multi(W.to_numpy_bits(q), W.to_numpy_bits(k), W.to_numpy_bits(v), off, lens, w.scale)
    p = F.fairkv_default_params(256, n_slots=pieces, min_chunk=16, overhead_tokens=0)
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale, params=p)
    assert layer.plan.items["n_chunks"].max() == pieces
    counters = F.fairkv_workspace_counter_bytes(1)
    for _ in range(3):
        layer.out.fill_(float("nan"))
        layer.workspace[counters:].fill_(0xFF)
        layer.run()
        for got, ref in zip((layer.out, layer.lse), want):
            assert np.abs(got.cpu().numpy() - ref).max() <= w.tol
        assert int(layer.workspace[:counters].count_nonzero()) == 0
