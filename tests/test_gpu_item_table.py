"""A slot's item list is walked in batches of 64 items, each fetched in halves of 32 (the vector-ALU kernel: item by item).  Slots of
300 items, i.e. five batches, and of just as many as fill a half or a batch, or one more: every element against the fp64 oracle for
every kind of cache, with empty pairs and pairs of 1 to 16 tokens on both sides of a batch's end (where some waves have no
tile), with short pairs (run by single waves) and without, two calls each."""
import numpy as np
import pytest

import workloads as W
from oracle import attention as OA
from test_gpu_parity import _kv8_case, make_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

B, HKV, SLOTS, BATCH = 75, 8, 2, 64


def _lens(short):
    rng = np.random.default_rng(31 + short)
    if not short:
        return rng.integers(97, 200, size=(B, HKV)).astype(np.int32)      # no pair that a single wave runs
    n = rng.integers(0, 130, size=B * HKV)
    for end in range(BATCH, 5 * BATCH, BATCH):      # pair i is item i // SLOTS of slot i % SLOTS when whole pairs are dealt in turn
        around = np.arange(SLOTS * (end - 9), SLOTS * (end + 9))
        n[around] = rng.integers(0, 17, size=around.size)
    return n.reshape(B, HKV).astype(np.int32)


def _two_calls(layer, want, tol):
    for _ in range(2):
        layer.out.fill_(float("nan"))
        layer.lse.fill_(float("nan"))
        layer.run()
        for got, ref in zip((layer.out, layer.lse), want):
            got = got.cpu().numpy().astype(np.float64)
            assert np.array_equal(np.isneginf(got), np.isneginf(ref))
            seen = np.isfinite(ref)
            assert np.abs(got[seen] - ref[seen]).max() <= tol


@pytest.mark.parametrize("policy", [0, 3])
@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("kind,D,G,q_len", [("bf16", 128, 4, 1), ("bf16", 128, 8, 2), ("bf16", 64, 8, 1), ("kv8", 128, 8, 1),
                                            ("kv8", 64, 2, 1), ("f32", 128, 8, 1), ("f32", 64, 1, 1), ("valu", 128, 2, 1)])
def test_five_batches_per_slot(kind, D, G, q_len, short, policy):
    import paper_2502_15804_amd as F
    from paper_2502_15804_amd.runtime import DecodeLayer
    lens, kv8 = _lens(short), kind == "kv8"
    if kv8:
        w, off, q, k, v, ks, vs = _kv8_case(B, HKV, G, lens, seed=G, D=D)
        want = OA.attention_kv8(W.to_numpy_bits(q), k.numpy(), v.numpy(), off, lens, w.scale, ks, vs)
    else:
        w, off, q, k, v = make_case(B, HKV * G, HKV, D, "f32" if kind == "f32" else "bf16", lens, seed=G, gap_rows=1)
        ks = vs = 1.0
        if q_len > 1:
            q = torch.randn((B, q_len, HKV * G, D), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16)
        attention = OA.attention_multi if q_len > 1 else OA.attention
        want = attention(W.to_numpy_bits(q), W.to_numpy_bits(k), W.to_numpy_bits(v), off, lens, w.scale)
    p = F.fairkv_default_params(256, n_slots=SLOTS, policy=policy)
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale, params=p, k_scale=ks, v_scale=vs,
                        bf16_on_valu=kind == "valu")
    assert np.diff(layer.plan.slot_ptr).max() > 4 * BATCH
    alone = (layer.plan.items["n_chunks"] == 1) & (layer.plan.items["tok_count"] <= F.FAIRKV_SHORT_PAIR_TOKENS)
    assert alone.any() == short
    _two_calls(layer, want, w.tol)


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("items", [31, 32, 33, 63, 64, 65, 96, 97, 128, 129])
@pytest.mark.parametrize("kind", ["bf16", "kv8", "f32"])
def test_lists_that_end_with_a_batch(kind, items, short):
    import paper_2502_15804_amd as F
    from paper_2502_15804_amd.runtime import DecodeLayer
    rng = np.random.default_rng(items + short)
    lens = (rng.integers(0, 130, size=(items, SLOTS)) if short else rng.integers(97, 130, size=(items, SLOTS))).astype(np.int32)
    if short:       # the last item of a list is one that a single wave runs, in one slot, and an empty one in the other
        lens[-1] = 5, 0
    if kind == "kv8":
        w, off, q, k, v, ks, vs = _kv8_case(items, SLOTS, 8, lens, seed=items)
        want = OA.attention_kv8(W.to_numpy_bits(q), k.numpy(), v.numpy(), off, lens, w.scale, ks, vs)
    else:
        w, off, q, k, v = make_case(items, SLOTS * 8, SLOTS, 128, kind, lens, seed=items, gap_rows=1)
        ks = vs = 1.0
        want = OA.attention(W.to_numpy_bits(q), W.to_numpy_bits(k), W.to_numpy_bits(v), off, lens, w.scale)
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale, params=F.fairkv_default_params(256, n_slots=SLOTS, policy=0),
                        k_scale=ks, v_scale=vs)
    assert np.diff(layer.plan.slot_ptr).tolist() == [items] * SLOTS      # whole pairs are dealt in turn
    _two_calls(layer, want, w.tol)
