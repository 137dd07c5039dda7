"""The fp32 decode kernel at the edges of its 16-token tiles, its four-wave rounds, the early start's 384 tokens and
the cuts, against the fp64 oracle at the fp32 bar; and what a row that is read again past a pair's end may not do."""
import numpy as np
import pytest

from test_gpu_parity import check, make_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LENS = np.array([[1, 15, 16, 17], [63, 64, 65, 0], [383, 384, 385, 400], [1000, 2049, 5, 31]], dtype=np.int32)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("plan", [dict(n_slots=3), dict(n_slots=16, policy=0), dict(n_slots=64),
                                  dict(n_slots=320, tile=16, min_chunk=16, overhead_tokens=0)])
def test_edges_of_tiles_rounds_and_cuts(D, G, plan):
    w, off, q, k, v = make_case(4, 4 * G, 4, D, "f32", LENS, seed=11 * D + G)
    _, layer = check(w, q, k, v, off, LENS, calls=2, **plan)
    if plan["n_slots"] == 320:
        assert layer.plan.items["n_chunks"].max() >= 32      # the two-level merge


@pytest.mark.parametrize("n", [1, 17, 33, 65])
def test_infinity_in_the_last_row_stays_in_its_coordinate(n):
    from paper_2502_15804_amd.runtime import DecodeLayer
    lens = np.full((1, 1), n, np.int32)
    w, off, q, k, v = make_case(1, 8, 1, 128, "f32", lens, seed=n)
    v[n - 1, 5] = float("inf")
    out, _ = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale).run()
    out = out.cpu()
    assert torch.isposinf(out[..., 5]).all()
    out[..., 5] = 0
    assert torch.isfinite(out).all()
