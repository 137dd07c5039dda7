"""A pair in few pieces, in as many as the two-level merge starts with (16), in whole groups of 8 and one more or less:
every element against the fp64 oracle, and the counters left at zero by every call."""
import numpy as np
import pytest

from test_gpu_parity import check, make_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 8), ("bf16", 64, 1), ("f32", 128, 4)])
@pytest.mark.parametrize("pieces", [8, 9, 15, 16, 17, 23, 24, 25, 33])
def test_pieces_around_the_groups(dtype, D, G, pieces):
    lens = np.full((1, 1), 48 * pieces, np.int32)
    w, off, q, k, v = make_case(1, G, 1, D, dtype, lens, seed=pieces)
    _, layer = check(w, q, k, v, off, lens, calls=3, n_slots=pieces, tile=16, min_chunk=16, overhead_tokens=0)
    assert layer.plan.items["n_chunks"].max() == pieces
