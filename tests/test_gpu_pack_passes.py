"""fairkv_pack at the edges of its passes: a workgroup moves 8, 16 or 32 rows per pass (rows of 512, 256 or 128 bytes) and
four, two (from 321 slots on) or one (from 2049 on, on a cache this small) workgroups share an item's passes.  Byte for byte
what indexing gives."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,D", [(torch.float32, 128), (torch.bfloat16, 128), (torch.uint8, 128), (torch.bfloat16, 64)])
@pytest.mark.parametrize("n_slots", [1, 5, 64, 320, 321, 2048, 2049])
def test_passes_and_their_remainders(dtype, D, n_slots):
    import paper_2502_15804_amd as F
    B, H, T = 3, 5, 300
    lens = np.array([[1, 7, 8, 9, 15], [16, 17, 31, 32, 33], [63, 64, 65, 0, 257]], dtype=np.int32)
    rng = np.random.default_rng(D + n_slots)
    keep = [np.sort(rng.choice(T, int(n), replace=False)).astype(np.int32) for n in lens.reshape(-1)]
    ptr = np.concatenate([[0], np.cumsum(lens.reshape(-1))]).astype(np.int64)
    off = ptr[:-1] + 3 * np.arange(B * H)                                 # gaps: rows of no pair
    rows = int(off[-1] + lens[-1, -1] + 3)
    k, v = (torch.randint(0, 256, (B, H, T, D * torch.empty(0, dtype=dtype).element_size()), dtype=torch.uint8).view(dtype) for _ in "kv")
    plan = F.fairkv_plan(lens, off, B, H, F.fairkv_default_params(n_slots))
    got = [torch.full((rows, D), 7, dtype=dtype, device="cuda") for _ in "kv"]
    want = [torch.full((rows, D), 7, dtype=dtype) for _ in "kv"]
    for p in range(B * H):
        for w, x in zip(want, (k, v)):
            w[off[p]:off[p] + len(keep[p])] = x.reshape(B * H, T, D)[p][torch.from_numpy(keep[p]).long()]
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    F.fairkv_pack(k.cuda(), v.cuda(), torch.from_numpy(ptr).cuda(), torch.from_numpy(np.concatenate(keep)).cuda(),
                  torch.from_numpy(off).cuda(), torch.from_numpy(plan.items.view(np.uint8).copy()).cuda(),
                  torch.from_numpy(plan.slot_ptr).cuda(), *got, bad=bad)
    for g, w in zip(got, want):
        assert torch.equal(g.cpu().view(torch.uint8), w.view(torch.uint8))
    assert int(bad) == 0
