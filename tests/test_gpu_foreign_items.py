"""A device list that is not the host's: a kernel checks every item again and drops one that does not belong to the problem, also where the
sums of a check are more than its integers hold.  The other pairs get what they would have got."""
import numpy as np
import pytest

import paper_2502_15804_amd as F
import workloads as W
from test_gpu_parity import _kv8_case, make_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

B, HKV, G, D, BROKEN = 3, 2, 2, 128, 4
FAR, MANY = 2 ** 63 - 1, 2 ** 31 - 1


@pytest.mark.parametrize("wrong", [dict(row=FAR), dict(row=FAR - 5), dict(row=FAR, tok_count=MANY), dict(n_chunks=MANY), dict(n_chunks=2, part=MANY),
                                   dict(n_chunks=MANY, chunk=MANY - 1, part=MANY), dict(b=B), dict(h=HKV), dict(row=-1), dict(part=-1, chunk=-1)])
@pytest.mark.parametrize("kind", ["bf16", "kv8", "f32", "valu"])
def test_such_an_item_is_dropped(kind, wrong):
    from paper_2502_15804_amd.runtime import DecodeLayer
    lens = np.array([[40, 100], [130, 200], [70, 17]], np.int32)
    if kind == "kv8":
        w, off, q, k, v, ks, vs = _kv8_case(B, HKV, G, lens, seed=G, D=D)
    else:
        w, off, q, k, v = make_case(B, HKV * G, HKV, D, "f32" if kind == "f32" else "bf16", lens, seed=G)
        ks = vs = 1.0
    # all pairs whole, in one slot: nothing of the broken item is in the arguments of the launch
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale, params=F.fairkv_default_params(256, n_slots=1, min_chunk=4096),
                        k_scale=ks, v_scale=vs, bf16_on_valu=kind == "valu")
    assert len(layer.plan.items) == B * HKV and (layer.plan.items["n_chunks"] == 1).all()
    want = [x.clone() for x in layer.run()]
    items = layer.plan.items.copy()
    b, h = int(items["b"][BROKEN]), int(items["h"][BROKEN])
    for field, value in wrong.items():
        items[field][BROKEN] = value
    layer.items_d.copy_(torch.from_numpy(items.view(np.uint8).copy()))
    layer.out.fill_(7.0)
    layer.lse.fill_(7.0)
    layer.run()
    heads = slice(h * G, (h + 1) * G)
    want[0][b, heads] = 7.0
    want[1][b, heads] = 7.0
    assert torch.equal(layer.out, want[0]) and torch.equal(layer.lse, want[1])
