"""What fairkv_decode_attn_kv8 takes as a scale: a number in any of its forms, or one per KV head; also one of each."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
import paper_2502_15804_amd as F

HKV = 2
NUMBERS = [0.5, 1, True, "0.5", np.float32(0.5), np.float64(0.5), np.int32(2), np.array(0.5), np.array(0.5, np.float32), np.array(2),
           np.float64([0.25, 0.5])[1:].reshape(()), torch.tensor(0.5), torch.tensor(0.5, dtype=torch.float64), np.array("0.5")]
PER_HEAD = [[0.5, 0.25], (1, 2), np.array([0.5, 0.25]), np.array([0.5, 0.25], np.float32), np.array([0.5, 0.25, 1.0, 2.0], np.float32)[::2],
            np.array([0.5], np.float32), torch.tensor([0.5, 0.25]), np.array([0.5, 0.25], ">f4")]


def _kind(x):
    return f"{type(x).__name__}-{getattr(x, 'dtype', '')}-{np.ndim(x)}"


def wanted(scale):
    """The numbers that a scale stands for, one per KV head, in fp32."""
    return np.broadcast_to(np.asarray(scale, dtype=np.float32) if np.ndim(scale) else np.float32(float(scale)), (HKV,))


@pytest.mark.parametrize("v_scale", [0.125, np.array(0.125), [0.125, 2.0]], ids=_kind)
@pytest.mark.parametrize("k_scale", NUMBERS + PER_HEAD, ids=_kind)
def test_what_the_native_part_is_given(monkeypatch, k_scale, v_scale):
    class Recorder:
        def decode_8bit(self, *args):
            self.k, self.v, self.per_head = args[4], args[5], args[16]
            return F.FAIRKV_OK

    got = Recorder()
    monkeypatch.setattr(F, "_native_module", got)
    F.fairkv_decode_attn_kv8(*[None] * 3, k_scale, v_scale, *[None] * 7, 1.0, HKV)
    assert got.per_head == bool(np.ndim(k_scale) or np.ndim(v_scale))
    for scale, given in ((k_scale, got.k), (v_scale, got.v)):
        if got.per_head:
            assert type(given) is np.ndarray and given.dtype == np.float32 and given.dtype.isnative and given.flags.c_contiguous and given.shape == (HKV,)
        else:
            assert type(given) is float
        assert np.array_equal(np.broadcast_to(np.float32(given), (HKV,)), wanted(scale))


ONES = np.ones(HKV, np.float32)


@pytest.mark.parametrize("k_scale,v_scale,per_head", [
    (ONES, ONES, False), (ONES, 1.0, True), (1.0, ONES, True), (1.0, 1.0, True), (ONES.astype(np.float64), ONES, True), (ONES, ONES[:1], True),
    (np.ones(4, np.float32)[::2], ONES, True), (ONES, ONES[None], True), (np.array(1.0, np.float32), ONES, True), (ONES, [1.0, 1.0], True),
    (ONES.astype(">f4"), ONES, True), (None, 1.0, False)])
def test_what_the_native_part_refuses(k_scale, v_scale, per_head):
    q = torch.zeros((1, 8, 128), dtype=torch.bfloat16)
    k = torch.zeros((4, 128), dtype=torch.uint8)
    with pytest.raises(TypeError):
        F._native().decode_8bit(F._torch()[1], q, k, k, k_scale, v_scale, k, np.zeros(1, F.ITEM_DTYPE), np.zeros(2, np.int32), 1, k, q, None, 1.0,
                                HKV, None, per_head)


@pytest.mark.gpu
@pytest.mark.parametrize("v_scale", [0.125, np.array(0.125), [0.125, 2.0]], ids=_kind)
@pytest.mark.parametrize("k_scale", NUMBERS + PER_HEAD + [pytest.param("device tensor", id="device tensor")], ids=_kind)
def test_every_form_gives_the_same(k_scale, v_scale):
    from paper_2502_15804_amd.runtime import DecodeLayer
    from test_gpu_parity import _kv8_case
    lens = np.array([[5, 40], [70, 1]], np.int32)
    w, off, q, k, v, _, _ = _kv8_case(2, HKV, 4, lens, seed=3, D=64)
    if isinstance(k_scale, str) and k_scale == "device tensor":
        k_scale = torch.tensor(0.5, device="cuda")
    layer = DecodeLayer(q.cuda(), k.cuda(), v.cuda(), off, lens, w.scale)
    args = layer.items_d, layer.plan.items, layer.plan.slot_ptr, layer.plan.n_parts, layer.workspace

    def run(ks, vs):
        out, lse = torch.full_like(layer.out, float("nan")), torch.full_like(layer.lse, float("nan"))
        F.fairkv_decode_attn_kv8(layer.q, layer.k, layer.v, ks, vs, *args, out, lse, w.scale, HKV)
        return out.cpu(), lse.cpu()

    # a scale for all heads and the same one for each of them may round differently: in lists only if it was one
    want = [float(x) for x in wanted(k_scale.cpu() if isinstance(k_scale, torch.Tensor) else k_scale)], [float(x) for x in wanted(v_scale)]
    if not np.ndim(k_scale) and not np.ndim(v_scale):
        want = want[0][0], want[1][0]
    if isinstance(k_scale, torch.Tensor) and k_scale.is_cuda and np.ndim(v_scale):      # numpy does not read device memory
        with pytest.raises(TypeError):
            run(k_scale, v_scale)
        return
    for got, ref in zip(run(k_scale, v_scale), run(*want)):
        assert torch.equal(got, ref)
