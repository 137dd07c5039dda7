"""What a decode call accepts as a plan: lists in the order of their partial slots are checked item by item, any other order by counting.
Both have to say the same, so every list is given in its own order and in another (CPU only: the element type is one that is refused,
which a call does after its look at the plan)."""
import ctypes

import numpy as np
import pytest

import paper_2502_15804_amd as F

B, HKV, HQ, D, N_ROWS = 5, 4, 8, 128, 6000


def _verdict(items, n_slots=1, q_len=1, n_parts=None):
    items = np.ascontiguousarray(items)
    slot_ptr = np.linspace(0, len(items), n_slots + 1).astype(np.int32)
    p = ctypes.c_void_p(1 << 20)      # never read: the call ends before
    rc = F.lib().fairkv_decode_attn_multi(p, p, p, N_ROWS, p, items.ctypes.data, len(items), slot_ptr.ctypes.data, n_slots,
                                          len(items) if n_parts is None else n_parts, p, 1 << 30, p, p, B, q_len, HQ, HKV, D, 99, F.FAIRKV_F32,
                                          0.1, None)
    return {F.FAIRKV_EINVAL: False, F.FAIRKV_EUNSUPPORTED: True}[rc]


def _plan(seed, **params):
    lens = np.random.default_rng(seed).integers(1, 280, (B, HKV)).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])[:-1]
    return F.fairkv_plan(lens, off, B, HKV, F.fairkv_default_params(32, tile=16, min_chunk=16, overhead_tokens=8, **params)).items


def _orders(items, seed):
    yield items
    yield items[::-1]
    yield items[np.random.default_rng(seed).permutation(len(items))]


@pytest.mark.parametrize("q_len", [1, 4])
@pytest.mark.parametrize("seed", range(4))
def test_whole_plans_pass_in_any_order(seed, q_len):
    items = _plan(seed)
    assert items["n_chunks"].max() > 1 and np.array_equal(items["part"], np.arange(len(items)))
    short = (items["n_chunks"] > 1) & (items["chunk"] == items["n_chunks"] - 1) & (items["tok_count"] < q_len - 1)
    for order in _orders(items, seed):
        assert _verdict(order, q_len=q_len) == (not short.any())
        assert _verdict(order, n_parts=len(items) + 7, q_len=q_len) == (not short.any())      # slots that no piece uses
        assert _verdict(order, n_slots=7, q_len=q_len) == (not short.any())


@pytest.mark.parametrize("field,values", [
    ("row", (-1, N_ROWS, N_ROWS + 1, 2 ** 62, -2 ** 63)), ("tok_count", (-1, N_ROWS + 1, 2 ** 31 - 1, -2 ** 31)),
    ("b", (-1, B, 2 ** 31 - 1, -2 ** 31)), ("h", (-1, HKV, 2 ** 31 - 1, -2 ** 31)), ("chunk", (-1, 1, 2, 3, 200, 2 ** 31 - 1, -2 ** 31)),
    ("n_chunks", (-1, 0, 2, 5, 200, 2 ** 31 - 1, -2 ** 31)), ("part", (-1, 0, 1, 5, 10 ** 6, 2 ** 31 - 1, -2 ** 31))])
def test_one_wrong_field_is_refused_in_any_order(field, values):
    items = _plan(1)
    for i in (0, 1, len(items) // 2, len(items) - 1):
        for value in values:
            wrong = items.copy()
            wrong[field][i] = value
            if wrong[field][i] == items[field][i] or (field == "row" and 0 <= value <= N_ROWS - items["tok_count"][i]):
                continue
            for order in _orders(wrong, i):
                assert not _verdict(order), (field, i, value)


@pytest.mark.parametrize("row", [2 ** 63 - 1, 2 ** 63 - N_ROWS, 2 ** 63 - 2 ** 31 + N_ROWS + 2])
@pytest.mark.parametrize("tokens", [1, N_ROWS, N_ROWS + 2, 2 ** 31 - 2, 2 ** 31 - 1])
def test_a_first_row_near_the_largest_number_is_refused_in_any_order(row, tokens):
    """The row behind the item, and the rows that are left in front of it, are numbers that 64 bits do not hold."""
    items = _plan(1)
    for i in (0, len(items) // 2, len(items) - 1):
        wrong = items.copy()
        wrong["row"][i], wrong["tok_count"][i] = row, tokens
        for order in _orders(wrong, i):
            assert not _verdict(order), i


@pytest.mark.parametrize("seed", range(3))
def test_missing_doubled_and_swapped_pieces_are_refused(seed):
    items = _plan(seed)
    for i in range(len(items)):
        if items["n_chunks"][i] > 1:
            for order in _orders(np.delete(items, i), i):
                assert not _verdict(order, n_parts=len(items))
        for order in _orders(np.insert(items, i, items[i]), i):
            assert not _verdict(order)


def test_shorter_last_pieces_than_the_rows_that_new_tokens_hide():
    items = _plan(2)
    last = np.flatnonzero((items["n_chunks"] > 1) & (items["chunk"] == items["n_chunks"] - 1))[0]
    items["tok_count"][last] = 2
    for order in _orders(items, 2):
        assert [_verdict(order, q_len=n) for n in (1, 2, 3, 4)] == [True, True, True, False]
