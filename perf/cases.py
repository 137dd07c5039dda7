"""The work a user of this library has it do, as cases that can be timed and checked.

A case is a decode step's attention over the layers of a model (one call per layer over that layer's packed
ragged cache), the gathering of a compressed cache, or a decode step that appends its new rows and attends.
Sizes are those of the repository's own workloads (workloads.py, bench.py) or generic ones; the per-head
budgets, the cache contents and the queries are drawn from the seed with the same distributions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2502_15804_amd as F
from paper_2502_15804_amd.runtime import DecodeLayer, device_compute_units

DEV = "cuda"
SCALE8 = (0.02, 0.03)        # what a stored byte of an 8-bit K and V cache is multiplied by, as in bench.py
RECENT = 32                  # most recent tokens that a per-head compressor always keeps


def _case(name, op, dtype, B, Hq, Hkv, D, budgets, mean, layers, graph, out="f32", q_len=1, T=0):
    c = dict(op=op, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, D=D, budgets=budgets, mean=mean, layers=layers, graph=graph,
             out=out, q_len=q_len, T=T)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: two short sequences, fp32, one call: a unit test's or a toy model's size; launch and latency.
        _case("tiny_f32", "decode", "f32", 2, 8, 4, 64, "uniform128", 64, 1, False),
        # One user alone on the GPU: eight pairs cut over the whole chip, the step captured in a graph as a server does.
        _case("single_sequence_bf16", "decode", "bf16", 1, 64, 8, 128, "lognormal", 1024, 8, True, "bf16"),
        # The headline: a 70B model's layer, batch 16, lognormal budgets; eight layers of a captured decode step.
        _case("llama70b_bf16", "decode", "bf16", 16, 64, 8, 128, "lognormal", 1024, 8, True),
        # A 24B model's layer, two of eight KV heads heavy; outputs in bf16 as the next projection wants them.
        _case("mistral24b_bf16", "decode", "bf16", 32, 32, 8, 128, "heavy", 512, 4, True, "bf16"),
        # One GPU's share under Fair-Copying: a full head and a replicated heavy head for half of the batch.
        _case("faircopy_bf16", "decode", "bf16", 64, 16, 2, 128, "replica", 2048, 4, True),
        # Many short pairs and a few very long ones: Pareto budgets at batch 128.
        _case("stress_bf16", "decode", "bf16", 128, 64, 8, 128, "pareto", 32, 8, True),
        # The largest: a full batch of equal budgets, called layer by layer from Python.
        _case("large_uniform_bf16", "decode", "bf16", 256, 64, 8, 128, "equal", 1024, 2, False, "bf16"),
        # The fp32 mode on a model's shape: what reference runs and accuracy checks of a compressor use.
        _case("llama70b_f32", "decode", "f32", 16, 64, 8, 128, "lognormal", 1024, 4, False),
        # The cache stored as 8-bit floats with a scale per KV head.
        _case("llama70b_kv8", "decode", "kv8", 16, 64, 8, 128, "lognormal", 1024, 8, True, "bf16"),
        # Verification of a draft of four tokens per sequence.
        _case("verify4_bf16", "decode", "bf16", 32, 32, 8, 128, "heavy", 512, 4, True, "bf16", q_len=4),
        # After a prompt: the kept rows of one layer's dense cache are gathered into the packed layout.
        _case("pack_bf16", "pack", "bf16", 16, 64, 8, 128, "lognormal", 1024, 1, False, T=8192),
        # An eager decode step of a small model at an odd batch: append the new rows, attend over the grown cache.
        _case("append_attend_bf16", "append", "bf16", 13, 32, 8, 64, "lognormal", 700, 8, False, "bf16"),
    ]


def draw(rng):
    """One more case of the same ranges: every operation, type, group size and head size, sizes spread over their logarithm."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["decode", "decode", "decode", "decode", "pack", "append"])
    dtype = rng.choice(["bf16", "bf16", "f32", "kv8"]) if op == "decode" else rng.choice(["bf16", "bf16", "f32"])
    D = rng.choice([64, 128, 128])
    G = rng.choice([1, 2, 4, 8])
    Hkv = rng.choice([1, 2, 4, 8])
    q_len = rng.choice([1, 1, 1] + [n for n in (2, 4, 8) if G * n <= 16]) if op == "decode" and dtype != "f32" else 1
    B = log_int(1, 200)
    budgets = rng.choice(["lognormal", "lognormal", "heavy", "pareto", "equal"])
    # tokens per layer: from about a thousand to the largest listed case's, no more than its cost
    most = min(4096, max(24, 1_400_000 // (B * Hkv)))
    mean = 32 if budgets == "pareto" else log_int(24, most)
    if budgets == "heavy":
        mean = max(16, mean // 3)
    T = 0
    if op == "pack":
        T = max(64, min(8192, 2 * mean + rng.randrange(0, 500), 2_000_000 // (B * Hkv)))
        mean = min(mean, max(16, T // 3))
        budgets = "lognormal"
    tokens = B * Hkv * (mean if budgets != "pareto" else 160)
    layers = 1 if op == "pack" else max(1, min(6, 400_000 // max(1, tokens)))
    graph = op == "decode" and rng.random() < 0.6
    return _case(None, op, dtype, B, G * Hkv, Hkv, D, budgets, mean, layers, graph, rng.choice(["f32", "bf16"]), q_len, T)


# ---- inputs -------------------------------------------------------------------------------------------
def _lens(case, seed, layer):
    """Tokens that every (sequence, KV head) pair of a layer keeps, int32 [B][Hkv].  The budgets are the case's own, so
    that every seed is the same amount of work; the seed says which sequence has which."""
    rng = np.random.default_rng([layer, 7])
    deal = np.random.default_rng([int(seed), layer, 11])
    B, H, mean, kind = case["B"], case["Hkv"], case["mean"], case["budgets"]

    def lognormal(m, hi):
        return np.clip(np.rint(m * np.exp(0.6 * rng.standard_normal((B, H)) - 0.18)), 16, hi)

    if kind == "uniform128":
        n = rng.integers(1, 129, (B, H))
    elif kind == "lognormal":
        n = lognormal(mean, 8192)
    elif kind == "heavy":                            # KV heads 2 and 5 of eight keep eight times as much
        n = lognormal(mean, 16384)
        heavy = lognormal(8 * mean, 16384)
        n[:, 2::3] = heavy[:, 2::3]
    elif kind == "replica":                          # the second head: heavy, served for the upper half of the batch only
        n = lognormal(mean, 32768)
        n[:, 1] = lognormal(3 * mean, 32768)[:, 1]
        n[: B // 2, 1] = 0
    elif kind == "pareto":
        n = np.clip(np.floor(mean * rng.random((B, H)) ** (-1 / 1.2)), mean, 32768)
    else:
        n = np.full((B, H), mean)
    if case["T"]:
        n = np.minimum(n, case["T"])
    if kind in ("heavy", "replica"):                 # a heavy head stays heavy
        for h in range(H):
            rows = slice(B // 2 if kind == "replica" and h == 1 else 0, B)
            n[rows, h] = deal.permutation(n[rows, h])
    else:
        n = deal.permutation(n.reshape(-1)).reshape(B, H)
    return np.ascontiguousarray(np.maximum(n, 0 if kind == "replica" else case["q_len"]), dtype=np.int32)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _randn(shape, gen, dt):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dt)


def _gen(seed, layer):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + layer * 7919 + 4242) & 0x7FFFFFFF)
    return g


def _scales(case):
    h = np.arange(case["Hkv"])
    return [float(SCALE8[0] * (1 + 0.1 * i)) for i in h], [float(SCALE8[1] * (1 - 0.05 * i)) for i in h]


def _decode_inputs(case, seed, layer):
    """lens, off, q, k, v of one layer; an 8-bit cache as the bytes of torch.float8_e4m3fn."""
    lens, dt, g = _lens(case, seed, layer), _dtype(case), _gen(seed, layer)
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])
    rows, B, Hq, D = max(1, int(off[-1])), case["B"], case["Hq"], case["D"]
    q = _randn((B, case["q_len"], Hq, D) if case["q_len"] > 1 else (B, Hq, D), g, dt)
    k, v = _randn((rows, D), g, dt), _randn((rows, D), g, dt)
    if case["dtype"] == "kv8":
        k, v = ((x.float() / s).clamp(-448, 448).to(torch.float8_e4m3fn) for x, s in ((k, SCALE8[0]), (v, SCALE8[1])))
    return lens, off[:-1].reshape(lens.shape), q, k, v


def _append_inputs(case, seed, layer):
    """A cache whose pairs have eight rows to spare, and the new rows of one step."""
    lens, dt, g = _lens(case, seed, layer), _dtype(case), _gen(seed, layer)
    cap = lens + 8
    off = np.concatenate([[0], np.cumsum(cap.reshape(-1).astype(np.int64))])
    B, H, D = case["B"], case["Hkv"], case["D"]
    q = _randn((B, case["Hq"], D), g, dt)
    k, v = _randn((int(off[-1]), D), g, dt), _randn((int(off[-1]), D), g, dt)
    k_new, v_new = _randn((B, H, D), g, dt), _randn((B, H, D), g, dt)
    return lens, cap, off[:-1].reshape(lens.shape), q, k, v, k_new, v_new


def _pack_inputs(case, seed):
    """A dense cache and the ascending positions that each pair keeps: the most recent ones and a scattered rest."""
    lens, g = _lens(case, seed, 0), _gen(seed, 0)
    B, H, T, D = case["B"], case["Hkv"], case["T"], case["D"]
    k, v = _randn((B, H, T, D), g, _dtype(case)), _randn((B, H, T, D), g, _dtype(case))
    n = torch.from_numpy(lens.reshape(-1, 1).astype(np.int64)).to(DEV)
    key = torch.rand((B * H, T), generator=g, device=DEV)
    key[:, max(0, T - RECENT):] = -1.0
    rank = key.argsort(dim=1, stable=True).argsort(dim=1)
    keep_t = (rank < n).nonzero()[:, 1].to(torch.int32).contiguous()
    off = np.concatenate([[0], np.cumsum(lens.reshape(-1).astype(np.int64))])
    return lens, off, k, v, keep_t


def _out_dtype(case):
    return torch.bfloat16 if case["out"] == "bf16" else torch.float32


def prepare(case, seed):
    if case["op"] == "pack":
        lens, off, k, v, keep_t = _pack_inputs(case, seed)
        plan = F.fairkv_plan(lens, off[:-1], case["B"], case["Hkv"], F.fairkv_default_params(device_compute_units()))
        rows = int(off[-1])
        return {"op": "pack", "args": (k, v, torch.from_numpy(off).to(DEV), keep_t, torch.from_numpy(off[:-1].copy()).to(DEV),
                                       torch.from_numpy(plan.items.view(np.uint8).copy()).to(DEV),
                                       torch.from_numpy(plan.slot_ptr).to(DEV),
                                       torch.empty((rows, case["D"]), dtype=k.dtype, device=DEV),
                                       torch.empty((rows, case["D"]), dtype=k.dtype, device=DEV))}
    scale = 1.0 / math.sqrt(case["D"])
    state = {"op": case["op"], "layers": [], "graph": None}
    for i in range(case["layers"]):
        if case["op"] == "append":
            lens, cap, off, q, k, v, k_new, v_new = _append_inputs(case, seed, i)
            # the plan of the lengths before the step, grown by the step's row on the host as the step goes
            layer = DecodeLayer(q, k, v, off, lens, scale, out_dtype=_out_dtype(case))
            n_host = lens.reshape(-1).copy()
            F.fairkv_plan_grow(layer.plan.items, case["B"], case["Hkv"], n_host, cap.reshape(-1).copy())
            layer.items_d.copy_(torch.from_numpy(layer.plan.items.view(np.uint8).copy()))
            dev = [torch.from_numpy(x).to(DEV) for x in (off.reshape(-1), lens.reshape(-1), lens.reshape(-1).copy(), cap.reshape(-1))]
            state["layers"].append((layer, k_new, v_new, *dev))
        else:
            lens, off, q, k, v = _decode_inputs(case, seed, i)
            scales = dict(zip(("k_scale", "v_scale"), _scales(case))) if case["dtype"] == "kv8" else {}
            state["layers"].append(DecodeLayer(q, k, v, off, lens, scale, out_dtype=_out_dtype(case), **scales))
    if case["graph"]:                                # the decode step is captured once and replayed for every token
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for layer in state["layers"]:
                layer.run()
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for layer in state["layers"]:
                layer.run()
    return state


def run(state):
    if state["op"] == "pack":
        F.fairkv_pack(*state["args"])
        return state["args"][-2:]
    if state["op"] == "append":
        got = []
        for layer, k_new, v_new, off, n0, n, cap in state["layers"]:
            n.copy_(n0)                              # the last step's token was refused: back to the lengths before it
            F.fairkv_append(k_new, v_new, off, n, cap, layer.k, layer.v)
            got.append((*layer.run(), n, layer.k, layer.v))
        return got
    if state["graph"] is not None:
        state["graph"].replay()
        return [(layer.out, layer.lse) for layer in state["layers"]]
    return [layer.run() for layer in state["layers"]]


# ---- what a pass cannot do without, and what it should give ----------------------------------------------
def work(case):
    elem = {"bf16": 2, "f32": 4, "kv8": 1}[case["dtype"]]
    D, q_rows = case["D"], case["B"] * case["q_len"] * case["Hq"]
    total = {"bytes": 0, "flops": 0}
    for i in range(case["layers"]):
        tokens = int(_lens(case, 0, i).astype(np.int64).sum())
        if case["op"] == "pack":                     # an index and two rows in, two rows out
            total["bytes"] += tokens * (4 + 4 * D * elem)
            continue
        if case["op"] == "append":                   # a row of K and of V in and out, the lengths in and out
            pairs = case["B"] * case["Hkv"]
            total["bytes"] += pairs * (4 * D * elem + 8)
            tokens += pairs
        total["bytes"] += 2 * tokens * D * elem + q_rows * D * (4 if case["dtype"] == "f32" else 2)
        total["bytes"] += q_rows * (D * (2 if case["out"] == "bf16" else 4) + 4)
        total["flops"] += 4 * tokens * case["Hq"] // case["Hkv"] * case["q_len"] * D
    return total


def tolerance(case):
    if case["op"] == "pack":
        return "exact"
    if case["dtype"] == "f32":
        # fp32 sums in another order; a bf16 output adds its own rounding
        return {"rel": 2e-6} if case["out"] == "f32" else {"rel": 8e-3, "max": 0.1}
    # softmax weights rounded to bf16 (2**-9 each, against one another and against the largest weight seen so far)
    return {"rel": 8e-3, "max": 0.1}


def exact(case, seed):
    if case["op"] == "pack":
        return None                                  # bytes are moved, nothing is computed
    got = []
    for i in range(case["layers"]):
        if case["op"] == "append":
            lens, cap, off, q, k, v, k_new, v_new = _append_inputs(case, seed, i)
            last = torch.from_numpy((off + lens).reshape(-1)).to(DEV)
            k[last], v[last] = k_new.reshape(-1, case["D"]), v_new.reshape(-1, case["D"])
            out, lse = _attend(case, lens + 1, off, q, k, v)
            got.append((out, lse, None, None, None))
        else:
            got.append(_attend(case, *_decode_inputs(case, seed, i)))
    return got


def _attend(case, lens, off, q, k, v):
    B, n_q, Hq, Hkv, D = case["B"], case["q_len"], case["Hq"], case["Hkv"], case["D"]
    G = Hq // Hkv
    ks, vs = _scales(case) if case["dtype"] == "kv8" else ([1.0] * Hkv, [1.0] * Hkv)
    q4 = q.reshape(B, n_q, Hq, D)
    out = torch.zeros((B, n_q, Hq, D), dtype=torch.float64, device=DEV)
    lse = torch.full((B, n_q, Hq), -math.inf, dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(Hkv):
            n, r = int(lens[b, h]), int(off[b, h])
            if n == 0:
                continue
            cols = q4[b, :, h * G:(h + 1) * G].reshape(n_q * G, D).double()
            kd, vd = k[r:r + n].double() * ks[h], v[r:r + n].double() * vs[h]
            s = (cols @ kd.t()) / math.sqrt(D)
            for t in range(n_q - 1):                 # new token t does not see the rows of the new tokens after it
                s[t * G:(t + 1) * G, n - (n_q - 1 - t):] = -math.inf
            m = torch.logsumexp(s, dim=1)
            out[b, :, h * G:(h + 1) * G] = (torch.exp(s - m[:, None]) @ vd).reshape(n_q, G, D)
            lse[b, :, h * G:(h + 1) * G] = m.reshape(n_q, G)
    shape = tuple(q.shape)
    return out.reshape(shape), lse.reshape(shape[:-1])
