"""Device-side plumbing around the C ABI: keeps one layer's tensors and plan resident.

Nothing here computes: it allocates torch tensors, copies the host plan to the device
once, and forwards to fairkv_decode_attn.  Budgets are static after compression (the
paper's scheme is a static, load-aware one: Section 4.1), so a layer is planned once
and the plan is reused for every decode step.
"""
from __future__ import annotations

import numpy as np

from . import (FAIRKV_SHORT_PAIR_TOKENS, FAIRKV_STATIC_WORKSPACE_BYTES, Plan, fairkv_decode_attn, fairkv_decode_attn_kv8, fairkv_default_params, fairkv_plan,
               fairkv_workspace_bytes)


def device_compute_units(device=None) -> int:
    import torch
    return int(torch.cuda.get_device_properties(device if device is not None else torch.cuda.current_device())
               .multi_processor_count)


def _plan_params(n_cu, kv8, f32, D, lens):
    """The planner's parameters for a layer that brings none: the library's defaults with what was measured for the kind of cache.

    The overheads are what an item costs in units of streamed tokens, so they fall with the bytes of a token; the values are
    measured, not scaled.  us per layer with the overhead of an item and of a short whole pair in tokens:

                                      bf16 160/48   96/48   |  fp32 80/32   64/32  |  8-bit 256/96  256/128
      Llama-70B shape                       16.04   16.01   |       28.89   28.49  |         11.05    11.08
      24B shape, two heavy heads            33.19   32.87   |       65.81   65.12  |         20.55    20.55
      Pareto budgets, batch 128             20.76   20.87   |       39.12   38.49  |         16.80    16.66
      128 pairs of 60 (8-bit: 120) tokens       -       -   |        8.67    8.69  |          7.78     7.28
      1024 pairs of 60 (fp32: 40) tokens    13.11   12.62   |       17.50   15.98  |             -        -
      256 pairs of 64 tokens                 7.32    4.90   |        7.38    7.37  |          6.85     6.83

    The smallest piece of a bf16 pair: a smaller one fills more compute units and makes more partials to merge.  us per layer
    with pieces of at least 32, 64, 96 and 128 tokens: one sequence of eight pairs of 1024 tokens 9.35, 8.75, 8.76, 8.92, of 256
    6.82, 6.33, 6.85, 6.50, of 200 on the average 7.57, 7.00, 6.94, 7.31; Pareto budgets at batch 8 9.33, 9.31, 9.52, 9.52 and at
    batch 128 21.62, 21.37, 21.16, 21.09; 24B shape 33.76, 33.53, 33.55, 33.47; with D = 64, where a token is half the bytes, one
    sequence 8.87, 8.69, 8.53, 8.37 and the Llama-70B shape 11.34, 11.18, 11.08, 11.09.  Hence 64 up to 128 tokens per compute unit.

    With no more pairs than compute units a short pair costs what any item costs: two of them on one unit leave another idle.
    us per layer with the short pairs' own overhead and without: 256 pairs of 64 tokens on an 8-bit cache 7.49 and 5.33, of 40 on
    the average 8.34 and 6.15 (bf16 7.53 and 6.90), 200 of 100 8.48 and 7.53 (8.41 and 7.58), 64 of 90 6.98 and 7.04 (6.97 and 7.01);
    with 384 pairs of 50 8.62 and 8.72 (8.87 and 9.08), with 512 of 64 7.91 and 7.59 (8.33 and 8.38).  On an fp32 cache it is the
    other way round: 200 pairs of 30 8.14 and 8.81, 256 of 40 9.24 and 9.57."""
    if f32:      # twice the bytes
        return fairkv_default_params(n_cu, overhead_tokens=64, short_overhead_tokens=32)
    if kv8:      # half the bytes per token, and a step covers 32 tokens
        p = fairkv_default_params(n_cu, tile=32, min_chunk=64, overhead_tokens=256, short_overhead_tokens=128)
    else:
        p = fairkv_default_params(n_cu, overhead_tokens=96,
                                  min_chunk=64 if D == 128 and int(lens.sum(dtype=np.int64)) < 128 * n_cu else 128)
    if np.count_nonzero(lens) <= n_cu and ((lens > 0) & (lens <= FAIRKV_SHORT_PAIR_TOKENS)).any():      # (empty pairs alone: 0.6 % slower)
        p.short_overhead_tokens = p.overhead_tokens
    return p


def _other_plan_params(n_cu, kv8, f32, D, lens, cols):
    """What layers were planned with at other times.  The plans of _plan_params may need more partial slots than these (against the
    first, fp32: up to 143 more over 1500 random layers, bf16 5, 8-bit 13), so a workspace of a given size that held a layer's plan still
    has one to hold.  The last makes larger pieces of large layers with 16 columns: up to a fifth faster with equal budgets, but an output's
    error is up to 2 % larger, so such plans serve workspaces that hold no other."""
    if kv8:
        yield fairkv_default_params(n_cu, tile=32, min_chunk=64, overhead_tokens=256, short_overhead_tokens=96)
    elif f32:
        yield fairkv_default_params(n_cu, overhead_tokens=80, short_overhead_tokens=32)
    else:
        yield fairkv_default_params(n_cu)
        if cols == 16 and int(lens.sum(dtype=np.int64)) >= 384 * n_cu:
            p = _plan_params(n_cu, kv8, f32, D, lens)
            p.min_chunk = 256
            yield p


class DecodeLayer:
    """One layer's packed ragged KV cache, its plan and its output buffers on the GPU."""

    def __init__(self, q, k, v, off, lens, scale, params=None, out_dtype=None, want_lse=True,
                 workspace=None, k_scale=1.0, v_scale=1.0, static_workspace=False, bf16_on_valu=False):
        import torch

        dev = q.device
        self.q, self.k, self.v = q, k, v
        self.kv8 = k.dtype in (torch.uint8, torch.float8_e4m3fn)   # a cache of 8-bit floats, one scale per tensor
        self.k_scale = k_scale if np.ndim(k_scale) else float(k_scale)     # a number, or one per KV head
        self.v_scale = v_scale if np.ndim(v_scale) else float(v_scale)
        self.q_len = q.shape[1] if q.dim() == 4 else 1     # several new tokens per sequence: q [B,q_len,Hq,D]
        self.B, self.Hq, self.D = q.shape[0], q.shape[-2], q.shape[-1]
        lens_h = np.ascontiguousarray(np.asarray(lens, dtype=np.int32))
        off_h = np.ascontiguousarray(np.asarray(off, dtype=np.int64))
        self.Hkv = lens_h.shape[1]
        self.G = self.Hq // self.Hkv
        self.scale = float(scale)
        given = params is not None
        if not given:
            kind = device_compute_units(dev), self.kv8, q.dtype == torch.float32, self.D, lens_h
            params = _plan_params(*kind)
        room = FAIRKV_STATIC_WORKSPACE_BYTES if static_workspace else None if workspace is None else workspace.numel()

        def plan_and_need(params):
            plan = fairkv_plan(lens_h, off_h, self.B, self.Hkv, params)
            return plan, fairkv_workspace_bytes(plan.n_parts, self.B * self.Hkv, self.G * self.q_len, self.D)

        plan, need = plan_and_need(params)
        for other in () if given or room is None else _other_plan_params(*kind, self.G * self.q_len):
            if need > room:
                plan, need = plan_and_need(other)
        self.plan: Plan = plan
        self.items_d = torch.from_numpy(self.plan.items.view(np.uint8).copy()).to(dev)
        self.bf16_on_valu = bf16_on_valu
        if static_workspace:
            workspace = None                                               # the library's own (fairkv_decode_attn_static)
        elif workspace is None:
            workspace = torch.zeros(need, dtype=torch.uint8, device=dev)   # arrival counters start at zero
        elif workspace.numel() < need:
            raise ValueError("shared workspace too small for this layer")
        self.workspace = workspace
        self.out = torch.empty(tuple(q.shape), dtype=out_dtype or torch.float32, device=dev)
        self.lse = torch.empty(tuple(q.shape[:-1]), dtype=torch.float32, device=dev) if want_lse else None

    def run(self, stream=None, trace=None):
        if self.kv8:
            fairkv_decode_attn_kv8(self.q, self.k, self.v, self.k_scale, self.v_scale, self.items_d, self.plan.items,
                                   self.plan.slot_ptr, self.plan.n_parts, self.workspace, self.out, self.lse,
                                   self.scale, self.Hkv, stream)
            return self.out, self.lse
        fairkv_decode_attn(self.q, self.k, self.v, self.items_d, self.plan.items, self.plan.slot_ptr, self.plan.n_parts,
                           self.workspace, self.out, self.lse, self.scale, self.Hkv, stream,
                           bf16_on_valu=self.bf16_on_valu, trace=trace)
        return self.out, self.lse


def gpu_share(lens, shares, gpu):
    """One GPU's part of a placement made by fairkv_place: (heads, len_local).

    heads      the KV heads this GPU holds, ascending
    len_local  int32 [B][len(heads)]: len[b][head] for the batch rows this GPU serves of that
               head, 0 for the rows another copy serves (such pairs get empty items, no K/V).
    The GPU then runs fairkv_plan + fairkv_decode_attn on len_local like on any other cache.
    """
    lens = np.asarray(lens)
    mine = [s for s in shares if int(s["gpu"]) == int(gpu)]
    heads = sorted(int(s["head"]) for s in mine)
    out = np.zeros((lens.shape[0], len(heads)), dtype=np.int32)
    for s in mine:
        col = heads.index(int(s["head"]))
        out[int(s["row_begin"]):int(s["row_end"]), col] = lens[int(s["row_begin"]):int(s["row_end"]), int(s["head"])]
    return heads, out
