"""Thin Python binding of libfairkv.so (see include/fairkv.h for the contract).

The functions carry the names of the C entry points and only marshal arguments:
planning runs in the library's host code and attention runs in its HIP kernels.
PyTorch appears solely as the owner of device memory and streams.  There is no
fallback: if the shared libraries have not been built, the first call raises.
"""
from __future__ import annotations

import ctypes
import os
from dataclasses import dataclass

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libfairkv.so")
BINDING_PATH = os.path.join(_HERE, "_binding.so")

FAIRKV_OK, FAIRKV_EINVAL, FAIRKV_ECAP, FAIRKV_EWORKSPACE, FAIRKV_EUNSUPPORTED, FAIRKV_EHIP = 0, -1, -2, -3, -4, -5
FAIRKV_BF16, FAIRKV_F32, FAIRKV_E4M3, FAIRKV_BF16_VALU = 0, 1, 2, 3
FAIRKV_TRACE_STAMPS = 16
FAIRKV_SHORT_PAIR_TOKENS = 96
FAIRKV_STATIC_WORKSPACE_BYTES = 8 << 20
FAIRKV_POLICY_NAIVE, FAIRKV_POLICY_LPT, FAIRKV_POLICY_LPT_SPLIT, FAIRKV_POLICY_FAIR = 0, 1, 2, 3

FAIRKV_PLACE_AUTO, FAIRKV_PLACE_EXACT, FAIRKV_PLACE_GREEDY = 0, 1, 2

EXPORTS = ("fairkv_default_params", "fairkv_plan", "fairkv_workspace_bytes", "fairkv_workspace_counter_bytes",
           "fairkv_decode_attn",
           "fairkv_decode_attn_multi", "fairkv_decode_attn_kv8", "fairkv_decode_attn_kv8_per_head",
           "fairkv_decode_attn_static", "fairkv_decode_attn_trace",
           "fairkv_place", "fairkv_pack", "fairkv_append", "fairkv_plan_grow", "fairkv_stream_probe", "fairkv_stream_probe_shape", "fairkv_workspace_reset",
           "fairkv_strerror", "fairkv_version")


class fairkv_item(ctypes.Structure):
    _fields_ = [("row", ctypes.c_int64)] + [(n, ctypes.c_int32) for n in
                                            ("tok_count", "b", "h", "chunk", "n_chunks", "part")]


class fairkv_plan_params(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in
                ("n_slots", "tile", "min_chunk", "max_split", "oversub", "overhead_tokens", "policy", "short_overhead_tokens")]


class fairkv_plan_summary(ctypes.Structure):
    _fields_ = [("total_tokens", ctypes.c_int64), ("max_slot_load", ctypes.c_int64),
                ("min_slot_load", ctypes.c_int64), ("n_items", ctypes.c_int32), ("n_parts", ctypes.c_int32)]


class fairkv_place_params(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("tp", "max_extra", "max_copies", "mode")]


class fairkv_share(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("head", "gpu", "copy", "n_copies", "row_begin", "row_end")]


class fairkv_place_summary(ctypes.Structure):
    _fields_ = [("den", ctypes.c_int64), ("delta_num", ctypes.c_int64), ("max_load_num", ctypes.c_int64),
                ("min_load_num", ctypes.c_int64), ("efficiency", ctypes.c_double), ("n_shares", ctypes.c_int32),
                ("exact", ctypes.c_int32)]


SHARE_DTYPE = np.dtype([(n, np.int32) for n, _ in fairkv_share._fields_])
assert SHARE_DTYPE.itemsize == ctypes.sizeof(fairkv_share) == 24

ITEM_DTYPE = np.dtype([("row", np.int64)] + [(n, np.int32) for n, _ in fairkv_item._fields_[1:]])
assert ITEM_DTYPE.itemsize == ctypes.sizeof(fairkv_item) == 32


class FairKVError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {strerror(code)} ({code})")


_lib = None


def lib() -> ctypes.CDLL:
    """The loaded shared library; raises if it was never built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing: build it with "
                              f"`python -m paper_2502_15804_amd.build` (there is no fallback path)")
        try:
            # PyTorch ships a HIP runtime of its own: load it first, so that this library binds to the same one
            # (two runtimes in one process do not share streams or code objects, and every launch would fail)
            import torch  # noqa: F401
        except ImportError:
            pass
        L = ctypes.CDLL(LIB_PATH)
        vp, i32, i64p = ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p
        L.fairkv_default_params.restype = ctypes.c_int
        L.fairkv_default_params.argtypes = [ctypes.POINTER(fairkv_plan_params), i32]
        L.fairkv_plan.restype = ctypes.c_int
        L.fairkv_plan.argtypes = [vp, i64p, i32, i32, ctypes.POINTER(fairkv_plan_params), vp, i32, vp, vp,
                                  ctypes.POINTER(fairkv_plan_summary)]
        L.fairkv_workspace_counter_bytes.restype = ctypes.c_size_t
        L.fairkv_workspace_counter_bytes.argtypes = [i32]
        L.fairkv_workspace_bytes.restype = ctypes.c_size_t
        L.fairkv_workspace_bytes.argtypes = [i32, i32, i32, i32]
        L.fairkv_decode_attn.restype = ctypes.c_int
        L.fairkv_decode_attn.argtypes = [vp, vp, vp, ctypes.c_int64, vp, vp, i32, vp, i32, i32, vp, ctypes.c_size_t, vp,
                                         vp, i32, i32, i32, i32, i32, i32, ctypes.c_float, vp]
        L.fairkv_place.restype = ctypes.c_int
        L.fairkv_place.argtypes = [vp, i32, i32, ctypes.POINTER(fairkv_place_params), vp, i32, vp,
                                   ctypes.POINTER(fairkv_place_summary)]
        L.fairkv_pack.restype = ctypes.c_int
        L.fairkv_pack.argtypes = [vp, vp, i32, i32, i32, i32, i32, vp, vp, vp, vp, vp, i32, vp, vp, ctypes.c_int64, vp, vp]
        L.fairkv_append.restype = ctypes.c_int
        L.fairkv_append.argtypes = [vp, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, ctypes.c_int64, vp, vp]
        L.fairkv_plan_grow.restype = ctypes.c_int
        L.fairkv_plan_grow.argtypes = [vp, i32, i32, i32, vp, vp]
        L.fairkv_stream_probe.restype = ctypes.c_int
        L.fairkv_stream_probe.argtypes = [vp, vp, ctypes.c_int64, i32, vp, vp]
        L.fairkv_workspace_reset.restype = ctypes.c_int
        L.fairkv_workspace_reset.argtypes = [vp, ctypes.c_size_t, i32, vp]
        L.fairkv_stream_probe_shape.restype = ctypes.c_int
        L.fairkv_stream_probe_shape.argtypes = [vp, vp, ctypes.c_int64, i32, i32, i32, i32, vp, vp]
        L.fairkv_decode_attn_multi.restype = ctypes.c_int
        L.fairkv_decode_attn_multi.argtypes = [vp, vp, vp, ctypes.c_int64, vp, vp, i32, vp, i32, i32, vp,
                                               ctypes.c_size_t, vp, vp, i32, i32, i32, i32, i32, i32, i32,
                                               ctypes.c_float, vp]
        L.fairkv_decode_attn_kv8.restype = ctypes.c_int
        L.fairkv_decode_attn_kv8.argtypes = [vp, vp, vp, ctypes.c_int64, ctypes.c_float, ctypes.c_float, vp, vp, i32, vp,
                                             i32, i32, vp, ctypes.c_size_t, vp, vp, i32, i32, i32, i32, i32, i32,
                                             ctypes.c_float, vp]
        L.fairkv_decode_attn_kv8_per_head.restype = ctypes.c_int
        L.fairkv_decode_attn_kv8_per_head.argtypes = [vp, vp, vp, ctypes.c_int64, vp, vp, vp, vp, i32, vp,
                                                      i32, i32, vp, ctypes.c_size_t, vp, vp, i32, i32, i32, i32, i32, i32,
                                                      ctypes.c_float, vp]
        L.fairkv_decode_attn_static.restype = ctypes.c_int
        L.fairkv_decode_attn_static.argtypes = [vp, vp, vp, ctypes.c_int64, vp, vp, i32, vp, i32, i32, vp, vp,
                                                i32, i32, i32, i32, i32, i32, i32, ctypes.c_float, vp]
        L.fairkv_decode_attn_trace.restype = ctypes.c_int
        L.fairkv_decode_attn_trace.argtypes = [vp, vp, vp, ctypes.c_int64, vp, vp, i32, vp, i32, i32, vp, ctypes.c_size_t,
                                               vp, vp, i32, i32, i32, i32, ctypes.c_float, vp, ctypes.c_size_t, vp]
        L.fairkv_strerror.restype = ctypes.c_char_p
        L.fairkv_strerror.argtypes = [ctypes.c_int]
        L.fairkv_version.restype = ctypes.c_int
        _lib = L
    return _lib


def strerror(code: int) -> str:
    return lib().fairkv_strerror(int(code)).decode()


def fairkv_version() -> int:
    return int(lib().fairkv_version())


def fairkv_default_params(n_compute_units: int, **overrides) -> fairkv_plan_params:
    p = fairkv_plan_params()
    rc = lib().fairkv_default_params(ctypes.byref(p), int(n_compute_units))
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_default_params")
    for k, v in overrides.items():
        if k not in dict(fairkv_plan_params._fields_):
            raise TypeError(f"unknown plan parameter {k!r}")
        setattr(p, k, int(v))
    return p


@dataclass
class Plan:
    """Host-side result of fairkv_plan (numpy arrays, ready to copy to the device)."""
    items: np.ndarray        # structured array of fairkv_item, grouped by slot
    slot_ptr: np.ndarray     # int32 [n_slots+1]
    part_base: np.ndarray    # int32 [B*Hkv+1]
    summary: fairkv_plan_summary
    params: fairkv_plan_params

    @property
    def n_items(self) -> int:
        return int(self.summary.n_items)

    @property
    def n_parts(self) -> int:
        return int(self.summary.n_parts)

    @property
    def n_slots(self) -> int:
        return int(self.params.n_slots)

    def slot_loads(self) -> np.ndarray:
        short = ((self.items["n_chunks"] == 1) & (self.items["tok_count"] <= FAIRKV_SHORT_PAIR_TOKENS)
                 & (int(self.params.short_overhead_tokens) > 0))
        cost = self.items["tok_count"].astype(np.int64) + np.where(short, int(self.params.short_overhead_tokens),
                                                                   int(self.params.overhead_tokens))
        csum = np.concatenate([[0], np.cumsum(cost)])
        return csum[self.slot_ptr[1:]] - csum[self.slot_ptr[:-1]]


def fairkv_plan(lens, off, B: int, Hkv: int, params: fairkv_plan_params) -> Plan:
    """Two calls into the library: one to size the work list, one to fill it."""
    lens = np.ascontiguousarray(np.asarray(lens).reshape(-1), dtype=np.int32)
    off = np.ascontiguousarray(np.asarray(off).reshape(-1), dtype=np.int64)
    if lens.size != int(B) * int(Hkv) or off.size != lens.size:
        raise ValueError("lens and off must have B*Hkv entries")
    L = lib()
    summary = fairkv_plan_summary()
    n_slots = max(int(params.n_slots), 0)
    slot_ptr = np.zeros(n_slots + 1, dtype=np.int32)
    part_base = np.zeros(int(B) * int(Hkv) + 1, dtype=np.int32)
    rc = L.fairkv_plan(lens.ctypes.data, off.ctypes.data, B, Hkv, ctypes.byref(params), None, 0,
                       slot_ptr.ctypes.data, part_base.ctypes.data, ctypes.byref(summary))
    if rc not in (FAIRKV_OK, FAIRKV_ECAP):
        raise FairKVError(rc, "fairkv_plan")
    items = np.zeros(int(summary.n_items), dtype=ITEM_DTYPE)
    if summary.n_items > 0:
        rc = L.fairkv_plan(lens.ctypes.data, off.ctypes.data, B, Hkv, ctypes.byref(params), items.ctypes.data,
                           items.size, slot_ptr.ctypes.data, part_base.ctypes.data, ctypes.byref(summary))
        if rc != FAIRKV_OK:
            raise FairKVError(rc, "fairkv_plan")
    return Plan(items, slot_ptr, part_base, summary, params)


@dataclass
class Placement:
    """Host-side result of fairkv_place."""
    shares: np.ndarray       # structured array of fairkv_share, ordered by (head, copy)
    gpu_load: np.ndarray     # int64 [tp], in units of 1/summary.den tokens
    summary: fairkv_place_summary
    params: fairkv_place_params


def fairkv_place(W, B: int, tp: int, max_extra: int = 0, max_copies: int = 1, mode: int = FAIRKV_PLACE_AUTO) -> Placement:
    W = np.ascontiguousarray(np.asarray(W).reshape(-1), dtype=np.int64)
    p = fairkv_place_params(int(tp), int(max_extra), int(max_copies), int(mode))
    s = fairkv_place_summary()
    shares = np.zeros(W.size + max(int(max_extra), 0), dtype=SHARE_DTYPE)
    load = np.zeros(max(int(tp), 1), dtype=np.int64)
    rc = lib().fairkv_place(W.ctypes.data, W.size, int(B), ctypes.byref(p), shares.ctypes.data, shares.size,
                            load.ctypes.data, ctypes.byref(s))
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_place")
    return Placement(shares[:s.n_shares].copy(), load, s, p)


def fairkv_workspace_counter_bytes(n_pairs: int) -> int:
    return int(lib().fairkv_workspace_counter_bytes(int(n_pairs)))


def fairkv_workspace_bytes(n_parts: int, n_pairs: int, G: int, D: int) -> int:
    return int(lib().fairkv_workspace_bytes(int(n_parts), int(n_pairs), int(G), int(D)))


# What every call needs of PyTorch, looked up once: (module, the function that gives a device's current stream as a number).
_pt = None


def _torch():
    global _pt
    if _pt is None:
        import torch
        raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)    # not a public name: a build may lack it
        if raw_stream is None:
            raw_stream = lambda device: torch.cuda.current_stream(device).cuda_stream
        _pt = (torch, raw_stream)
    return _pt


# The per-call part of this binding: a call on the GPU is worth 5 to 20 us, so arguments are checked and converted in native code
# (csrc/binding.cpp), which gets the addresses of the library's functions from here.
_native_module = None


def _native():
    global _native_module
    if _native_module is None:
        L = lib()
        if not os.path.exists(BINDING_PATH):
            raise ImportError(f"{BINDING_PATH} is missing: build it with "
                              f"`python -m paper_2502_15804_amd.build` (there is no fallback path)")
        _torch()                                             # the libraries that it is linked with
        from .build import binding_is_made_for_this
        if not binding_is_made_for_this():
            raise ImportError(f"{BINDING_PATH} was built for another Python or PyTorch: build it again with "
                              f"`python -m paper_2502_15804_amd.build`")
        from importlib import machinery, util
        name = __name__ + "._binding"                        # the loader enters it in sys.modules: not under a name of the program's own
        loader = machinery.ExtensionFileLoader(name, BINDING_PATH)
        m = util.module_from_spec(util.spec_from_file_location(name, BINDING_PATH, loader=loader))
        loader.exec_module(m)
        m.init(ITEM_DTYPE, *(ctypes.cast(f, ctypes.c_void_p).value for f in (
            L.fairkv_decode_attn_multi, L.fairkv_decode_attn_static, L.fairkv_decode_attn_trace, L.fairkv_decode_attn_kv8,
            L.fairkv_decode_attn_kv8_per_head, L.fairkv_pack, L.fairkv_append)))
        _native_module = m
    return _native_module


def _ptr(t):
    return t.data_ptr() if t is not None else None


def _stream(stream, t):
    """The stream to enqueue on: the caller's, or the current one of the device of tensor t."""
    return stream.cuda_stream if stream is not None else _torch()[1](t.get_device())


def fairkv_decode_attn(q, k, v, items, items_host, slot_ptr, n_parts, workspace, out, lse, scale, Hkv, stream=None,
                       bf16_on_valu=False, trace=None):
    """Enqueue decode attention for one layer on `stream` (default: torch's current stream).

    workspace=None calls fairkv_decode_attn_static (the library's own workspace); trace (a zero-filled int64 device
    tensor of n_slots * FAIRKV_TRACE_STAMPS) calls fairkv_decode_attn_trace; bf16_on_valu passes FAIRKV_BF16_VALU.

    Tensor arguments are CUDA/HIP torch tensors owned by the caller: q [B,Hq,D], or [B,q_len,Hq,D] for
    several new tokens per sequence (fairkv_decode_attn_multi; out and lse then carry q_len too); k, v [rows,D];
    items: uint8 view of the plan's item array (n_items * 32 bytes); workspace uint8, zero-filled
    before its first use; out [B,Hq,D] float32 or bfloat16; lse float32 [B,Hq] or None.
    items_host and slot_ptr are the plan's HOST arrays (numpy: fairkv_item records, int32
    [n_slots+1]).  Nothing is allocated or synchronised here.
    """
    rc = (_native_module or _native()).decode((_pt or _torch())[1], q, k, v, items, items_host, slot_ptr, n_parts, workspace, out, lse,
                                              scale, Hkv, stream, bf16_on_valu, trace)
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_decode_attn_trace" if trace is not None else "fairkv_decode_attn_static" if workspace is None else
                          "fairkv_decode_attn_multi" if q.dim() == 4 and q.shape[1] > 1 else "fairkv_decode_attn")


def fairkv_decode_attn_kv8(q, k8, v8, k_scale, v_scale, items, items_host, slot_ptr, n_parts, workspace, out, lse,
                           scale, Hkv, stream=None):
    """fairkv_decode_attn over a cache stored as 8-bit floats (E4M3, finite-only "fn" encoding).

    k8, v8 [rows,D]: torch.float8_e4m3fn or uint8 holding the same bytes; a stored byte stands for
    value * k_scale (v_scale).  k_scale and v_scale are two numbers, or two sequences of Hkv numbers (a scale
    per KV head: fairkv_decode_attn_kv8_per_head).  q [B,Hq,D] or [B,q_len,Hq,D] bfloat16.  Everything else as in
    fairkv_decode_attn.
    """
    per_head = (type(k_scale) is not float or type(v_scale) is not float) and bool(np.ndim(k_scale) or np.ndim(v_scale))
    if per_head:
        k_scale = np.ascontiguousarray(np.broadcast_to(np.asarray(k_scale, dtype=np.float32), (Hkv,)))
        v_scale = np.ascontiguousarray(np.broadcast_to(np.asarray(v_scale, dtype=np.float32), (Hkv,)))
    else:
        k_scale, v_scale = float(k_scale), float(v_scale)    # also arrays and tensors of no dimension
    rc = (_native_module or _native()).decode_8bit((_pt or _torch())[1], q, k8, v8, k_scale, v_scale, items, items_host, slot_ptr, n_parts,
                                                   workspace, out, lse, scale, Hkv, stream, per_head)
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_decode_attn_kv8_per_head" if per_head else "fairkv_decode_attn_kv8")


def _check_dev(**tensors):
    for name, t in tensors.items():
        if t is not None and (not t.is_cuda or not t.is_contiguous()):
            raise ValueError(f"{name} must be a contiguous device tensor")


def fairkv_pack(k_dense, v_dense, keep_ptr, keep_t, off, items, slot_ptr, k_out, v_out, bad=None, stream=None):
    """Enqueue the gather of the kept rows.  All arguments are device tensors: k_dense, v_dense
    [B][Hkv][T][D]; keep_ptr int64 [B*Hkv+1]; keep_t int32; off int64 [B*Hkv]; items uint8 view of a
    plan's item array; slot_ptr int32 [n_slots+1]; k_out, v_out [n_rows][D]; bad int32 [1] or None."""
    rc = (_native_module or _native()).pack((_pt or _torch())[1], k_dense, v_dense, keep_ptr, keep_t, off, items, slot_ptr, k_out, v_out,
                                            bad, stream)
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_pack")


def fairkv_append(k_new, v_new, off, lens, cap, k, v, full=None, stream=None):
    """Enqueue the append of one new row per pair.  Device tensors: k_new, v_new [B][Hkv][D]; off int64,
    lens int32 (updated in place), cap int32, all [B*Hkv]; k, v packed [n_rows][D]; full int32 [1] or None."""
    rc = (_native_module or _native()).append((_pt or _torch())[1], k_new, v_new, off, lens, cap, k, v, full, stream)
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_append")


def fairkv_plan_grow(items: np.ndarray, B: int, Hkv: int, lens: np.ndarray, cap: np.ndarray) -> None:
    """Host arrays, updated in place: items (a whole plan, ITEM_DTYPE), lens int32 [B*Hkv]; cap int32 [B*Hkv]."""
    if items.dtype != ITEM_DTYPE or not items.flags.c_contiguous:
        raise TypeError("items must be a contiguous fairkv_item array")
    if lens.dtype != np.int32 or cap.dtype != np.int32 or not lens.flags.c_contiguous or not cap.flags.c_contiguous:
        raise TypeError("lens and cap must be contiguous int32 arrays")
    if lens.size != B * Hkv or cap.size != B * Hkv:
        raise ValueError("lens and cap must have B*Hkv entries")
    rc = lib().fairkv_plan_grow(items.ctypes.data, items.size, int(B), int(Hkv), lens.ctypes.data, cap.ctypes.data)
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_plan_grow")


def fairkv_workspace_reset(workspace, n_pairs, stream=None):
    """Enqueue the kernel that zeroes the counter bytes of a device workspace (see the header)."""
    _check_dev(workspace=workspace)
    rc = lib().fairkv_workspace_reset(_ptr(workspace), workspace.numel() * workspace.element_size(), int(n_pairs),
                                      _stream(stream, workspace))
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_workspace_reset")


def fairkv_stream_probe(k, v, n_workgroups, sink, stream=None, shape=None):
    """Enqueue the do-nothing reader over all of the device tensors k and v (see the header).
    shape: (waves, stages, tile_kib) for fairkv_stream_probe_shape; None = the decode kernel's shape."""
    _check_dev(k=k, v=v, sink=sink)
    if sink.numel() * sink.element_size() < 4 * n_workgroups:
        raise ValueError("sink too small")
    nbytes = min(k.numel() * k.element_size(), v.numel() * v.element_size())
    if shape is not None:
        rc = lib().fairkv_stream_probe_shape(_ptr(k), _ptr(v), nbytes, int(n_workgroups), int(shape[0]), int(shape[1]),
                                             int(shape[2]), _ptr(sink), _stream(stream, k))
    else:
        rc = lib().fairkv_stream_probe(_ptr(k), _ptr(v), nbytes, int(n_workgroups), _ptr(sink),
                                       _stream(stream, k))
    if rc != FAIRKV_OK:
        raise FairKVError(rc, "fairkv_stream_probe")
