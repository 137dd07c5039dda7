// The per-call part of the Python binding: checks the arguments of a call and makes it.  The functions of __init__.py hand
// their arguments on; everything else of the binding (planning, errors, documentation) is there.
//
// What bounds an eager decode step of a small model is the host.  In Python the thirty looks at shapes, types and pointers and
// the conversion of twenty arguments took 6 us of a call's 10.7, 4 of an append's 6.7; here they take 0.3 us, so that what is
// left is the launch.  The library itself stays a plain C one: its functions come as addresses (init), of whichever file was loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#define NPY_NO_DEPRECATED_API NPY_2_0_API_VERSION
#include <numpy/arrayobject.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "fairkv.h"
#include "fairkv_measure.h"

namespace {

decltype(&fairkv_decode_attn_multi) decode_multi;
decltype(&fairkv_decode_attn_static) decode_static;
decltype(&fairkv_decode_attn_trace) decode_trace;
decltype(&fairkv_decode_attn_kv8) decode_kv8;
decltype(&fairkv_decode_attn_kv8_per_head) decode_kv8_per_head;
decltype(&fairkv_pack) pack_rows;
decltype(&fairkv_append) append_rows;
PyArray_Descr *item_descr;      // of the plan's item array

struct Refused {};              // a Python exception is set

[[noreturn]] void refuse(PyObject *type, const char *why)
{
    PyErr_SetString(type, why);
    throw Refused{};
}

// A tensor argument; None gives an undefined tensor.
const at::Tensor &tensor(PyObject *o, const char *name, bool optional = false)
{
    static const at::Tensor none;
    if (optional && o == Py_None) return none;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        throw Refused{};
    }
    return THPVariable_Unpack(o);
}
void on_device(const at::Tensor &t, const char *name)
{
    if (t.defined() && (!t.is_cuda() || !t.is_contiguous())) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous device tensor", name);
        throw Refused{};
    }
}
void *ptr(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }
bool is(const at::Tensor &t, at::ScalarType type) { return t.scalar_type() == type; }

int32_t dtype_code(const at::Tensor &t)      // -1: none of the library's
{
    switch (t.scalar_type()) {
    case at::kBFloat16: return FAIRKV_BF16;
    case at::kFloat: return FAIRKV_F32;
    case at::kByte:
    case at::kFloat8_e4m3fn: return FAIRKV_E4M3;
    default: return -1;
    }
}
bool is_q_or_out(const at::Tensor &t) { return is(t, at::kBFloat16) || is(t, at::kFloat); }

int32_t low_word(PyObject *i)      // of an int, whose reference it takes
{
    if (!i) throw Refused{};
    const auto v = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(i));
    Py_DECREF(i);
    return v;
}
int32_t int_of(PyObject *o) { return low_word(PyNumber_Long(o)); }        // whatever int() takes
int32_t index_of(PyObject *o) { return low_word(PyNumber_Index(o)); }     // integers only
float float_of(PyObject *o)                                               // whatever float() takes
{
    PyObject *f = PyNumber_Float(o);
    if (!f) throw Refused{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return static_cast<float>(v);
}

// The stream to enqueue on: the caller's, or what `current` (device number -> stream) says of the tensor's device.  A caller's is
// whatever has a cuda_stream: a number, a ctypes.c_void_p, or None for the null stream.
void *stream_of(PyObject *stream, PyObject *current, const at::Tensor &t)
{
    PyObject *s = stream != Py_None ? PyObject_GetAttrString(stream, "cuda_stream") : nullptr;
    if (stream == Py_None) {
        PyObject *device = PyLong_FromLong(t.get_device());
        s = device ? PyObject_CallOneArg(current, device) : nullptr;
        Py_XDECREF(device);
    }
    if (s && s != Py_None && !PyLong_Check(s)) {
        PyObject *value = PyObject_GetAttrString(s, "value");
        Py_DECREF(s);
        s = value;
    }
    if (!s) throw Refused{};
    void *p = s == Py_None ? nullptr : PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw Refused{};
    return p;
}

// The plan's arguments of a decode call.
struct PlanArgs {
    const fairkv_item *items, *items_host;
    const int32_t *slot_ptr;
    int32_t n_items, n_slots, n_parts;
};
PlanArgs plan_args(const at::Tensor &items, PyObject *items_host, PyObject *slot_ptr, PyObject *n_parts)
{
    if (!PyArray_Check(slot_ptr)) refuse(PyExc_TypeError, "slot_ptr must be a contiguous host int32 array");
    auto *s = reinterpret_cast<PyArrayObject *>(slot_ptr);
    if (!PyArray_EquivTypenums(PyArray_TYPE(s), NPY_INT32) || !PyArray_ISNOTSWAPPED(s) || !PyArray_IS_C_CONTIGUOUS(s))
        refuse(PyExc_TypeError, "slot_ptr must be a contiguous host int32 array");
    if (PyArray_SIZE(s) < 2) refuse(PyExc_ValueError, "shape mismatch");
    const int64_t bytes = static_cast<int64_t>(items.nbytes());
    if (bytes % 32 != 0) refuse(PyExc_ValueError, "items must be a whole number of 32-byte records");
    auto *h = reinterpret_cast<PyArrayObject *>(items_host);
    if (!PyArray_Check(items_host) || (PyArray_DESCR(h) != item_descr && !PyArray_EquivTypes(PyArray_DESCR(h), item_descr)) ||
        !PyArray_IS_C_CONTIGUOUS(h) || PyArray_SIZE(h) * 32 != bytes)
        refuse(PyExc_TypeError, "items_host must be the plan's contiguous item array, as many records as `items`");
    return PlanArgs{static_cast<const fairkv_item *>(items.data_ptr()), static_cast<const fairkv_item *>(PyArray_DATA(h)),
                    static_cast<const int32_t *>(PyArray_DATA(s)), static_cast<int32_t>(bytes / 32),
                    static_cast<int32_t>(PyArray_SIZE(s) - 1), int_of(n_parts)};
}

struct Shape {
    int32_t B, q_len, Hq, D;
};
// q, and what has to agree with it: out, lse, and the D of k (v has k's shape).
Shape shape_of(const at::Tensor &q, const at::Tensor &k, const at::Tensor &v, const at::Tensor &out, const at::Tensor &lse, bool two_dims)
{
    const auto d = q.sizes();
    if (d.size() != 3 && d.size() != 4) refuse(PyExc_ValueError, "q must be [B, Hq, D] or [B, q_len, Hq, D]");
    if (lse.defined() && !is(lse, at::kFloat)) refuse(PyExc_TypeError, "lse must be float32");
    if (k.dim() < 2 || (two_dims && k.dim() != 2) || k.size(1) != d.back() || v.sizes() != k.sizes() || out.sizes() != d)
        refuse(PyExc_ValueError, "shape mismatch");
    if (lse.defined() && lse.sizes() != d.slice(0, d.size() - 1)) refuse(PyExc_ValueError, "lse must have q's shape without the last dimension");
    const bool multi = d.size() == 4;
    return Shape{static_cast<int32_t>(d[0]), multi ? static_cast<int32_t>(d[1]) : 1, static_cast<int32_t>(d[d.size() - 2]),
                 static_cast<int32_t>(d.back())};
}

// Runs `call` (which throws Refused with an exception set, or what PyTorch throws) and returns its code to Python.
template <class Call>
PyObject *guarded(Py_ssize_t got, Py_ssize_t want, Call call)
{
    if (got != want) return PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
    try {
        return PyLong_FromLong(call());
    } catch (const Refused &) {
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}
// A library call without the interpreter's lock, as any call through ctypes (a pointer that PyTorch does not give throws).
template <class Call>
int unlocked(Call call)
{
    struct Unlocked {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    } lock;
    return call();
}

// (current, q, k, v, items, items_host, slot_ptr, n_parts, workspace, out, lse, scale, Hkv, stream, bf16_on_valu, trace)
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 16, [&]() -> int {
        const int32_t Hkv = index_of(a[12]);
        const at::Tensor &q = tensor(a[1], "q"), &k = tensor(a[2], "k"), &v = tensor(a[3], "v"), &items = tensor(a[4], "items"),
                         &workspace = tensor(a[8], "workspace", true), &out = tensor(a[9], "out"), &lse = tensor(a[10], "lse", true),
                         &trace = tensor(a[15], "trace", true);
        if (!is_q_or_out(q) || k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type() || !is_q_or_out(out))
            refuse(PyExc_TypeError, "q/k/v must share bf16 or fp32; out must be bf16 or fp32");
        on_device(q, "q"), on_device(k, "k"), on_device(v, "v"), on_device(items, "items"), on_device(workspace, "workspace");
        on_device(out, "out"), on_device(lse, "lse"), on_device(trace, "trace");
        const Shape s = shape_of(q, k, v, out, lse, false);
        const int on_valu = PyObject_IsTrue(a[14]);
        if (on_valu < 0) throw Refused{};
        const int32_t in_dt = on_valu && is(q, at::kBFloat16) ? FAIRKV_BF16_VALU : dtype_code(q);
        const PlanArgs p = plan_args(items, a[5], a[6], a[7]);
        const float scale = float_of(a[11]);
        void *st = stream_of(a[13], a[0], q);
        float *l = static_cast<float *>(ptr(lse));
        if (trace.defined()) {
            if (s.q_len != 1 || !workspace.defined() || !is(trace, at::kLong))
                refuse(PyExc_ValueError, "a traced call is a single-token call with a caller's workspace and an int64 trace buffer");
            return unlocked([&] {
                return decode_trace(q.data_ptr(), k.data_ptr(), v.data_ptr(), k.size(0), p.items, p.items_host, p.n_items, p.slot_ptr, p.n_slots,
                                    p.n_parts, workspace.data_ptr(), workspace.nbytes(), out.data_ptr(), l, s.B, s.Hq, Hkv, s.D, scale,
                                    static_cast<uint64_t *>(trace.data_ptr()), trace.nbytes(), st);
            });
        }
        if (!workspace.defined())
            return unlocked([&] {
                return decode_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), k.size(0), p.items, p.items_host, p.n_items, p.slot_ptr, p.n_slots,
                                     p.n_parts, out.data_ptr(), l, s.B, s.q_len, s.Hq, Hkv, s.D, in_dt, dtype_code(out), scale, st);
            });
        return unlocked([&] {
            return decode_multi(q.data_ptr(), k.data_ptr(), v.data_ptr(), k.size(0), p.items, p.items_host, p.n_items, p.slot_ptr, p.n_slots,
                                p.n_parts, workspace.data_ptr(), workspace.nbytes(), out.data_ptr(), l, s.B, s.q_len, s.Hq, Hkv, s.D, in_dt,
                                dtype_code(out), scale, st);
        });
    });
}

// The numbers of a scale per KV head.
const float *scale_array(PyObject *o, int32_t Hkv, const char *name)
{
    auto *s = reinterpret_cast<PyArrayObject *>(o);
    if (!PyArray_Check(o) || PyArray_TYPE(s) != NPY_FLOAT || !PyArray_ISCARRAY_RO(s) || PyArray_NDIM(s) != 1 || PyArray_SIZE(s) != Hkv) {
        PyErr_Format(PyExc_TypeError, "%s must be a contiguous float32 array of one number per KV head", name);
        throw Refused{};
    }
    return static_cast<const float *>(PyArray_DATA(s));
}

// (current, q, k8, v8, k_scale, v_scale, items, items_host, slot_ptr, n_parts, workspace, out, lse, scale, Hkv, stream, per_head); the scales
// are two float32 arrays if per_head is true, else two numbers
PyObject *decode_8bit(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 17, [&]() -> int {
        const int32_t Hkv = index_of(a[14]);
        const int per_head = PyObject_IsTrue(a[16]);
        if (per_head < 0) throw Refused{};
        const float *k_scales = nullptr, *v_scales = nullptr;
        float k_scale = 1.f, v_scale = 1.f;
        if (per_head)
            k_scales = scale_array(a[4], Hkv, "k_scale"), v_scales = scale_array(a[5], Hkv, "v_scale");
        else
            k_scale = float_of(a[4]), v_scale = float_of(a[5]);
        const at::Tensor &q = tensor(a[1], "q"), &k = tensor(a[2], "k8"), &v = tensor(a[3], "v8"), &items = tensor(a[6], "items"),
                         &workspace = tensor(a[10], "workspace"), &out = tensor(a[11], "out"), &lse = tensor(a[12], "lse", true);
        if (!is(q, at::kBFloat16) || dtype_code(k) != FAIRKV_E4M3 || dtype_code(v) != FAIRKV_E4M3 || !is_q_or_out(out))
            refuse(PyExc_TypeError, "q must be bf16, k8/v8 float8_e4m3fn or uint8, out bf16 or fp32");
        on_device(q, "q"), on_device(k, "k8"), on_device(v, "v8"), on_device(items, "items"), on_device(workspace, "workspace");
        on_device(out, "out"), on_device(lse, "lse");
        const Shape s = shape_of(q, k, v, out, lse, true);
        const PlanArgs p = plan_args(items, a[7], a[8], a[9]);
        const float scale = float_of(a[13]);
        void *st = stream_of(a[15], a[0], q);
        float *l = static_cast<float *>(ptr(lse));
        if (per_head)
            return unlocked([&] {
                return decode_kv8_per_head(q.data_ptr(), k.data_ptr(), v.data_ptr(), k.size(0), k_scales, v_scales, p.items, p.items_host, p.n_items,
                                           p.slot_ptr, p.n_slots, p.n_parts, workspace.data_ptr(), workspace.nbytes(), out.data_ptr(), l, s.B,
                                           s.q_len, s.Hq, Hkv, s.D, dtype_code(out), scale, st);
            });
        return unlocked([&] {
            return decode_kv8(q.data_ptr(), k.data_ptr(), v.data_ptr(), k.size(0), k_scale, v_scale, p.items, p.items_host, p.n_items, p.slot_ptr,
                              p.n_slots, p.n_parts, workspace.data_ptr(), workspace.nbytes(), out.data_ptr(), l, s.B, s.q_len, s.Hq, Hkv, s.D,
                              dtype_code(out), scale, st);
        });
    });
}

// (current, k_dense, v_dense, keep_ptr, keep_t, off, items, slot_ptr, k_out, v_out, bad, stream)
PyObject *pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> int {
        const at::Tensor &k = tensor(a[1], "k_dense"), &v = tensor(a[2], "v_dense"), &keep_ptr = tensor(a[3], "keep_ptr"),
                         &keep_t = tensor(a[4], "keep_t"), &off = tensor(a[5], "off"), &items = tensor(a[6], "items"),
                         &slot_ptr = tensor(a[7], "slot_ptr"), &k_out = tensor(a[8], "k_out"), &v_out = tensor(a[9], "v_out"),
                         &bad = tensor(a[10], "bad", true);
        if (k.dim() != 4) refuse(PyExc_ValueError, "k_dense must be [B, Hkv, T, D]");
        on_device(k, "k_dense"), on_device(v, "v_dense"), on_device(keep_ptr, "keep_ptr"), on_device(keep_t, "keep_t"), on_device(off, "off");
        on_device(items, "items"), on_device(slot_ptr, "slot_ptr"), on_device(k_out, "k_out"), on_device(v_out, "v_out"), on_device(bad, "bad");
        if (v.sizes() != k.sizes() || k_out.sizes() != v_out.sizes() || k_out.dim() < 2 || k_out.size(1) != k.size(3) ||
            k_out.scalar_type() != k.scalar_type() || v_out.scalar_type() != k.scalar_type() || v.scalar_type() != k.scalar_type())
            refuse(PyExc_ValueError, "shape or dtype mismatch");
        const int64_t pairs = k.size(0) * k.size(1);
        if (!is(keep_ptr, at::kLong) || !is(off, at::kLong) || !is(keep_t, at::kInt) || !is(slot_ptr, at::kInt) || keep_ptr.numel() != pairs + 1 ||
            off.numel() != pairs || (bad.defined() && !is(bad, at::kInt)))
            refuse(PyExc_TypeError, "keep_ptr/off must be int64, keep_t/slot_ptr/bad int32, sized for B*Hkv pairs");
        const int32_t dtype = dtype_code(k);
        if (dtype < 0) refuse(PyExc_KeyError, "rows must be bf16, fp32 or bytes");
        void *st = stream_of(a[11], a[0], k);
        return unlocked([&] {
            return pack_rows(k.data_ptr(), v.data_ptr(), static_cast<int32_t>(k.size(0)), static_cast<int32_t>(k.size(1)),
                             static_cast<int32_t>(k.size(2)), static_cast<int32_t>(k.size(3)), dtype, static_cast<const int64_t *>(keep_ptr.data_ptr()),
                             static_cast<const int32_t *>(keep_t.data_ptr()), static_cast<const int64_t *>(off.data_ptr()),
                             static_cast<const fairkv_item *>(items.data_ptr()), static_cast<const int32_t *>(slot_ptr.data_ptr()),
                             static_cast<int32_t>(slot_ptr.numel() - 1), k_out.data_ptr(), v_out.data_ptr(), k_out.size(0),
                             static_cast<int32_t *>(ptr(bad)), st);
        });
    });
}

// (current, k_new, v_new, off, lens, cap, k, v, full, stream)
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 10, [&]() -> int {
        const at::Tensor &k_new = tensor(a[1], "k_new"), &v_new = tensor(a[2], "v_new"), &off = tensor(a[3], "off"), &lens = tensor(a[4], "lens"),
                         &cap = tensor(a[5], "cap"), &k = tensor(a[6], "k"), &v = tensor(a[7], "v"), &full = tensor(a[8], "full", true);
        if (k_new.dim() != 3) refuse(PyExc_ValueError, "k_new must be [B, Hkv, D]");
        on_device(k_new, "k_new"), on_device(v_new, "v_new"), on_device(off, "off"), on_device(lens, "lens"), on_device(cap, "cap");
        on_device(k, "k"), on_device(v, "v"), on_device(full, "full");
        if (v_new.sizes() != k_new.sizes() || k.sizes() != v.sizes() || k.dim() < 2 || k.size(1) != k_new.size(2) ||
            k.scalar_type() != k_new.scalar_type() || v.scalar_type() != k_new.scalar_type() || v_new.scalar_type() != k_new.scalar_type())
            refuse(PyExc_ValueError, "shape or dtype mismatch");
        const int64_t pairs = k_new.size(0) * k_new.size(1);
        if (!is(off, at::kLong) || !is(lens, at::kInt) || !is(cap, at::kInt) || off.numel() != pairs || lens.numel() != pairs ||
            cap.numel() != pairs || (full.defined() && !is(full, at::kInt)))
            refuse(PyExc_TypeError, "off must be int64, lens/cap/full int32, sized for B*Hkv pairs");
        const int32_t dtype = dtype_code(k_new);
        if (dtype < 0) refuse(PyExc_KeyError, "rows must be bf16, fp32 or bytes");
        void *st = stream_of(a[9], a[0], k_new);
        return unlocked([&] {
            return append_rows(k_new.data_ptr(), v_new.data_ptr(), static_cast<int32_t>(k_new.size(0)), static_cast<int32_t>(k_new.size(1)),
                               static_cast<int32_t>(k_new.size(2)), dtype, static_cast<const int64_t *>(off.data_ptr()),
                               static_cast<int32_t *>(lens.data_ptr()), static_cast<const int32_t *>(cap.data_ptr()), k.data_ptr(), v.data_ptr(),
                               k.size(0), static_cast<int32_t *>(ptr(full)), st);
        });
    });
}

// (dtype of the plan's items, addresses of the library's functions in the order of the pointers above)
PyObject *init(PyObject *, PyObject *args)
{
    PyObject *dtype;
    unsigned long long f[7];
    if (!PyArg_ParseTuple(args, "OKKKKKKK", &dtype, f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6)) return nullptr;
    if (!PyArray_DescrCheck(dtype)) return PyErr_Format(PyExc_TypeError, "a numpy dtype is expected");
    Py_INCREF(dtype);
    Py_XDECREF(reinterpret_cast<PyObject *>(item_descr));
    item_descr = reinterpret_cast<PyArray_Descr *>(dtype);
    auto set = [&](auto &fn, int i) { fn = reinterpret_cast<std::decay_t<decltype(fn)>>(static_cast<uintptr_t>(f[i])); };
    set(decode_multi, 0), set(decode_static, 1), set(decode_trace, 2), set(decode_kv8, 3), set(decode_kv8_per_head, 4);
    set(pack_rows, 5), set(append_rows, 6);
    Py_RETURN_NONE;
}

// What this file is compiled against (build.py), found in the built file before that is loaded.
[[gnu::used]] const char made_for[] = MADE_FOR;

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(decode)), METH_FASTCALL, nullptr},
    {"decode_8bit", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(decode_8bit)), METH_FASTCALL, nullptr},
    {"pack", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(pack)), METH_FASTCALL, nullptr},
    {"append", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(append)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    import_array();
    return PyModule_Create(&module);
}
