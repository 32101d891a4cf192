// The Python binding's calls that a program makes once per decoded token or per layer, in native code: checks, output
// tensors, the current stream and the C call behind one METH_FASTCALL function each.  squat.py gives them their names,
// keywords and defaults.  With ctypes a call cost the host 5.5 to 11.3 us (a decoded token: 13 us for an append and its logits,
// of which the GPU works 8), of which the launches are 2.5 each.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "squat.h"

namespace {

struct Raised {};                          // a Python exception is set

PyObject* squat_error = nullptr;           // the class of squat.py: SquatError(status, where)

[[noreturn]] void raise(PyObject* type, const char* message) {
    PyErr_SetString(type, message);
    throw Raised{};
}

void check(int rc, const char* where) {
    if (rc == 0) return;
    PyObject* e = squat_error ? PyObject_CallFunction(squat_error, "is", rc, where) : nullptr;
    if (e) {
        PyErr_SetObject(squat_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_SetString(PyExc_RuntimeError, where);
    }
    throw Raised{};
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_AttributeError, "'%s' object is no torch.Tensor", Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}

// An int, or what stands for one (numpy's, a tensor of one: __index__), as ctypes takes it in the calls that go through it.
long long integer(PyObject* o) {
    long long v;
    if (PyLong_Check(o)) {
        v = PyLong_AsLongLong(o);
    } else {
        PyObject* i = PyNumber_Index(o);
        if (!i) throw Raised{};
        v = PyLong_AsLongLong(i);
        Py_DECREF(i);
    }
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

int small(PyObject* o) {
    const long long v = integer(o);
    if (v < INT32_MIN || v > INT32_MAX) raise(PyExc_OverflowError, "integer out of range");
    return static_cast<int>(v);
}

float number(PyObject* o) {                // whatever float() takes
    if (PyFloat_CheckExact(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
    PyObject* f = PyNumber_Float(o);
    if (!f) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return static_cast<float>(v);
}

squat_dtype dtype(PyObject* o, const at::Tensor& t) {
    switch (t.scalar_type()) {
        case at::kFloat: return SQUAT_F32;
        case at::kHalf: return SQUAT_F16;
        case at::kBFloat16: return SQUAT_BF16;
        default: break;
    }
    PyObject* dt = PyObject_GetAttrString(o, "dtype");
    if (dt) {
        PyErr_SetObject(PyExc_KeyError, dt);
        Py_DECREF(dt);
    }
    throw Raised{};
}

// A stream's handle, or None: the current device's current stream.
squat_stream stream(PyObject* o) {
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    void* s = PyLong_AsVoidPtr(o);
    if (!s && PyErr_Occurred()) throw Raised{};
    return s;
}

void need_device(const at::Tensor& t) {
    if (!t.is_cuda()) raise(PyExc_ValueError, "libsquat takes device tensors only");
}

// Device memory, or pinned host memory, which kernels reach as well (where calls have taken that before).
void need_reachable(const at::Tensor& t) {
    if (!t.is_cuda() && !t.is_pinned()) raise(PyExc_ValueError, "libsquat takes device tensors only (here: or pinned host memory)");
}

template <typename T>
T* pointer(const at::Tensor& t) {
    return static_cast<T*>(t.data_ptr());
}

void need_dims(const at::Tensor& t, int64_t dims) {
    if (t.dim() == dims) return;
    PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions is needed, got %d", static_cast<int>(dims), static_cast<int>(t.dim()));
    throw Raised{};
}

// Leaves the interpreter to other threads for as long as it lives.
struct Free {
    PyThreadState* const state = PyEval_SaveThread();
    ~Free() { PyEval_RestoreThread(state); }
};

// To be called with the interpreter free, as torch.empty does: an allocator that has to grow or to give back memory waits for the device.
at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

// An output: the caller's, or none yet (None: made beside `like` by the call that fills it).
at::Tensor given(PyObject* o, const at::Tensor& like) {
    if (o == Py_None) {
        need_device(like);
        return {};
    }
    need_reachable(tensor(o));
    return tensor(o);
}

PyObject* three(const at::Tensor& a, const at::Tensor& b, const at::Tensor& c) {
    PyObject* out = PyTuple_New(3);
    if (!out) throw Raised{};
    const at::Tensor* t[3] = {&a, &b, &c};
    for (int i = 0; i < 3; ++i) {
        PyObject* p = THPVariable_Wrap(*t[i]);
        if (!p) {
            Py_DECREF(out);
            throw Raised{};
        }
        PyTuple_SET_ITEM(out, i, p);
    }
    return out;
}

// The C call, with the interpreter free; f makes its outputs before it, so that the interpreter is left and taken once a call.
template <typename F>
void call(const char* where, F&& f) {
    int rc;
    {
        const Free free;
        rc = f();
    }
    check(rc, where);
}

template <typename F>
PyObject* guarded(Py_ssize_t got, Py_ssize_t want, F&& f) {
    HANDLE_TH_ERRORS
    if (got != want) {
        PyErr_Format(PyExc_TypeError, "%d arguments are needed, got %d", static_cast<int>(want), static_cast<int>(got));
        return nullptr;
    }
    try {
        return f();
    } catch (const Raised&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// k, update, bits, group, g, codes, scale, zero, stream
template <bool PC>
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() -> PyObject* {
        const at::Tensor& k = tensor(a[0]);
        need_device(k);
        const bool has_update = a[1] != Py_None;
        if (has_update) need_device(tensor(a[1]));
        need_dims(k, 4);
        const int64_t b = k.size(0), h = k.size(1), tokens = k.size(2), d = k.size(3);
        if (k.stride(3) != 1) raise(PyExc_ValueError, "k must have unit channel stride");
        const int bits = small(a[2]), group = small(a[3]), g = small(a[4]);
        if (PC && (group <= 0 || tokens % group)) raise(PyExc_ValueError, "n_tokens must be a multiple of group");
        int64_t usb = 0;
        const float* update = nullptr;
        if (has_update) {
            const at::Tensor& u = tensor(a[1]);
            if (u.scalar_type() != at::kFloat || !u.is_contiguous()) raise(PyExc_ValueError, "update must be dense float32");
            if (u.dim() == 4) usb = u.stride(0);
            update = pointer<const float>(u);
        }
        if (group == 0 && (a[6] == Py_None || a[7] == Py_None)) raise(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        const int per = group == 0 ? 1 : group;          // (outputs given: the library refuses the group)
        at::Tensor codes = given(a[5], k), scale = given(a[6], k), zero = given(a[7], k);
        const squat_dtype dt = dtype(a[0], k);
        const squat_stream s = stream(a[8]);
        const void* kp = pointer<void>(k);
        const int64_t s0 = k.stride(0), s1 = k.stride(1), s2 = k.stride(2);
        call(PC ? "squat_quantize_keys_per_channel" : "squat_quantize_keys", [&] {
            if (!codes.defined()) codes = PC ? empty({b, h, tokens / 32, d, bits}, at::kInt, k) : empty({b, h, tokens, d * bits / 32}, at::kInt, k);
            if (!scale.defined()) scale = PC ? empty({b, h, tokens / per, d}, at::kHalf, k) : empty({b, h, tokens, d / per}, at::kHalf, k);
            if (!zero.defined()) zero = PC ? empty({b, h, tokens / per, d}, at::kHalf, k) : empty({b, h, tokens, d / per}, at::kHalf, k);
            auto* cp = pointer<uint32_t>(codes);
            auto* sp = pointer<uint16_t>(scale);
            auto* zp = pointer<uint16_t>(zero);
            return (PC ? squat_quantize_keys_per_channel : squat_quantize_keys)(
                kp, dt, b, static_cast<int>(h), tokens, static_cast<int>(d), s0, s1, s2, update, usb, bits, group, g, cp, sp, zp, s);
        });
        return three(codes, scale, zero);
    });
}

void need_dense_store(const at::Tensor& codes, const at::Tensor& scale, const at::Tensor& zero) {
    if (!(codes.is_contiguous() && scale.is_contiguous() && zero.is_contiguous()))
        raise(PyExc_ValueError, "codes/scale/zero must be dense");
}

int64_t channels(int64_t words, int bits) {
    if (bits == 0) raise(PyExc_ZeroDivisionError, "integer division or modulo by zero");
    return words * 32 / bits;
}

// codes, scale, zero, bits, group, out_dtype (of an output made here; None: torch's default), out, stream
template <bool PC>
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 8, [&]() -> PyObject* {
        const at::Tensor &codes = tensor(a[0]), &scale = tensor(a[1]), &zero = tensor(a[2]);
        need_device(codes);
        need_device(scale);
        need_device(zero);
        need_dims(codes, PC ? 5 : 4);
        const int bits = small(a[3]), group = small(a[4]);
        const int64_t b = codes.size(0), h = codes.size(1);
        const int64_t tokens = PC ? codes.size(2) * 32 : codes.size(2);
        const int64_t d = PC ? codes.size(3) : channels(codes.size(3), bits);
        if (PC && codes.size(4) != bits) raise(PyExc_ValueError, "codes must be [B, H, n/32, d, bits]");
        need_dense_store(codes, scale, zero);
        at::Tensor out;
        if (a[6] == Py_None) {
            if (a[5] != Py_None && !THPDtype_Check(a[5])) raise(PyExc_TypeError, "out_dtype must be a torch.dtype");
            const at::ScalarType type = a[5] == Py_None ? at::get_default_dtype_as_scalartype() : reinterpret_cast<THPDtype*>(a[5])->scalar_type;
            const Free free;
            out = empty({b, h, tokens, d}, type, codes);
        } else {
            out = tensor(a[6]);
            need_reachable(out);
        }
        PyObject* wrapped = a[6] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(a[6]);
        if (!wrapped) throw Raised{};
        try {
            const squat_dtype dt = dtype(wrapped, out);
            const squat_stream s = stream(a[7]);
            const auto* cp = pointer<const uint32_t>(codes);
            const auto* sp = pointer<const uint16_t>(scale);
            const auto* zp = pointer<const uint16_t>(zero);
            void* op = pointer<void>(out);
            const int64_t s0 = out.stride(0), s1 = out.stride(1), s2 = out.stride(2);
            call(PC ? "squat_dequantize_keys_per_channel" : "squat_dequantize_keys", [&] {
                return (PC ? squat_dequantize_keys_per_channel : squat_dequantize_keys)(
                    cp, sp, zp, b, static_cast<int>(h), tokens, static_cast<int>(d), bits, group, op, dt, s0, s1, s2, s);
            });
        } catch (...) {
            Py_DECREF(wrapped);
            throw;
        }
        return wrapped;
    });
}

// q, codes, scale, zero, bits, group, q_per_kv, inv_freq, pos0, out_scale, out, stream; without rope inv_freq and pos0 are not looked
// at.  (Two functions and not one that goes by inv_freq: a caller who lacks the frequencies gets an error, no unrotated logits.)
template <bool PC, bool rope>
PyObject* key_scores(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 12, [&]() -> PyObject* {
        const at::Tensor &q = tensor(a[0]), &codes = tensor(a[1]), &scale = tensor(a[2]), &zero = tensor(a[3]);
        const int bits = small(a[4]), group = small(a[5]), qpk = small(a[6]);
        if constexpr (rope) need_device(tensor(a[7]));
        (PC && !rope ? need_reachable : need_device)(q);
        (PC && !rope ? need_reachable : need_device)(codes);
        (PC || rope ? need_reachable : need_device)(scale);
        (PC || rope ? need_reachable : need_device)(zero);
        need_dims(codes, PC ? 5 : 4);
        const int64_t b = codes.size(0), h = codes.size(1);
        const int64_t tokens = PC ? codes.size(2) * 32 : codes.size(2);
        const int64_t d = PC ? codes.size(3) : (rope ? 128 : channels(codes.size(3), bits));
        if (PC && (codes.size(4) != bits || scale.sizes() != at::IntArrayRef({b, h, codes.size(2), d}) || zero.sizes() != scale.sizes()))
            raise(PyExc_ValueError, "codes [B,H,n/32,d,bits], scale/zero [B,H,n/32,d] expected");
        const float* freq = nullptr;
        if constexpr (rope) {
            const at::Tensor& f = tensor(a[7]);
            if (f.scalar_type() != at::kFloat || f.numel() != 64 || !f.is_contiguous())
                raise(PyExc_ValueError, "inv_freq must be 64 dense float32 values");
            freq = pointer<const float>(f);
        }
        if (q.dim() != 3 || q.size(0) != b || q.size(1) != h * qpk || q.size(2) != d || q.stride(2) != 1)
            raise(PyExc_ValueError, "q must be [B, n_kv_heads*q_per_kv, d] with unit channel stride");
        need_dense_store(codes, scale, zero);
        at::Tensor out = given(a[10], codes);
        if (out.defined() && (out.scalar_type() != at::kFloat || out.stride(2) != 1 || out.size(0) != b || out.size(1) != h * qpk))
            raise(PyExc_ValueError, "out must be float32 [B, n_q_heads, >= n] with unit token stride");
        const squat_dtype dt = dtype(a[0], q);
        const long long pos0 = rope ? integer(a[8]) : 0;
        const float out_scale = number(a[9]);
        const squat_stream s = stream(a[11]);
        const auto* cp = pointer<const uint32_t>(codes);
        const auto* sp = pointer<const uint16_t>(scale);
        const auto* zp = pointer<const uint16_t>(zero);
        const void* qp = pointer<void>(q);
        const int64_t q0 = q.stride(0), q1 = q.stride(1);
        const int hi = static_cast<int>(h), di = static_cast<int>(d);
        auto make = [&] {
            if (!out.defined()) out = empty({b, h * qpk, tokens}, at::kFloat, codes);
        };
        if constexpr (rope)
            call(PC ? "squat_key_scores_rope_per_channel" : "squat_key_scores_rope", [&] {
                make();
                return (PC ? squat_key_scores_rope_per_channel : squat_key_scores_rope)(
                    cp, sp, zp, b, hi, tokens, di, bits, group, freq, pos0, qp, dt, qpk, q0, q1, out_scale, pointer<float>(out), out.stride(0),
                    out.stride(1), s);
            });
        else
            call(PC ? "squat_key_scores_per_channel" : "squat_key_scores", [&] {
                make();
                return (PC ? squat_key_scores_per_channel : squat_key_scores)(cp, sp, zp, b, hi, tokens, di, bits, group, qp, dt, qpk, q0, q1,
                                                                             out_scale, pointer<float>(out), out.stride(0), out.stride(1), s);
            });
        return a[10] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(a[10]);
    });
}

squat_cache* cache(PyObject* o) {            // None (a destroyed cache): the library refuses it
    if (o == Py_None) return nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Raised{};
    return static_cast<squat_cache*>(p);
}

// handle, k, v, stream
PyObject* cache_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 4, [&]() -> PyObject* {
        squat_cache* c = cache(a[0]);
        const at::Tensor& k = tensor(a[1]);
        need_device(k);
        const void* vp = nullptr;
        if (a[2] != Py_None) {
            const at::Tensor& v = tensor(a[2]);
            need_device(v);
            if (v.strides() != k.strides()) raise(PyExc_ValueError, "k and v must share their strides");
            vp = pointer<void>(v);
        }
        const void* kp = pointer<void>(k);
        const int64_t s0 = k.stride(0), s1 = k.stride(1);
        const squat_stream s = stream(a[3]);
        call("squat_cache_append", [&] { return squat_cache_append(c, kp, vp, s0, s1, s); });
        Py_RETURN_NONE;
    });
}

// handle, q, inv_freq, pos0, out_scale, out, stream; without rope inv_freq and pos0 are not looked at
template <bool rope>
PyObject* cache_key_scores(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&]() -> PyObject* {
        const at::Tensor& q = tensor(a[1]);
        need_device(q);
        squat_cache* c = cache(a[0]);
        const float* freq = nullptr;
        if constexpr (rope) {
            const at::Tensor& f = tensor(a[2]);
            need_device(f);
            if (f.scalar_type() != at::kFloat || !f.is_contiguous()) raise(PyExc_ValueError, "inv_freq must be dense float32");
            freq = pointer<const float>(f);
        }
        squat_cache_counts counts;
        check(squat_cache_state(c, &counts), "squat_cache_state");
        at::Tensor out;
        if (a[5] == Py_None) {
            if (q.dim() < 2) raise(PyExc_IndexError, "q must be [B, H*q_per_kv, d]");
        } else {
            out = tensor(a[5]);
            need_reachable(out);
        }
        const squat_dtype dt = dtype(a[1], q);
        const long long pos0 = rope ? integer(a[3]) : 0;
        const float out_scale = number(a[4]);
        const squat_stream s = stream(a[6]);
        const void* qp = pointer<void>(q);
        const int64_t q0 = q.stride(0), q1 = q.stride(1);
        call(rope ? "squat_cache_key_scores_rope" : "squat_cache_key_scores", [&] {
            if (!out.defined()) out = empty({q.size(0), q.size(1), counts.keys_quantized + counts.keys_residual}, at::kFloat, q);
            float* op = pointer<float>(out);
            const int64_t o0 = out.stride(0), o1 = out.stride(1);
            if constexpr (rope) return squat_cache_key_scores_rope(c, qp, dt, q0, q1, freq, pos0, out_scale, op, o0, o1, s);
            else return squat_cache_key_scores(c, qp, dt, q0, q1, out_scale, op, o0, o1, s);
        });
        return a[5] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(a[5]);
    });
}

PyObject* set_error(PyObject*, PyObject* cls) {
    Py_XINCREF(cls);
    Py_XSETREF(squat_error, cls);
    Py_RETURN_NONE;
}

#define SQUAT_FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SQUAT_FAST("quantize_keys", quantize<false>),
    SQUAT_FAST("quantize_keys_per_channel", quantize<true>),
    SQUAT_FAST("dequantize_keys", dequantize<false>),
    SQUAT_FAST("dequantize_keys_per_channel", dequantize<true>),
    SQUAT_FAST("key_scores", (key_scores<false, false>)),
    SQUAT_FAST("key_scores_per_channel", (key_scores<true, false>)),
    SQUAT_FAST("key_scores_rope", (key_scores<false, true>)),
    SQUAT_FAST("key_scores_rope_per_channel", (key_scores<true, true>)),
    SQUAT_FAST("cache_append", cache_append),
    SQUAT_FAST("cache_key_scores", cache_key_scores<false>),
    SQUAT_FAST("cache_key_scores_rope", cache_key_scores<true>),
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_squat_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__squat_torch() { return PyModule_Create(&module); }
