// _tkcall: the Python call path of the C entry points (include/tk_attn.h) in C++.
//
// A short call's cost is on the host: marshalled in Python (checks, output
// allocation, current stream, ctypes conversions) a call took 10 to 12 us while
// its kernel runs for 2 to 5, so small prompts, training steps and appends waited
// for the interpreter. Here the same steps take about the launch itself.
//
//   prefill, prefill_lse, prefill_backward, cache_append, project_heads
//       the plain entry points' arguments in binding.py's order. They return None
//       for any call that they do not take (tensors that are not plain CUDA ones,
//       shapes or types that do not fit, a stream given, active function or
//       dispatch modes): binding.py then marshals it, and raises what is wrong with
//       it. A C status other than TK_OK is returned as an int.
//   bind(name, args)
//       a callable that makes the C call with the tuple's arguments and returns its
//       status. It reads them anew each time (a ctypes object's value can be set).
//   plain_args(args)
//       whether they are a tuple of ints, floats, None and ctypes pointers alone.
//
// The library's functions are reached through addresses set by connect(), which
// binding.py takes from the library it has loaded: one copy of it per process.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include <string.h>

#include <memory>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>

#include "tk_attn.h"

namespace {

struct Entries {
    decltype(&tk_attn_prefill) prefill = nullptr;
    decltype(&tk_attn_prefill_lse) prefill_lse = nullptr;
    decltype(&tk_attn_prefill_backward) prefill_backward = nullptr;
    decltype(&tk_attn_prefill_backward_workspace_bytes) backward_workspace = nullptr;
    decltype(&tk_attn_decode) decode = nullptr;
    decltype(&tk_attn_decode_noalloc) decode_noalloc = nullptr;
    decltype(&tk_cache_append) append = nullptr;
    decltype(&tk_project_heads) project = nullptr;
} g;

struct NoGil {
    PyThreadState* state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

// ------------------------------------------------------------------ plain calls

// A plain strided, contiguous CUDA tensor of this type and rank: no subclass, no
// wrapper of a transform. Null otherwise.
const at::Tensor* plain(PyObject* o, at::ScalarType type, int64_t dim) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    constexpr c10::DispatchKeySet odd{c10::DispatchKey::Python, c10::DispatchKey::FuncTorchGradWrapper,
                                      c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::Functionalize};
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || t.key_set().has_any(odd)) return nullptr;
    if (t.scalar_type() != type || t.dim() != dim || !t.is_contiguous()) return nullptr;
    return &t;
}
bool modes_active() {
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}
bool is_bool(PyObject* o) { return o == Py_True || o == Py_False; }
// An output: the given tensor if it fits, a new one for None; `ok` false otherwise.
at::Tensor output(PyObject* o, at::IntArrayRef shape, const at::Tensor& like, at::ScalarType type, bool& ok) {
    if (o == Py_None) return {};
    const at::Tensor* t = plain(o, type, (int64_t)shape.size());
    ok = ok && t && t->sizes() == shape && t->device() == like.device();
    return t ? *t : at::Tensor();
}
void fill_in(at::Tensor& t, at::IntArrayRef shape, const at::Tensor& like, at::ScalarType type) {
    if (!t.defined()) t = at::empty(shape, like.options().dtype(type).requires_grad(false));
}
template <class... T>
bool fit_int(T... sizes) {
    return ((sizes <= 0x7fffffffL) && ...);
}
hipStream_t stream_now() { return c10::hip::getCurrentHIPStream().stream(); }
PyObject* status_of(tk_status s) { return PyLong_FromLong((long)s); }

struct Shapes {
    int64_t B, Hq, Hkv, Sq, Sk, r, dv;
};
bool prefill_shapes(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, Shapes& s) {
    s = {q.size(0), q.size(1), v.size(1), q.size(2), v.size(2), q.size(3), v.size(3)};
    return k.size(0) == s.B && k.size(1) == s.Hkv && k.size(2) == s.Sk && k.size(3) == s.r && v.size(0) == s.B &&
           fit_int(s.B, s.Hq, s.Hkv, s.Sq, s.Sk, s.r, s.dv);
}

// (Q, K, V, O, causal, scale, stream)
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 7 || a[6] != Py_None || !is_bool(a[4]) || !PyFloat_CheckExact(a[5]) || modes_active()) Py_RETURN_NONE;
    const at::Tensor* q = plain(a[0], at::kBFloat16, 4);
    const at::ScalarType type = q ? at::kBFloat16 : at::kFloat;
    if (!q) q = plain(a[0], at::kFloat, 4);
    const at::Tensor *k = plain(a[1], type, 4), *v = plain(a[2], type, 4);
    Shapes s;
    if (!q || !k || !v || !prefill_shapes(*q, *k, *v, s)) Py_RETURN_NONE;
    bool ok = true;
    const int64_t shape[4] = {s.B, s.Hq, s.Sq, s.dv};
    at::Tensor o = output(a[3], shape, *q, type, ok);
    if (!ok) Py_RETURN_NONE;
    const bool causal = a[4] == Py_True;
    const float scale = (float)PyFloat_AS_DOUBLE(a[5]);
    tk_status st;
    {
        NoGil nogil;
        fill_in(o, shape, *q, type);
        st = g.prefill(q->data_ptr(), k->data_ptr(), v->data_ptr(), o.data_ptr(), (int)s.B, (int)s.Hq, (int)s.Hkv,
                       (int)s.Sq, (int)s.Sk, (int)s.r, (int)s.dv, causal, scale,
                       type == at::kBFloat16 ? TK_BF16 : TK_F32, stream_now());
    }
    if (st != TK_OK) return status_of(st);
    if (a[3] != Py_None) return Py_NewRef(a[3]);
    return THPVariable_Wrap(std::move(o));
    END_HANDLE_TH_ERRORS
}

// (Q, K, V, O, lse, causal, scale, stream)
PyObject* prefill_lse(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 8 || a[7] != Py_None || !is_bool(a[5]) || !PyFloat_CheckExact(a[6]) || modes_active()) Py_RETURN_NONE;
    const at::Tensor *q = plain(a[0], at::kBFloat16, 4), *k = plain(a[1], at::kBFloat16, 4),
                     *v = plain(a[2], at::kBFloat16, 4);
    Shapes s;
    if (!q || !k || !v || !prefill_shapes(*q, *k, *v, s)) Py_RETURN_NONE;
    bool ok = true;
    const int64_t shape[4] = {s.B, s.Hq, s.Sq, s.dv};
    at::Tensor o = output(a[3], shape, *q, at::kBFloat16, ok);
    at::Tensor lse = output(a[4], at::IntArrayRef(shape, 3), *q, at::kFloat, ok);
    if (!ok) Py_RETURN_NONE;
    const bool causal = a[5] == Py_True;
    const float scale = (float)PyFloat_AS_DOUBLE(a[6]);
    tk_status st;
    {
        NoGil nogil;
        fill_in(o, shape, *q, at::kBFloat16);
        fill_in(lse, at::IntArrayRef(shape, 3), *q, at::kFloat);
        st = g.prefill_lse(q->data_ptr(), k->data_ptr(), v->data_ptr(), o.data_ptr(), (float*)lse.data_ptr(),
                           (int)s.B, (int)s.Hq, (int)s.Hkv, (int)s.Sq, (int)s.Sk, (int)s.r, (int)s.dv, causal, scale,
                           stream_now());
    }
    if (st != TK_OK) return status_of(st);
    THPObjectPtr po(a[3] != Py_None ? Py_NewRef(a[3]) : THPVariable_Wrap(std::move(o)));
    THPObjectPtr pl(a[4] != Py_None ? Py_NewRef(a[4]) : THPVariable_Wrap(std::move(lse)));
    return po && pl ? PyTuple_Pack(2, po.get(), pl.get()) : nullptr;
    END_HANDLE_TH_ERRORS
}

// (Q, K, V, O, dO, lse, causal, scale, dQ, dK, dV, workspace, stream)
PyObject* prefill_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 13 || a[11] != Py_None || a[12] != Py_None || !is_bool(a[6]) || !PyFloat_CheckExact(a[7]) ||
        modes_active())
        Py_RETURN_NONE;
    const at::Tensor *q = plain(a[0], at::kBFloat16, 4), *k = plain(a[1], at::kBFloat16, 4),
                     *v = plain(a[2], at::kBFloat16, 4), *o = plain(a[3], at::kBFloat16, 4),
                     *d_o = plain(a[4], at::kBFloat16, 4), *lse = plain(a[5], at::kFloat, 3);
    Shapes s;
    if (!q || !k || !v || !o || !d_o || !lse || !prefill_shapes(*q, *k, *v, s)) Py_RETURN_NONE;
    const int64_t shape[4] = {s.B, s.Hq, s.Sq, s.dv};
    if (o->sizes() != at::IntArrayRef(shape) || d_o->sizes() != at::IntArrayRef(shape) ||
        lse->sizes() != at::IntArrayRef(shape, 3))
        Py_RETURN_NONE;
    bool ok = true;
    const at::Tensor* like[3] = {q, k, v};
    at::Tensor grad[3];
    for (int i = 0; i < 3; ++i) grad[i] = output(a[8 + i], like[i]->sizes(), *q, at::kBFloat16, ok);
    if (!ok) Py_RETURN_NONE;
    const bool causal = a[6] == Py_True;
    const float scale = (float)PyFloat_AS_DOUBLE(a[7]);
    tk_status st;
    {
        NoGil nogil;
        for (int i = 0; i < 3; ++i) fill_in(grad[i], like[i]->sizes(), *like[i], at::kBFloat16);
        const size_t bytes = g.backward_workspace((int)s.B, (int)s.Hq, (int)s.Sq);
        at::Tensor ws;
        fill_in(ws, (int64_t)bytes, *q, at::kByte);
        st = g.prefill_backward(q->data_ptr(), k->data_ptr(), v->data_ptr(), o->data_ptr(), d_o->data_ptr(),
                                (const float*)lse->data_ptr(), grad[0].data_ptr(), grad[1].data_ptr(),
                                grad[2].data_ptr(), (int)s.B, (int)s.Hq, (int)s.Hkv, (int)s.Sq, (int)s.Sk, (int)s.r,
                                (int)s.dv, causal, scale, ws.data_ptr(), bytes, stream_now());
    }
    if (st != TK_OK) return status_of(st);
    THPObjectPtr out(PyTuple_New(3));
    if (!out) return nullptr;
    for (int i = 0; i < 3; ++i) {
        PyObject* t = a[8 + i] != Py_None ? Py_NewRef(a[8 + i]) : THPVariable_Wrap(std::move(grad[i]));
        if (!t) return nullptr;
        PyTuple_SET_ITEM(out.get(), i, t);
    }
    return out.release();
    END_HANDLE_TH_ERRORS
}

// (X, Wt, n_heads, Y, stream)
PyObject* project_heads(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 5 || a[4] != Py_None || !PyLong_CheckExact(a[2]) || modes_active()) Py_RETURN_NONE;
    const at::Tensor *x = plain(a[0], at::kBFloat16, 3), *w = plain(a[1], at::kBFloat16, 2);
    int over = 0;
    const int64_t heads = PyLong_AsLongAndOverflow(a[2], &over);
    if (!x || !w || over || heads <= 0 || heads > 0x7fffffffL || w->size(0) % heads || w->size(1) != x->size(2))
        Py_RETURN_NONE;
    const int64_t width = w->size(0) / heads;
    const int64_t shape[4] = {x->size(0), heads, x->size(1), width};
    if (!fit_int(shape[0], shape[2], width, x->size(2))) Py_RETURN_NONE;
    bool ok = true;
    at::Tensor y = output(a[3], shape, *x, at::kBFloat16, ok);
    if (!ok) Py_RETURN_NONE;
    tk_status st;
    {
        NoGil nogil;
        fill_in(y, shape, *x, at::kBFloat16);
        st = g.project(x->data_ptr(), w->data_ptr(), y.data_ptr(), (int)shape[0], (int)shape[2], (int)x->size(2),
                       (int)heads, (int)width, stream_now());
    }
    if (st != TK_OK) return status_of(st);
    if (a[3] != Py_None) return Py_NewRef(a[3]);
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

// (K_new, V_new, positions, K_cache, V_cache, k_scale, block_table, block_size, stream); True when done
PyObject* cache_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 9 || a[8] != Py_None || !PyLong_CheckExact(a[7]) || modes_active()) Py_RETURN_NONE;
    const at::Tensor *kn = plain(a[0], at::kBFloat16, 4), *vn = plain(a[1], at::kBFloat16, 4),
                     *pos = plain(a[2], at::kInt, 1), *kc = plain(a[3], at::kBFloat16, 4),
                     *vc = plain(a[4], at::kBFloat16, 4);
    const bool quantised = !kc;
    if (!kc) kc = plain(a[3], at::kByte, 4);
    if (!kn || !vn || !pos || !kc || !vc) Py_RETURN_NONE;
    const int64_t B = kn->size(0), Hkv = kn->size(1), T = kn->size(2), r = kn->size(3), dv = vn->size(3);
    if (vn->size(0) != B || vn->size(1) != Hkv || vn->size(2) != T || pos->size(0) != B) Py_RETURN_NONE;
    tk_dtype format = TK_BF16;
    if (quantised) {
        if (kc->size(3) == r)
            format = TK_FP8_E4M3;
        else if (kc->size(3) * 2 == r)
            format = TK_INT4;
        else
            Py_RETURN_NONE;
    } else if (kc->size(3) != r) {
        Py_RETURN_NONE;
    }
    const at::Tensor* scale = nullptr;
    if (quantised != (a[5] != Py_None)) Py_RETURN_NONE;
    if (quantised && !(scale = plain(a[5], at::kFloat, 3))) Py_RETURN_NONE;
    for (int i = 0; i < 3; ++i) {
        if (kc->size(i) != vc->size(i)) Py_RETURN_NONE;
        if (scale && scale->size(i) != kc->size(i)) Py_RETURN_NONE;
    }
    if (kc->size(1) != Hkv || vc->size(3) != dv) Py_RETURN_NONE;
    int64_t max_ctx = 0, mb = 0, blocks = 0, block = 0;
    const at::Tensor* table = nullptr;
    if (a[6] == Py_None) {
        if (kc->size(0) != B) Py_RETURN_NONE;
        max_ctx = kc->size(2);
    } else {
        int over = 0;
        block = PyLong_AsLongAndOverflow(a[7], &over);
        table = plain(a[6], at::kInt, 2);
        if (!table || over || table->size(0) != B || block != kc->size(2)) Py_RETURN_NONE;
        mb = table->size(1);
        blocks = kc->size(0);
    }
    if (!fit_int(B, Hkv, T, r, dv, max_ctx, mb, blocks, block)) Py_RETURN_NONE;
    tk_status st;
    {
        NoGil nogil;
        st = g.append(kn->data_ptr(), vn->data_ptr(), (int)B, (int)Hkv, (int)T, (int)r, (int)dv,
                      (const int32_t*)pos->data_ptr(), kc->data_ptr(), vc->data_ptr(), (int)max_ctx, format,
                      scale ? (float*)scale->data_ptr() : nullptr, table ? (const int32_t*)table->data_ptr() : nullptr,
                      (int)block, (int)mb, (int)blocks, stream_now());
    }
    if (st != TK_OK) return status_of(st);
    Py_RETURN_TRUE;
    END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------ bound calls

PyObject* c_void_p() {
    static PyObject* const type = [] {
        THPObjectPtr ctypes(PyImport_ImportModule("ctypes"));
        return ctypes ? PyObject_GetAttrString(ctypes.get(), "c_void_p") : nullptr;
    }();
    return type;
}

// A c_void_p's value, from its storage (its attribute would first become a Python integer).
bool read_pointer(PyObject* o, void** out) {
    Py_buffer at;
    if (PyObject_GetBuffer(o, &at, PyBUF_SIMPLE) < 0) return false;
    memcpy(out, at.buf, sizeof *out);
    PyBuffer_Release(&at);
    return true;
}

// One marshalled argument (an int, a float, None, or a ctypes object holding one),
// converted as ctypes does: integers modulo the type's width, None and a c_void_p for
// pointers alone.
template <class T>
bool convert(PyObject* o, T& out) {
    static PyObject* const value = PyUnicode_InternFromString("value");
    THPObjectPtr held;
    if (o == Py_None || (PyObject*)Py_TYPE(o) == c_void_p()) {
        if constexpr (std::is_pointer_v<T>) {
            out = nullptr;
            return o == Py_None || read_pointer(o, (void**)&out);
        }
        PyErr_SetString(PyExc_TypeError, "a number is needed");
        return false;
    }
    if (!PyLong_Check(o) && !PyFloat_Check(o)) {
        held = PyObject_GetAttr(o, value);
        if (!held) return false;
        o = held.get();
    }
    if constexpr (std::is_same_v<T, float>) {
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) return false;
        out = (float)v;
    } else {
        const unsigned long long v = o == Py_None ? 0 : PyLong_AsUnsignedLongLongMask(o);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
        if constexpr (std::is_pointer_v<T>)
            out = (T)(uintptr_t)v;
        else
            out = (T)v;
    }
    return true;
}

// An entry point called with a tuple's arguments: its status, or -1 with an error set.
// The tuple and its numbers cannot change, the value of a c_void_p can: that is read for
// each call (0.23 us of host work a prepared projection; 0.48 with every argument
// converted again, 0.19 with none).
struct Call {
    virtual ~Call() = default;
    virtual bool take(PyObject* args) = 0;
    virtual int run(PyObject* args) const = 0;
};
template <class... A>
struct Bound : Call {
    tk_status (*fn)(A...);
    std::tuple<A...> taken;
    bool reread[sizeof...(A)];
    explicit Bound(tk_status (*f)(A...)) : fn(f) {}
    bool take(PyObject* args) override {
        if (PyTuple_GET_SIZE(args) != (Py_ssize_t)sizeof...(A)) {
            PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
            return false;
        }
        return take(args, std::index_sequence_for<A...>{});
    }
    int run(PyObject* args) const override { return run(args, std::index_sequence_for<A...>{}); }
    template <size_t... I>
    bool take(PyObject* args, std::index_sequence<I...>) {
        ((reread[I] = (PyObject*)Py_TYPE(PyTuple_GET_ITEM(args, I)) == c_void_p()), ...);
        return (convert(PyTuple_GET_ITEM(args, I), std::get<I>(taken)) && ...);
    }
    template <size_t... I>
    int run(PyObject* args, std::index_sequence<I...>) const {
        std::tuple<A...> v = taken;
        if (!((!reread[I] || convert(PyTuple_GET_ITEM(args, I), std::get<I>(v))) && ...)) return -1;
        NoGil nogil;
        return std::apply(fn, v);
    }
};
template <class... A>
std::unique_ptr<Call> call_of(tk_status (*fn)(A...)) {
    return std::make_unique<Bound<A...>>(fn);
}

struct BoundObject {
    PyObject_HEAD
    Call* call;
    PyObject* args;
};
void bound_dealloc(PyObject* self) {
    delete ((BoundObject*)self)->call;
    Py_XDECREF(((BoundObject*)self)->args);
    Py_TYPE(self)->tp_free(self);
}
PyObject* bound_call(PyObject* self, PyObject*, PyObject*) {
    const BoundObject* b = (const BoundObject*)self;
    const int st = b->call->run(b->args);
    return st < 0 ? nullptr : PyLong_FromLong(st);
}
PyTypeObject BoundType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 2 || !PyUnicode_Check(a[0]) || !PyTuple_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "bind(name, args)");
        return nullptr;
    }
    const std::string name = PyUnicode_AsUTF8(a[0]);
    std::unique_ptr<Call> call;
    if (name == "tk_attn_prefill")
        call = call_of(g.prefill);
    else if (name == "tk_attn_prefill_lse")
        call = call_of(g.prefill_lse);
    else if (name == "tk_attn_prefill_backward")
        call = call_of(g.prefill_backward);
    else if (name == "tk_attn_decode")
        call = call_of(g.decode);
    else if (name == "tk_attn_decode_noalloc")
        call = call_of(g.decode_noalloc);
    else if (name == "tk_cache_append")
        call = call_of(g.append);
    else if (name == "tk_project_heads")
        call = call_of(g.project);
    else
        return PyErr_Format(PyExc_ValueError, "no entry point %s", name.c_str());
    if (!call->take(a[1])) return nullptr;
    BoundObject* o = PyObject_New(BoundObject, &BoundType);
    if (!o) return nullptr;
    o->call = call.release();
    o->args = Py_NewRef(a[1]);
    return (PyObject*)o;
    END_HANDLE_TH_ERRORS
}

// (args): whether bind() reads them as ctypes would, each being exactly one of the
// types that it converts
PyObject* plain_args(PyObject*, PyObject* args) {
    PyObject* const pointer = c_void_p();
    if (!pointer) return nullptr;
    bool plain = PyTuple_CheckExact(args);
    for (Py_ssize_t i = 0; plain && i < PyTuple_GET_SIZE(args); ++i) {
        PyObject* o = PyTuple_GET_ITEM(args, i);
        plain = o == Py_None || PyLong_CheckExact(o) || PyFloat_CheckExact(o) || (PyObject*)Py_TYPE(o) == pointer;
    }
    return PyBool_FromLong(plain);
}

// connect(address of each entry point, in this order)
PyObject* connect(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void** const to[] = {(void**)&g.prefill, (void**)&g.prefill_lse, (void**)&g.prefill_backward,
                         (void**)&g.backward_workspace, (void**)&g.decode, (void**)&g.decode_noalloc,
                         (void**)&g.append, (void**)&g.project};
    if (n != (Py_ssize_t)(sizeof to / sizeof *to)) {
        PyErr_SetString(PyExc_TypeError, "connect() takes one address per entry point");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        void* p = PyLong_AsVoidPtr(a[i]);
        if (!p) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
        *to[i] = p;
    }
    Py_RETURN_NONE;
}

#define METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(prefill),      METHOD(prefill_lse), METHOD(prefill_backward), METHOD(project_heads),
                         METHOD(cache_append), METHOD(bind),        METHOD(connect),          {"plain_args", plain_args, METH_O, nullptr},
                         {}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tkcall", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__tkcall(void) {
    BoundType.tp_name = "_tkcall.Bound";
    BoundType.tp_basicsize = sizeof(BoundObject);
    BoundType.tp_flags = Py_TPFLAGS_DEFAULT;
    BoundType.tp_dealloc = bound_dealloc;
    BoundType.tp_call = bound_call;
    if (PyType_Ready(&BoundType) < 0) return nullptr;
    return PyModule_Create(&module);
}
