// Marshalling of the hot entry points of binding.py in native code: argument checks, output and
// scratch allocation through torch's allocator, the current stream, the call.  A small call is bound
// by the host, and most of its time was this work done in Python and ctypes.
//
// Every function takes the arguments of its namesake in binding.py, in order, and returns its result,
// or None for whatever is not the plain case (a wrong shape, type or device, a tensor subclass, an
// active function mode, an argument that the library refuses): the caller then takes the Python path,
// which raises the error or does the unusual thing.  The library refuses arguments before it launches
// anything, so a call that returned None has had no effect.  A launch that fails is another matter: a
// state updated in place may have moved by then (the runtime also reports, with the next launch, an error
// that something else left in the thread), so that status is raised here and the call is not made again.
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <array>

#include "../../include/ltn_attn.h"

namespace {

// Entry points of the library that binding.py has opened (bind() below, in this order).
#define LTN_LIBRARY(X)                                                                                           \
    X(fwd, ltn_attn_fwd) X(fwd_gated, ltn_attn_fwd_gated) X(bwd, ltn_attn_bwd) X(gate_bwd, ltn_gate_bwd)         \
    X(decode_steps, ltn_attn_decode_steps) X(workspace_bytes, ltn_attn_workspace_bytes)                          \
    X(fwd_dkdv, ltn_attn_fwd_dkdv) X(bwd_dkdv, ltn_attn_bwd_dkdv)                                                \
    X(decode_steps_dkdv, ltn_attn_decode_steps_dkdv) X(workspace_bytes_dkdv, ltn_attn_workspace_bytes_dkdv)      \
    X(prologue_fwd, ltn_prologue_fwd) X(prologue_bwd, ltn_prologue_bwd)                                          \
    X(prologue_workspace_bytes, ltn_prologue_workspace_bytes)
struct Library {
#define LTN_FIELD(field, symbol) decltype(&symbol) field;
    LTN_LIBRARY(LTN_FIELD)
#undef LTN_FIELD
} lib = {};

PyObject* error_type = nullptr;            // binding.py's LtnError

// Thrown where the plain case ends; becomes None.
struct NotPlain {};

// Thrown with a status that may have come after a launch; becomes an LtnError.
struct Failed {
    const char* where;
    ltn_status status;
};

void need(bool ok) {
    if (!ok) throw NotPlain{};
}

// The call's device (the current one) and checks of single arguments against it.
struct Args {
    PyObject* const* a;
    c10::DeviceIndex device;

    Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : a(args) {
        need(n == want && lib.fwd && !at::impl::torch_function_mode_enabled());
        need(THPVariable_CheckExact(a[0]));
        const at::Tensor& t = THPVariable_Unpack(a[0]);
        need(t.is_cuda());
        device = t.device().index();
        need(c10::hip::current_device() == device);
    }
    // a plain, contiguous tensor with storage on the call's device
    const at::Tensor& tensor(int i) const {
        need(THPVariable_CheckExact(a[i]));
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        need(t.is_cuda() && t.device().index() == device && t.layout() == c10::kStrided && t.has_storage() &&
             t.is_contiguous() && !t.is_neg());
        return t;
    }
    bool none(int i) const { return a[i] == Py_None; }
    bool flag(int i) const {
        need(PyBool_Check(a[i]));
        return a[i] == Py_True;
    }
    long long integer(int i) const {
        need(PyLong_CheckExact(a[i]));
        const long long v = PyLong_AsLongLong(a[i]);
        if (v == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            throw NotPlain{};
        }
        return v;
    }
    int int32(int i) const {
        const long long v = integer(i);
        need(v >= INT32_MIN && v <= INT32_MAX);
        return (int)v;
    }
    float real(int i) const { return PyFloat_CheckExact(a[i]) ? (float)PyFloat_AS_DOUBLE(a[i]) : (float)int32(i); }
    const float* decay(int i, int64_t H) const {
        const at::Tensor& t = tensor(i);
        need(t.scalar_type() == at::kFloat && t.numel() == H);
        return (const float*)t.data_ptr();
    }
    // an fp32 state argument of the given shape, or nullptr
    float* state(int i, at::IntArrayRef shape) const {
        if (none(i)) return nullptr;
        const at::Tensor& t = tensor(i);
        need(t.scalar_type() == at::kFloat && t.sizes() == shape);
        return (float*)t.data_ptr();
    }
    void* stream() const { return c10::hip::getCurrentHIPStream(device).stream(); }
};

// An output: the caller's tensor (of the right type and with enough elements, in whatever shape), or a new
// one.
struct Out {
    PyObject* given = nullptr;
    at::Tensor made;
    void* ptr = nullptr;
    Out() = default;
    Out(const Args& args, int i, const at::Tensor& like) {
        if (args.none(i)) make(at::empty_like(like));
        else take(args, i, like.scalar_type(), like.numel());
    }
    void make(at::Tensor t) {
        made = std::move(t);
        ptr = made.data_ptr();
    }
    void take(const Args& args, int i, at::ScalarType type, int64_t numel) {
        const at::Tensor& t = args.tensor(i);
        need(t.scalar_type() == type && t.numel() >= numel);
        ptr = t.data_ptr();
        given = args.a[i];
    }
    // a state: the caller's, a new one when `want`, or none
    void state(const Args& args, int i, bool want, const std::array<int64_t, 4>& shape, const at::Tensor& like) {
        if (!args.none(i)) take(args, i, at::kFloat, shape[0] * shape[1] * shape[2] * shape[3]);
        else if (want) make(at::empty(shape, like.options().dtype(at::kFloat)));
    }
    PyObject* object() const {             // a new reference
        if (!given) return THPVariable_Wrap(made);
        Py_INCREF(given);
        return given;
    }
};

ltn_dtype dtype_of(const at::Tensor& t) {
    need(t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16);
    return t.scalar_type() == at::kFloat ? LTN_F32 : LTN_BF16;
}

void same(const at::Tensor& q, const at::Tensor& t) { need(t.scalar_type() == q.scalar_type() && t.sizes() == q.sizes()); }

struct Dims {
    int Bt, H, D;
    long long N;
    explicit Dims(const at::Tensor& q) {
        need(q.dim() == 4);
        for (int i : {0, 1, 3}) need(q.size(i) <= INT32_MAX);
        Bt = (int)q.size(0);
        H = (int)q.size(1);
        N = q.size(2);
        D = (int)q.size(3);
    }
};

at::Tensor scratch(size_t bytes, const at::Tensor& like) {
    return bytes ? at::empty({(int64_t)bytes}, like.options().dtype(at::kByte)) : at::Tensor();
}

// The interpreter is not held while one of these lives, and is again however its scope is left.
struct Released {
    PyThreadState* const state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
};

// The library's call `f`, as ctypes makes it: without the interpreter.  `f` also asks the tensors for
// their addresses, which may throw (a storage that refuses access, a lazy copy that finds no memory).
template <class F>
void call(const char* where, F&& f) {
    const ltn_status s = [&] {
        const Released released;
        return f();
    }();
    switch (s) {
        case LTN_OK: return;
        case LTN_ERR_NULL:                 // found before any launch
        case LTN_ERR_SHAPE:
        case LTN_ERR_UNSUPPORTED:
        case LTN_ERR_ALIGN: throw NotPlain{};
        default: throw Failed{where, s};
    }
}

void* at_or_null(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

template <int N>
PyObject* tuple(const Out* (&outs)[N]) {
    PyObject* t = PyTuple_New(N);
    if (!t) throw python_error();
    for (int i = 0; i < N; ++i) {
        PyObject* o = nullptr;
        if (outs[i]) {
            o = outs[i]->object();
        } else {
            Py_INCREF(Py_None);
            o = Py_None;
        }
        if (!o) {
            Py_DECREF(t);
            throw python_error();
        }
        PyTuple_SET_ITEM(t, i, o);
    }
    return t;
}

// q, k, v, decay, kv_in, return_state, block, out, kv_out
PyObject* fwd(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2);
    const Dims d(q);
    same(q, k);
    same(q, v);
    const ltn_dtype dt = dtype_of(q);
    const std::array<int64_t, 4> state = {d.Bt, d.H, d.D, d.D};
    const float* decay = x.decay(3, d.H);
    const float* kv_in = x.state(4, state);
    const bool want = x.flag(5);
    const int block = x.int32(6);
    const Out o(x, 7, q);
    Out kv;
    kv.state(x, 8, want, state, q);
    const size_t n = lib.workspace_bytes(d.Bt, d.H, d.N, d.D, block, dt, 0);
    const at::Tensor ws = scratch(n, q);
    call("ltn_attn_fwd", [&] {
        return lib.fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.ptr, decay, kv_in, (float*)kv.ptr, d.Bt, d.H, d.N, d.D,
                       block, dt, at_or_null(ws), n, x.stream());
    });
    if (!want && x.none(8)) return o.object();
    const Out* r[] = {&o, &kv};
    return tuple(r);
}

// q, k, v, u, decay, eps, kv_in, return_state, store_o, block, out, y_out, kv_out
PyObject* fwd_gated(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2), &u = x.tensor(3);
    const Dims d(q);
    same(q, k);
    same(q, v);
    same(q, u);
    const ltn_dtype dt = dtype_of(q);
    const std::array<int64_t, 4> state = {d.Bt, d.H, d.D, d.D};
    const float* decay = x.decay(4, d.H);
    const float eps = x.real(5);
    const float* kv_in = x.state(6, state);
    const bool want = x.flag(7), store_o = x.flag(8);
    const int block = x.int32(9);
    const Out o = store_o ? Out(x, 10, q) : Out();
    const Out y(x, 11, q);
    Out kv;
    kv.state(x, 12, want, state, q);
    const size_t n = lib.workspace_bytes(d.Bt, d.H, d.N, d.D, block, dt, 2);
    const at::Tensor ws = scratch(n, q);
    call("ltn_attn_fwd_gated", [&] {
        return lib.fwd_gated(q.data_ptr(), k.data_ptr(), v.data_ptr(), u.data_ptr(), o.ptr, y.ptr, decay, kv_in,
                             (float*)kv.ptr, eps, d.Bt, d.H, d.N, d.D, block, dt, at_or_null(ws), n, x.stream());
    });
    if (!want && x.none(12)) {
        const Out* r[] = {store_o ? &o : nullptr, &y};
        return tuple(r);
    }
    const Out* r[] = {store_o ? &o : nullptr, &y, &kv};
    return tuple(r);
}

// q, k, v, d_o, decay, block (the gradients are allocated here)
PyObject* bwd(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2), &g = x.tensor(3);
    const Dims d(q);
    same(q, k);
    same(q, v);
    same(q, g);
    const ltn_dtype dt = dtype_of(q);
    const float* decay = x.decay(4, d.H);
    const int block = x.int32(5);
    Out dq, dk, dv;
    for (Out* o : {&dq, &dk, &dv}) o->make(at::empty_like(q));
    const size_t n = lib.workspace_bytes(d.Bt, d.H, d.N, d.D, block, dt, 1);
    const at::Tensor ws = scratch(n, q);
    call("ltn_attn_bwd", [&] {
        return lib.bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), g.data_ptr(), dq.ptr, dk.ptr, dv.ptr, decay, d.Bt, d.H,
                       d.N, d.D, block, dt, at_or_null(ws), n, x.stream());
    });
    const Out* r[] = {&dq, &dk, &dv};
    return tuple(r);
}

// x, u, d_y, eps (the gradients are allocated here)
PyObject* gate_bwd(const Args& x) {
    const at::Tensor &t = x.tensor(0), &u = x.tensor(1), &g = x.tensor(2);
    need(t.dim() >= 1 && t.numel() > 0 && t.size(-1) <= INT32_MAX);
    same(t, u);
    same(t, g);
    const ltn_dtype dt = dtype_of(t);
    const float eps = x.real(3);
    const int D = (int)t.size(-1);
    Out dx, du;
    for (Out* o : {&dx, &du}) o->make(at::empty_like(t));
    call("ltn_gate_bwd", [&] {
        return lib.gate_bwd(t.data_ptr(), u.data_ptr(), g.data_ptr(), dx.ptr, du.ptr, eps, t.numel() / D, D, dt, x.stream());
    });
    const Out* r[] = {&dx, &du};
    return tuple(r);
}

// q, k, v, kv, decay, out: one token ([Bt,H,D]) or several ([Bt,H,S,D]) by `several`
PyObject* decode(const Args& x, bool several) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2), &kv = x.tensor(3);
    need(q.dim() == (several ? 4 : 3));
    same(q, k);
    same(q, v);
    const ltn_dtype dt = dtype_of(q);
    const int64_t Bt = q.size(0), H = q.size(1), S = several ? q.size(2) : 1, D = q.size(-1);
    for (int64_t n : {Bt, H, S, D}) need(n <= INT32_MAX);
    need(kv.scalar_type() == at::kFloat && kv.sizes() == at::IntArrayRef({Bt, H, D, D}));
    const float* decay = x.decay(4, H);
    const Out o(x, 5, q);
    call(several ? "ltn_attn_decode_steps" : "ltn_attn_decode_step", [&] {
        return lib.decode_steps(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.ptr, (float*)kv.data_ptr(), decay, (int)Bt, (int)H,
                                (int)S, (int)D, dt, x.stream());
    });
    return o.object();
}
PyObject* decode_step(const Args& x) { return decode(x, false); }
PyObject* decode_steps(const Args& x) { return decode(x, true); }

// Query/key width Dk, value width Dv.
struct Wide : Dims {
    int Dv;
    ltn_dtype dt;
    Wide(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v) : Dims(q) {
        same(q, k);
        need(v.dim() == 4 && v.scalar_type() == q.scalar_type() && v.sizes().slice(0, 3) == q.sizes().slice(0, 3) &&
             v.size(3) <= INT32_MAX);
        Dv = (int)v.size(3);
        dt = dtype_of(q);
    }
};

// q, k, v, decay, kv_in, return_state, block, out, kv_out
PyObject* fwd_dkdv(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2);
    const Wide d(q, k, v);
    const std::array<int64_t, 4> state = {d.Bt, d.H, d.D, d.Dv};
    const float* decay = x.decay(3, d.H);
    const float* kv_in = x.state(4, state);
    const bool want = x.flag(5);
    const int block = x.int32(6);
    const Out o(x, 7, v);
    Out kv;
    kv.state(x, 8, want, state, q);
    const size_t n = lib.workspace_bytes_dkdv(d.Bt, d.H, d.N, d.D, d.Dv, d.dt, 0);
    const at::Tensor ws = scratch(n, q);
    call("ltn_attn_fwd_dkdv", [&] {
        return lib.fwd_dkdv(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.ptr, decay, kv_in, (float*)kv.ptr, d.Bt, d.H, d.N,
                            d.D, d.Dv, block, d.dt, at_or_null(ws), n, x.stream());
    });
    if (!want && x.none(8)) return o.object();
    const Out* r[] = {&o, &kv};
    return tuple(r);
}

// q, k, v, d_o, decay, block
PyObject* bwd_dkdv(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2), &g = x.tensor(3);
    const Wide d(q, k, v);
    same(v, g);
    const float* decay = x.decay(4, d.H);
    const int block = x.int32(5);
    Out dq, dk, dv;
    dq.make(at::empty_like(q));
    dk.make(at::empty_like(k));
    dv.make(at::empty_like(v));
    const size_t n = lib.workspace_bytes_dkdv(d.Bt, d.H, d.N, d.D, d.Dv, d.dt, 1);
    const at::Tensor ws = scratch(n, q);
    call("ltn_attn_bwd_dkdv", [&] {
        return lib.bwd_dkdv(q.data_ptr(), k.data_ptr(), v.data_ptr(), g.data_ptr(), dq.ptr, dk.ptr, dv.ptr, decay, d.Bt, d.H,
                            d.N, d.D, d.Dv, block, d.dt, at_or_null(ws), n, x.stream());
    });
    const Out* r[] = {&dq, &dk, &dv};
    return tuple(r);
}

// q, k, v, kv, decay, out
PyObject* decode_steps_dkdv(const Args& x) {
    const at::Tensor &q = x.tensor(0), &k = x.tensor(1), &v = x.tensor(2), &kv = x.tensor(3);
    const Wide d(q, k, v);
    need(d.N <= INT32_MAX && kv.scalar_type() == at::kFloat && kv.sizes() == at::IntArrayRef({d.Bt, d.H, d.D, d.Dv}));
    const float* decay = x.decay(4, d.H);
    const Out o(x, 5, v);
    call("ltn_attn_decode_steps_dkdv", [&] {
        return lib.decode_steps_dkdv(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.ptr, (float*)kv.data_ptr(), decay, d.Bt, d.H,
                                     (int)d.N, d.D, d.Dv, d.dt, x.stream());
    });
    return o.object();
}

const float* theta_of(const Args& x, int i, const Dims& d) {
    if (x.none(i)) return nullptr;
    const at::Tensor& t = x.tensor(i);
    need(t.scalar_type() == at::kFloat && t.sizes() == at::IntArrayRef({d.H, d.D}));
    return (const float*)t.data_ptr();
}

// x, theta, act, pos0, out
PyObject* prologue_fwd(const Args& x) {
    const at::Tensor& t = x.tensor(0);
    const Dims d(t);
    const ltn_dtype dt = dtype_of(t);
    const float* theta = theta_of(x, 1, d);
    const bool act = x.flag(2);
    const long long pos0 = x.integer(3);
    const std::array<int64_t, 4> shape = {d.Bt, d.H, d.N, (theta ? 2 : 1) * (int64_t)d.D};
    Out y;
    if (x.none(4)) {
        y.make(at::empty(shape, t.options()));
    } else {
        y.take(x, 4, t.scalar_type(), 0);
        need(x.tensor(4).sizes() == at::IntArrayRef(shape));
    }
    call("ltn_prologue_fwd", [&] { return lib.prologue_fwd(t.data_ptr(), theta, y.ptr, act, d.Bt, d.H, d.N, d.D, pos0, dt, x.stream()); });
    return y.object();
}

// x, d_y, theta, act, pos0, want_dtheta
PyObject* prologue_bwd(const Args& x) {
    const at::Tensor &t = x.tensor(0), &g = x.tensor(1);
    const Dims d(t);
    const ltn_dtype dt = dtype_of(t);
    const float* theta = theta_of(x, 2, d);
    const bool act = x.flag(3);
    const long long pos0 = x.integer(4);
    const bool want = x.flag(5) && theta;
    need(g.scalar_type() == t.scalar_type() && g.sizes() == at::IntArrayRef({d.Bt, d.H, d.N, (theta ? 2 : 1) * (int64_t)d.D}));
    Out dx, dth;
    dx.make(at::empty_like(t));
    if (want) dth.make(at::empty({d.H, d.D}, t.options().dtype(at::kFloat)));
    const size_t n = want ? lib.prologue_workspace_bytes(d.Bt, d.H, d.N, d.D) : 0;
    const at::Tensor ws = scratch(n, t);
    call("ltn_prologue_bwd", [&] {
        return lib.prologue_bwd(t.data_ptr(), theta, g.data_ptr(), dx.ptr, (float*)dth.ptr, act, d.Bt, d.H, d.N, d.D, pos0,
                                dt, at_or_null(ws), n, x.stream());
    });
    const Out* r[] = {&dx, want ? &dth : nullptr};
    return tuple(r);
}

template <PyObject* (*F)(const Args&), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    try {
        return F(Args(args, n, N));
    } catch (const NotPlain&) {
        Py_RETURN_NONE;
    } catch (const Failed& f) {
        PyObject* e = PyObject_CallFunction(error_type, "is", (int)f.status, f.where);
        if (e) {
            PyErr_SetObject(error_type, e);
            Py_DECREF(e);
        }
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// The error class, then the addresses of the functions that `entry_points` names.
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    constexpr Py_ssize_t want = sizeof(Library) / sizeof(void*);
    if (n != 1 + want || !PyExceptionClass_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "an exception class and one address per entry point");
        return nullptr;
    }
    void* p[want];
    for (Py_ssize_t i = 0; i < want; ++i) {
        p[i] = PyLong_AsVoidPtr(args[1 + i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    static_assert(sizeof p == sizeof lib, "Library holds one function pointer per entry point");
    memcpy(&lib, p, sizeof lib);
    Py_INCREF(args[0]);
    Py_XSETREF(error_type, args[0]);
    Py_RETURN_NONE;
}

#define LTN_ENTRY(name, n) {#name, (PyCFunction)(void*)entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void*)bind, METH_FASTCALL, nullptr},
    LTN_ENTRY(fwd, 9), LTN_ENTRY(fwd_gated, 13), LTN_ENTRY(bwd, 6), LTN_ENTRY(gate_bwd, 4), LTN_ENTRY(decode_step, 6),
    LTN_ENTRY(decode_steps, 6), LTN_ENTRY(fwd_dkdv, 9), LTN_ENTRY(bwd_dkdv, 6), LTN_ENTRY(decode_steps_dkdv, 6),
    LTN_ENTRY(prologue_fwd, 5), LTN_ENTRY(prologue_bwd, 6), {nullptr, nullptr, 0, nullptr}};
#undef LTN_ENTRY
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ltn_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ltn_torch(void) {
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    PyObject* names = PyTuple_New(sizeof(Library) / sizeof(void*));
    bool ok = names != nullptr;
    Py_ssize_t i = 0;
#define LTN_NAME(field, symbol)                                \
    if (ok) {                                                  \
        PyObject* s = PyUnicode_FromString(#symbol);           \
        ok = s != nullptr;                                     \
        if (ok) PyTuple_SET_ITEM(names, i++, s);               \
    }
    LTN_LIBRARY(LTN_NAME)
#undef LTN_NAME
    // (LTN_BUILT_FOR: torch, the interpreter and the library's header, compared when the module is opened)
    ok = ok && PyModule_AddObjectRef(m, "entry_points", names) == 0 &&
         PyModule_AddStringConstant(m, "built_for", LTN_BUILT_FOR) == 0;
    Py_XDECREF(names);
    if (!ok) Py_CLEAR(m);
    return m;
}
