// The short way of the Python binding's per-call functions: checks, output allocation and the call in native code.
//
// What bounds a small call is the host: for 4096 x 4096 at one token the kernel takes 3.6 us, and with the checks and ctypes in
// Python a call took 6.6 to 7.  Each function here takes the arguments of the Python function of its name and serves the case that needs
// no explaining: plain tensors of the expected type, shape and device.  Anything else (another shape, a subclass, a tensor on
// another device, an exception out of torch) returns None without having launched anything, and the Python function, which states
// the checks, goes its own way: it decides what is accepted and what an error says.  bound() is what bound_call returns: the entry
// point with its arguments in its own types (eight launches of a small layer at four tokens took 33 us through ctypes, whose
// conversions are most of a launch there).
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <exception>
#include <memory>
#include <new>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/w4a8.h"

namespace {

// Entry points of the C ABI, whose addresses the Python module hands over: the library that it loaded is the one called.
struct Entries {
    decltype(&::w4a8_quantize_act) quantize_act;
    decltype(&::w4a8_quantize_act_strided) quantize_act_strided;
    decltype(&::w4a8_gemm) gemm;
    decltype(&::w4a8_gemm_tiled) gemm_tiled;
    decltype(&::w4a8_gemm_tiled_splitk) gemm_tiled_splitk;
    decltype(&::w8a8_gemm_tiled) w8a8_gemm_tiled;
    decltype(&::w4a8_linear_tiled_fp16) linear_tiled_fp16;
    decltype(&::w4a8_tiled_weight_bytes) w4a8_tiled_weight_bytes;
    decltype(&::w8a8_tiled_weight_bytes) w8a8_tiled_weight_bytes;
    decltype(&::w4a8_quantize_weights) quantize_weights;
    decltype(&::w4a8_tile_weights) tile_weights;
} entries;
PyObject *check = nullptr;  // check(code): raises for what an entry point returned

struct NotServed {};  // for the Python function to look at

const at::Tensor &plain(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw NotServed{};
    return THPVariable_Unpack(o);
}

// What a call's tensors have to be on, and the stream that torch has current there.  The device is asked for only once a call has
// shown a tensor on one.
struct Here {
    const c10::DeviceIndex device;
    explicit Here(PyObject *first) : device(plain(first).is_cuda() ? c10::hip::current_device() : throw NotServed{}) {}
    void *stream() const { return (void *)c10::hip::getCurrentHIPStream(device).stream(); }
};

int as_int(int64_t v) {
    if (v < 0 || v > INT_MAX) throw NotServed{};
    return (int)v;
}

const at::Tensor &view(PyObject *o, const Here &here, at::ScalarType type, int64_t dims) {
    const at::Tensor &t = plain(o);
    if (!t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type || t.dim() != dims || t.get_device() != here.device) throw NotServed{};
    return t;
}

const at::Tensor &dense(PyObject *o, const Here &here, at::ScalarType type, int64_t dims) {
    const at::Tensor &t = view(o, here, type, dims);
    if (!t.is_contiguous()) throw NotServed{};
    return t;
}

// the caller's output, or a new one
at::Tensor output(PyObject *o, const Here &here, at::ScalarType type, at::IntArrayRef shape, const at::Tensor &like) {
    if (o == Py_None) return at::empty(shape, like.options().dtype(type).requires_grad(false));
    const at::Tensor &t = dense(o, here, type, (int64_t)shape.size());
    if (t.sizes() != shape) throw NotServed{};
    return t;
}

// A reference given up with its scope unless it is handed on
struct Owned {
    PyObject *object;
    explicit Owned(PyObject *o) : object(o) {
        if (!o) throw NotServed{};
    }
    Owned(const Owned &) = delete;
    ~Owned() { Py_XDECREF(object); }
    PyObject *release() { return std::exchange(object, nullptr); }
};

// What a call returns, made before its launch: nothing behind a launch may fail, or the Python function would launch once more
PyObject *returned(PyObject *given, const at::Tensor &t) { return given == Py_None ? THPVariable_Wrap(t) : Py_NewRef(given); }
PyObject *returned(PyObject *given0, const at::Tensor &t0, PyObject *given1, const at::Tensor &t1) {
    const Owned r0(returned(given0, t0)), r1(returned(given1, t1));
    return PyTuple_Pack(2, r0.object, r1.object);
}

// The call itself, with the interpreter's lock given back as ctypes would (a launch waits where the queue is full).  False: the
// Python error is set.
template <class Call>
bool launched(Call call) {
    int code;
    {
        PyThreadState *const state = PyEval_SaveThread();
        code = call();
        PyEval_RestoreThread(state);
    }
    if (code == 0) return true;
    PyObject *r = PyObject_CallFunction(check, "i", code);
    if (r) {  // check raises for every code but 0
        Py_DECREF(r);
        PyErr_SetString(PyExc_RuntimeError, "w4a8: an error code was not raised");
    }
    return false;
}

template <class Body>
PyObject *serve(Py_ssize_t nargs, Py_ssize_t want, Body body) {
    // a mode that wants to see the allocations sees those of the Python function
    if (nargs != want || !check || at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled()) Py_RETURN_NONE;
    try {
        return body();
    } catch (const NotServed &) {
    } catch (const std::exception &) {  // of torch's, which the Python function will meet again and pass on
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

template <class T>
T *ptr(const at::Tensor &t) {
    return (T *)t.data_ptr();
}

// (x, xq, s_a)
template <bool STRIDED>
PyObject *quantize_act(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 3, [&]() -> PyObject * {
        const Here here(a[0]);
        const at::Tensor &x = STRIDED ? view(a[0], here, at::kHalf, 2) : dense(a[0], here, at::kHalf, 2);
        if (STRIDED && x.stride(1) != 1) throw NotServed{};
        const int M = as_int(x.size(0)), K = as_int(x.size(1));
        const at::Tensor xq = output(a[1], here, at::kChar, {M, K}, x), s_a = output(a[2], here, at::kFloat, {M}, x);
        const void *const px = ptr<void>(x);
        int8_t *const pq = ptr<int8_t>(xq);
        float *const ps = ptr<float>(s_a);
        const long long ldx = x.stride(0);
        void *const stream = here.stream();
        Owned both(returned(a[1], xq, a[2], s_a));
        if (!launched([=] { return STRIDED ? entries.quantize_act_strided(px, ldx, pq, ps, M, K, stream) : entries.quantize_act(px, pq, ps, M, K, stream); }))
            return nullptr;
        return both.release();
    });
}

// what the GEMMs have in common: codes, their scales, the channels' scales, the output
struct Operands {
    const Here here;
    const at::Tensor &xq, &s_a, &s_w;
    const int M, K, N;
    Operands(PyObject *q, PyObject *sa, PyObject *sw)
        : here(q), xq(dense(q, here, at::kChar, 2)), s_a(dense(sa, here, at::kFloat, 1)), s_w(dense(sw, here, at::kFloat, 1)), M(as_int(xq.size(0))),
          K(as_int(xq.size(1))), N(as_int(s_w.size(0))) {
        if (s_a.size(0) != M) throw NotServed{};
    }
    const uint8_t *tiled(PyObject *w, size_t (*bytes)(int, int)) const {
        const at::Tensor &wt = dense(w, here, at::kByte, 1);
        if ((size_t)wt.numel() != bytes(N, K) || wt.numel() == 0) throw NotServed{};
        return ptr<uint8_t>(wt);
    }
};

template <class Call>
PyObject *gemm_with(const Operands &o, PyObject *out_given, Call call) {
    const at::Tensor out = output(out_given, o.here, at::kHalf, {o.M, o.N}, o.xq);
    const int8_t *const xq = ptr<int8_t>(o.xq);
    const float *const s_a = ptr<float>(o.s_a), *const s_w = ptr<float>(o.s_w);
    void *const po = ptr<void>(out), *const stream = o.here.stream();
    Owned result(returned(out_given, out));
    if (!launched([&] { return call(xq, s_a, s_w, po, stream); })) return nullptr;
    return result.release();
}

// (xq, s_a, wp, s_w, out); the entry point makes no use of a workspace
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 5, [&] {
        const Operands o(a[0], a[1], a[3]);
        const at::Tensor &w = dense(a[2], o.here, at::kByte, 2);
        if (w.size(0) != o.N || w.size(1) * 2 != o.K) throw NotServed{};
        const uint8_t *const wp = ptr<uint8_t>(w);
        return gemm_with(o, a[4], [&](auto xq, auto s_a, auto s_w, void *out, void *st) { return entries.gemm(xq, s_a, wp, s_w, out, o.M, o.N, o.K, nullptr, 0, st); });
    });
}

// (xq, s_a, wt, s_w, out)
PyObject *gemm_tiled(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 5, [&] {
        const Operands o(a[0], a[1], a[3]);
        const uint8_t *const wt = o.tiled(a[2], entries.w4a8_tiled_weight_bytes);
        return gemm_with(o, a[4], [&](auto xq, auto s_a, auto s_w, void *out, void *st) { return entries.gemm_tiled(xq, s_a, wt, s_w, out, o.M, o.N, o.K, st); });
    });
}

// (xq, s_a, wt, s_w, ws, out): the library's choice of slices, in the caller's workspace
PyObject *gemm_tiled_splitk(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 6, [&] {
        const Operands o(a[0], a[1], a[3]);
        const uint8_t *const wt = o.tiled(a[2], entries.w4a8_tiled_weight_bytes);
        const at::Tensor &ws = plain(a[4]);
        if (!ws.is_cuda() || ws.layout() != at::kStrided || ws.scalar_type() != at::kByte || !ws.is_contiguous() || ws.get_device() != o.here.device)
            throw NotServed{};
        void *const pw = ptr<void>(ws);
        const size_t bytes = (size_t)ws.numel();
        return gemm_with(o, a[5], [&](auto xq, auto s_a, auto s_w, void *out, void *st) {
            return entries.gemm_tiled_splitk(xq, s_a, wt, s_w, out, o.M, o.N, o.K, 0, 0, pw, bytes, st);
        });
    });
}

// (xq, s_a, wt, s_w, out): fp16 output, the library's choice of tile
PyObject *w8a8_gemm_tiled(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 5, [&] {
        const Operands o(a[0], a[1], a[3]);
        const uint8_t *const wt = o.tiled(a[2], entries.w8a8_tiled_weight_bytes);
        return gemm_with(o, a[4], [&](auto xq, auto s_a, auto s_w, void *out, void *st) {
            return entries.w8a8_gemm_tiled(xq, s_a, wt, s_w, out, nullptr, o.M, o.N, o.K, 0, st);
        });
    });
}

// (x, wt, s_w, out, s_a_out)
PyObject *linear_tiled_fp16(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 5, [&]() -> PyObject * {
        const Here here(a[0]);
        const at::Tensor &x = view(a[0], here, at::kHalf, 2), &wt = dense(a[1], here, at::kByte, 1), &s_w = dense(a[2], here, at::kFloat, 1);
        const int M = as_int(x.size(0)), K = as_int(x.size(1)), N = as_int(s_w.size(0));
        if (x.stride(1) != 1 || wt.numel() == 0 || (size_t)wt.numel() != entries.w4a8_tiled_weight_bytes(N, K)) throw NotServed{};
        float *scales = nullptr;
        if (a[4] != Py_None) {
            const at::Tensor &s = dense(a[4], here, at::kFloat, 1);
            if (s.size(0) != M) throw NotServed{};
            scales = ptr<float>(s);
        }
        const at::Tensor out = output(a[3], here, at::kHalf, {M, N}, x);
        const void *const px = ptr<void>(x);
        const uint8_t *const pw = ptr<uint8_t>(wt);
        const float *const ps = ptr<float>(s_w);
        void *const po = ptr<void>(out), *const stream = here.stream();
        const long long ldx = x.stride(0);
        Owned result(returned(a[3], out));
        if (!launched([=] { return entries.linear_tiled_fp16(px, ldx, pw, ps, po, scales, M, N, K, stream); })) return nullptr;
        return result.release();
    });
}

// (w, wp, s_w)
PyObject *quantize_weights(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 3, [&]() -> PyObject * {
        const Here here(a[0]);
        const at::Tensor &w = dense(a[0], here, at::kHalf, 2);
        const int N = as_int(w.size(0)), K = as_int(w.size(1));
        const at::Tensor wp = output(a[1], here, at::kByte, {N, K / 2}, w), s_w = output(a[2], here, at::kFloat, {N}, w);
        const void *const pw = ptr<void>(w);
        uint8_t *const pp = ptr<uint8_t>(wp);
        float *const ps = ptr<float>(s_w);
        void *const stream = here.stream();
        Owned both(returned(a[1], wp, a[2], s_w));
        if (!launched([=] { return entries.quantize_weights(pw, pp, ps, N, K, stream); })) return nullptr;
        return both.release();
    });
}

// (wp, wt)
PyObject *tile_weights(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return serve(n, 2, [&]() -> PyObject * {
        const Here here(a[0]);
        const at::Tensor &wp = dense(a[0], here, at::kByte, 2);
        const int N = as_int(wp.size(0)), K = as_int(wp.size(1) * 2);
        const size_t bytes = entries.w4a8_tiled_weight_bytes(N, K);
        if (bytes == 0) throw NotServed{};
        const at::Tensor wt = output(a[1], here, at::kByte, {(int64_t)bytes}, wp);
        const uint8_t *const pp = ptr<uint8_t>(wp);
        uint8_t *const pt = ptr<uint8_t>(wt);
        void *const stream = here.stream();
        Owned result(returned(a[1], wt));
        if (!launched([=] { return entries.tile_weights(pp, pt, N, K, stream); })) return nullptr;
        return result.release();
    });
}

// ---- calls whose arguments are marshalled once

// One entry point with its arguments, all but the stream, which comes last.
struct Marshalled {
    virtual int operator()(void *stream) const = 0;
    virtual ~Marshalled() = default;
};

// What ctypes would take for a parameter of this type; false: leave it to ctypes
bool parse(PyObject *o, float *v) {
    if (!PyFloat_Check(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
template <class T>
std::enable_if_t<std::is_pointer_v<T>, bool> parse(PyObject *o, T *v) {
    if (o == Py_None) return *v = nullptr, true;
    if (!PyLong_Check(o)) return false;
    *v = (T)PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}
template <class T>
std::enable_if_t<std::is_integral_v<T>, bool> parse(PyObject *o, T *v) {
    if (!PyLong_Check(o)) return false;
    const long long x = PyLong_AsLongLong(o);
    *v = (T)x;
    return !PyErr_Occurred() && (long long)*v == x && (std::is_signed_v<T> || x >= 0);
}

template <class... A>
struct MarshalledCall final : Marshalled {
    using Args = std::tuple<A...>;
    static constexpr size_t kStream = sizeof...(A) - 1;
    int (*fn)(A...);
    Args args{};
    explicit MarshalledCall(int (*f)(A...)) : fn(f) {}
    int operator()(void *stream) const override {
        Args with = args;
        std::get<kStream>(with) = stream;
        return std::apply(fn, with);
    }
    template <size_t... I>
    bool take(PyObject *values, std::index_sequence<I...>) {
        return (parse(PyTuple_GET_ITEM(values, I), &std::get<I>(args)) && ...);
    }
};

template <class... A>
std::unique_ptr<Marshalled> marshal(int (*)(A...), void *address, PyObject *values) {
    static_assert(std::is_same_v<std::tuple_element_t<sizeof...(A) - 1, std::tuple<A...>>, void *>, "the stream comes last");
    if (PyTuple_GET_SIZE(values) != sizeof...(A) - 1) return nullptr;
    int (*fn)(A...);
    std::memcpy(&fn, &address, sizeof fn);
    auto call = std::make_unique<MarshalledCall<A...>>(fn);
    if (!call->take(values, std::make_index_sequence<sizeof...(A) - 1>{})) return nullptr;
    return call;
}

std::unique_ptr<Marshalled> marshal_by_name(const char *name, void *address, PyObject *values) {
#define W4A8_ENTRY(entry) \
    if (std::strcmp(name, #entry) == 0) return marshal((decltype(&::entry))nullptr, address, values);  /* its type only */
    W4A8_ENTRY(w4a8_quantize_act) W4A8_ENTRY(w4a8_quantize_act_strided) W4A8_ENTRY(w4a8_gemm) W4A8_ENTRY(w4a8_gemm_acc_i32)
    W4A8_ENTRY(w4a8_tile_weights) W4A8_ENTRY(w4a8_gemm_tiled) W4A8_ENTRY(w4a8_quantize_weights) W4A8_ENTRY(w4a8_quantize_weights_clipped)
    W4A8_ENTRY(w4a8_gemm_tiled_swiglu) W4A8_ENTRY(w4a8_gemm_tiled_splitk) W4A8_ENTRY(w4a8_gemm_tiled_splitk_static)
    W4A8_ENTRY(w4a8_linear_tiled_fp16) W4A8_ENTRY(w4a8_linear_tiled_swiglu_fp16) W4A8_ENTRY(w4a8_linear_tiled_norm_fp16)
    W4A8_ENTRY(w8a8_tile_weights) W4A8_ENTRY(w8a8_gemm_tiled) W4A8_ENTRY(w4a8_gemm_tiled_unsigned) W4A8_ENTRY(w4a8_gemm_fine_grained)
    W4A8_ENTRY(w4a8_silu_mul) W4A8_ENTRY(w4a8_silu_mul_quantize) W4A8_ENTRY(w4a8_add_rmsnorm_quantize)
#undef W4A8_ENTRY
    return nullptr;
}

struct BoundCall {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    Marshalled *call;
    PyObject *keep;  // the tensors behind the pointers
    PyObject *dict;  // attributes, __name__ and the like among them, and weak references, as a Python function has them
    PyObject *weak;
    c10::DeviceIndex device;
};

PyObject *bound_run(PyObject *self, PyObject *const *, size_t nargsf, PyObject *kwnames) {
    const BoundCall *const b = (BoundCall *)self;
    if (PyVectorcall_NARGS(nargsf) != 0 || (kwnames && PyTuple_GET_SIZE(kwnames) != 0)) {
        PyErr_SetString(PyExc_TypeError, "a bound call takes no arguments");
        return nullptr;
    }
    void *stream;
    try {
        stream = (void *)c10::hip::getCurrentHIPStream(b->device).stream();
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    if (!launched([&] { return (*b->call)(stream); })) return nullptr;
    Py_RETURN_NONE;
}

int bound_traverse(PyObject *self, visitproc visit, void *arg) {
    Py_VISIT(((BoundCall *)self)->keep);
    Py_VISIT(((BoundCall *)self)->dict);
    return 0;
}

int bound_clear(PyObject *self) {
    Py_CLEAR(((BoundCall *)self)->keep);
    Py_CLEAR(((BoundCall *)self)->dict);
    return 0;
}

void bound_dealloc(PyObject *self) {
    PyObject_GC_UnTrack(self);
    if (((BoundCall *)self)->weak) PyObject_ClearWeakRefs(self);
    bound_clear(self);
    delete ((BoundCall *)self)->call;
    PyObject_GC_Del(self);
}

// copy.copy, copy.deepcopy: itself, as of a function
PyObject *bound_copied(PyObject *self, PyObject *) { return Py_NewRef(self); }
PyMethodDef bound_methods[] = {{"__copy__", bound_copied, METH_NOARGS, nullptr}, {"__deepcopy__", bound_copied, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyGetSetDef bound_attributes[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};

PyTypeObject bound_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bound(name, address, values, device ordinal, tensors) -> a function of no arguments, or None where ctypes has to be asked
PyObject *bound(PyObject *, PyObject *args) {
    const char *name;
    PyObject *address, *values, *keep;
    int device;
    if (!PyArg_ParseTuple(args, "sO!O!iO", &name, &PyLong_Type, &address, &PyTuple_Type, &values, &device, &keep)) return nullptr;
    void *const entry = PyLong_AsVoidPtr(address);
    if (!entry || !check) return PyErr_Occurred() ? nullptr : Py_NewRef(Py_None);
    std::unique_ptr<Marshalled> call;
    try {
        call = marshal_by_name(name, entry, values);
    } catch (const std::bad_alloc &) {
        return PyErr_NoMemory();
    }
    if (!call) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    PyObject *const dict = Py_BuildValue("{ssssss}", "__name__", "call", "__qualname__", "bound_call.<locals>.call", "__module__", "paper_2311_09550_amd");
    BoundCall *const b = dict ? PyObject_GC_New(BoundCall, &bound_type) : nullptr;
    if (!b) {
        Py_XDECREF(dict);
        return nullptr;
    }
    b->dict = dict;
    b->weak = nullptr;
    b->vectorcall = bound_run;
    b->call = call.release();
    b->keep = Py_NewRef(keep);
    b->device = (c10::DeviceIndex)device;
    PyObject_GC_Track((PyObject *)b);
    return (PyObject *)b;
}

// bind(check, {name: address})
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *raises, *table;
    if (!PyArg_ParseTuple(args, "OO!", &raises, &PyDict_Type, &table)) return nullptr;
    Entries e;
    const struct {
        const char *name;
        void *slot;
    } wanted[] = {{"w4a8_quantize_act", &e.quantize_act},
                  {"w4a8_quantize_act_strided", &e.quantize_act_strided},
                  {"w4a8_gemm", &e.gemm},
                  {"w4a8_gemm_tiled", &e.gemm_tiled},
                  {"w4a8_gemm_tiled_splitk", &e.gemm_tiled_splitk},
                  {"w8a8_gemm_tiled", &e.w8a8_gemm_tiled},
                  {"w4a8_linear_tiled_fp16", &e.linear_tiled_fp16},
                  {"w4a8_tiled_weight_bytes", &e.w4a8_tiled_weight_bytes},
                  {"w8a8_tiled_weight_bytes", &e.w8a8_tiled_weight_bytes},
                  {"w4a8_quantize_weights", &e.quantize_weights},
                  {"w4a8_tile_weights", &e.tile_weights}};
    for (const auto &w : wanted) {
        PyObject *const address = PyDict_GetItemString(table, w.name);
        void *const p = address ? PyLong_AsVoidPtr(address) : nullptr;
        if (!p) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address for %s", w.name);
            return nullptr;
        }
        std::memcpy(w.slot, &p, sizeof p);
    }
    entries = e;
    Py_INCREF(raises);
    Py_XDECREF(check);
    check = raises;
    Py_RETURN_NONE;
}

#define W4A8_FAST(name, function) {name, (PyCFunction)(void (*)(void))function, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"bound", bound, METH_VARARGS, nullptr},
                         W4A8_FAST("quantize_act", quantize_act<false>),
                         W4A8_FAST("quantize_act_strided", quantize_act<true>),
                         W4A8_FAST("gemm", gemm),
                         W4A8_FAST("gemm_tiled", gemm_tiled),
                         W4A8_FAST("gemm_tiled_splitk", gemm_tiled_splitk),
                         W4A8_FAST("w8a8_gemm_tiled", w8a8_gemm_tiled),
                         W4A8_FAST("linear_tiled_fp16", linear_tiled_fp16),
                         W4A8_FAST("quantize_weights", quantize_weights),
                         W4A8_FAST("tile_weights", tile_weights),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Native short way of the binding's per-call functions.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    bound_type.tp_name = "paper_2311_09550_amd._binding.BoundCall";
    bound_type.tp_basicsize = sizeof(BoundCall);
    bound_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
    bound_type.tp_vectorcall_offset = offsetof(BoundCall, vectorcall);
    bound_type.tp_call = PyVectorcall_Call;
    bound_type.tp_dictoffset = offsetof(BoundCall, dict);
    bound_type.tp_weaklistoffset = offsetof(BoundCall, weak);
    bound_type.tp_methods = bound_methods;
    bound_type.tp_getset = bound_attributes;
    bound_type.tp_getattro = PyObject_GenericGetAttr;
    bound_type.tp_setattro = PyObject_GenericSetAttr;
    bound_type.tp_traverse = bound_traverse;
    bound_type.tp_clear = bound_clear;
    bound_type.tp_dealloc = bound_dealloc;
    if (PyType_Ready(&bound_type) < 0) return nullptr;
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", W4A8_BUILT_FOR_TORCH) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
