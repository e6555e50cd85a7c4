// The calling side of pb.py in native code: argument checks, device pointers, the current stream and the call into
// libpbatch.so.  The kernels of a batch-1 layer take 3 to 5 us and a launch 3 us of host time; the same steps through
// ctypes and Python took 8 to 11 us per call (two thirds of it in the per-argument checks and the stream lookup), so
// that a program that calls layer by layer waited for the host.  1024 x 1024, one vector: 11.4 -> 4.8 us per
// PackedLinear call.
//
// A function here takes the call if every argument is what it expects (positional, CUDA tensor of the right type,
// contiguous, ...).  Anything else, wrong or merely unusual, goes to the Python function of the same name in pb.py, which
// raises the errors: one place for their texts.  pb.py does without this extension where it is not built or was built for
// another torch or Python.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "pb.h"

namespace {

// what pb.py hands over once, when it has loaded the library
PyObject *g_desc_type = nullptr;    // the ctypes structure pb_desc
PyObject *g_error = nullptr;        // PbError(status, where)

enum Entry {
    kQuantizePack, kQuantizePackDesc, kQuantizePackMode, kUnpack, kMatmul, kMatmulStatic, kMatmulBiasAct, kMatmulAcc,
    kMatmulAccPairs, kActPrep, kMatmulPrepared, kFixedPoint, kLstmCell, kEntries
};
const char *const kNames[kEntries] = {
    "pb_quantize_pack", "pb_quantize_pack_desc", "pb_quantize_pack_mode", "pb_unpack", "pb_matmul", "pb_matmul_static",
    "pb_matmul_bias_act", "pb_matmul_acc", "pb_matmul_acc_pairs", "pb_act_prep", "pb_matmul_prepared", "pb_fixed_point",
    "pb_lstm_cell"};
void *g_fn[kEntries];               // null until bound: every call then goes to `slow`
PyObject *g_slow[kEntries];
PyObject *g_slow_linear = nullptr;

// ---- arguments: `load` says whether the object is what the fast path expects ----
template <typename T, at::ScalarType DT, bool NULLABLE = false>
struct Ptr {
    T *v = nullptr;
    bool load(PyObject *o)
    {
        if (NULLABLE && o == Py_None) return true;
        if (!THPVariable_CheckExact(o)) return false;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || t.scalar_type() != DT || !t.is_contiguous()) return false;
        v = static_cast<T *>(t.data_ptr());
        return true;
    }
    T *get() const { return v; }
};
using In = Ptr<const float, at::kFloat>;
using InOrNone = Ptr<const float, at::kFloat, true>;
using Out = Ptr<float, at::kFloat>;
using Bytes = Ptr<void, at::kByte>;
using Ints = Ptr<int32_t, at::kInt>;
using Longs = Ptr<int64_t, at::kLong>;

struct Int {
    int v = 0;
    bool load(PyObject *o)
    {
        if (!PyLong_CheckExact(o)) return false;
        const long x = PyLong_AsLong(o);
        if (x == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
        v = static_cast<int>(x);
        return v == x;
    }
    int get() const { return v; }
};

struct Address {
    void *v = nullptr;
    bool load(PyObject *o)
    {
        if (!PyLong_CheckExact(o)) return false;
        v = PyLong_AsVoidPtr(o);
        if (!v && PyErr_Occurred()) { PyErr_Clear(); return false; }
        return true;
    }
};

struct Desc {
    pb_desc v;
    bool load(PyObject *o)
    {
        if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != g_desc_type) return false;
        Py_buffer b;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
        const bool ok = b.len == (Py_ssize_t)sizeof(pb_desc);
        if (ok) v = *static_cast<const pb_desc *>(b.buf);
        PyBuffer_Release(&b);
        return ok;
    }
    const pb_desc *get() const { return &v; }
};

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

bool capturing() { return c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None; }

PyObject *status_result(int rc, const char *where)
{
    if (rc == PB_OK) Py_RETURN_NONE;
    PyObject *e = PyObject_CallFunction(g_error, "is", rc, where);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

template <typename... A, size_t... I>
bool load_all(std::tuple<A...> &a, PyObject *const *args, std::index_sequence<I...>)
{
    return (std::get<I>(a).load(args[I]) && ...);
}

// fn(args..., stream) of libpbatch.so
template <int E, typename... A>
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    constexpr Py_ssize_t N = sizeof...(A);
    const bool plain = !kwnames && (nargs == N || (nargs == N + 1 && args[N] == Py_None));
    if (plain && g_fn[E]) {
        try {
            std::tuple<A...> a;
            if (load_all(a, args, std::make_index_sequence<N>())) {
                void *stream = current_stream();
                int rc;
                Py_BEGIN_ALLOW_THREADS
                rc = std::apply(
                    [&](const A &...x) {
                        return reinterpret_cast<int (*)(decltype(std::declval<A>().get())..., void *)>(g_fn[E])(x.get()..., stream);
                    },
                    a);
                Py_END_ALLOW_THREADS
                return status_result(rc, kNames[E]);
            }
        } catch (const std::exception &) {   // (a tensor without memory of its own, say)
        }
    }
    return PyObject_Vectorcall(g_slow[E], args, nargs, kwnames);
}

PyObject *s_rows, *s_cols, *s_bits, *s_max_batch, *s_desc, *s_packed, *s_scales, *s_workspace, *s_home_stream;

// The attributes of `self` that a call uses, held until it returns: one that is computed on access, or replaced by another
// thread meanwhile, must not give its memory back before the launch.
struct Held {
    PyObject *o[9];
    int n = 0;
    int workspace = 0;   // which of them
    ~Held() { while (n) Py_DECREF(o[--n]); }
    template <typename T>
    bool load(PyObject *self, PyObject *name, T &x)
    {
        PyObject *a = PyObject_GetAttr(self, name);
        if (!a) { PyErr_Clear(); return false; }
        o[n++] = a;
        return x.load(a);
    }
};

// linear(self, X, bits_used, out): PackedLinear.__call__
PyObject *linear(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs == 4 && g_fn[kMatmul] && THPVariable_CheckExact(args[1])) {
        try {
            Int rows, cols, max_batch, m;
            Desc d;
            Bytes packed, workspace;
            In scales, x;
            Out y;
            Address home;
            Held held;   // (nine attributes at most)
            PyObject *self = args[0];
            const at::Tensor &X = THPVariable_Unpack(args[1]);
            bool ok = x.load(args[1]) && held.load(self, s_rows, rows) && held.load(self, s_cols, cols) &&
                      held.load(self, s_max_batch, max_batch) && held.load(self, s_desc, d) &&
                      held.load(self, s_packed, packed) && held.load(self, s_scales, scales) &&
                      held.load(self, s_workspace, workspace) && (held.workspace = held.n - 1, held.load(self, s_home_stream, home)) &&
                      (args[2] == Py_None ? held.load(self, s_bits, m) : m.load(args[2]) && m.v != 0);
            const int64_t n = X.numel();
            ok = ok && cols.v > 0 && n > 0 && n % cols.v == 0 && n / cols.v <= max_batch.v;
            if (ok) {
                const int batch = static_cast<int>(n / cols.v);
                at::Tensor out;
                if (args[3] == Py_None) {
                    out = at::empty({batch, rows.v}, X.options().requires_grad(false));
                    y.v = static_cast<float *>(out.data_ptr());
                } else {
                    ok = y.load(args[3]);
                }
                if (ok) {
                    void *stream = current_stream();
                    const auto matmul = reinterpret_cast<decltype(&pb_matmul)>(g_fn[kMatmul]);
                    int rc;
                    // A batch goes through the workspace.  The holder's own serves the stream it was made on (the library keeps the
                    // launches of two threads apart); on another stream the call has one of its own, and under capture: a graph
                    // may be replayed on any stream (the memory is then the graph's, as that of the output).
                    at::Tensor own;
                    if ((batch > 1 || d.v.layout == PB_LAYOUT_ROWMAJOR_V1 || d.v.layout == PB_LAYOUT_TILE16_PAIRS_V1) &&
                        (stream != home.v || capturing()))
                        own = at::empty_like(THPVariable_Unpack(held.o[held.workspace]));
                    void *const work = own.defined() ? own.data_ptr() : workspace.v;
                    Py_BEGIN_ALLOW_THREADS
                    rc = matmul(packed.v, scales.v, &d.v, m.v, x.v, batch, y.v, work, stream);
                    Py_END_ALLOW_THREADS
                    if (rc != PB_OK) return status_result(rc, kNames[kMatmul]);
                    if (args[3] != Py_None) {
                        Py_INCREF(args[3]);
                        return args[3];
                    }
                    return THPVariable_Wrap(std::move(out));
                }
            }
        } catch (const std::exception &) {
        }
    }
    return PyObject_Vectorcall(g_slow_linear, args, nargs, nullptr);
}

// bind(desc_type, error_type, {name: address})
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *desc, *error, *fns;
    if (!PyArg_ParseTuple(args, "OOO!", &desc, &error, &PyDict_Type, &fns)) return nullptr;
    void *p[kEntries];
    for (int e = 0; e < kEntries; ++e) {
        PyObject *a = PyDict_GetItemString(fns, kNames[e]);
        if (!a) return PyErr_Format(PyExc_KeyError, "%s", kNames[e]);
        p[e] = PyLong_AsVoidPtr(a);
        if (!p[e]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "%s", kNames[e]);
    }
    Py_INCREF(desc);
    Py_INCREF(error);
    Py_XDECREF(g_desc_type);
    Py_XDECREF(g_error);
    g_desc_type = desc;
    g_error = error;
    for (int e = 0; e < kEntries; ++e) g_fn[e] = p[e];
    Py_RETURN_NONE;
}

// set_slow({name: function}): the Python functions behind the fast ones ("linear" for PackedLinear.__call__)
PyObject *set_slow(PyObject *, PyObject *fns)
{
    if (!PyDict_Check(fns)) return PyErr_Format(PyExc_TypeError, "a dict of functions");
    for (int e = 0; e <= kEntries; ++e) {
        PyObject *f = PyDict_GetItemString(fns, e < kEntries ? kNames[e] : "linear");
        if (!f) return PyErr_Format(PyExc_KeyError, "%s", e < kEntries ? kNames[e] : "linear");
        PyObject **slot = e < kEntries ? &g_slow[e] : &g_slow_linear;
        Py_INCREF(f);
        Py_XDECREF(*slot);
        *slot = f;
    }
    Py_RETURN_NONE;
}

// as many arguments as the C function has, each convertible to the parameter in its place, and the stream as the last
template <typename F>
struct Params;
template <typename... P>
struct Params<int (*)(P...)> {
    template <typename... A>
    static constexpr bool take()
    {
        if constexpr (sizeof...(P) == sizeof...(A) + 1)
            return std::is_invocable_v<int (*)(P...), decltype(std::declval<const A &>().get())..., void *>;
        else
            return false;
    }
};
template <auto F, int E, typename... A>
PyMethodDef fast()
{
    static_assert(Params<decltype(F)>::template take<A...>(), "not the arguments of the C function");
    return {kNames[E], reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&call<E, A...>)), METH_FASTCALL | METH_KEYWORDS,
            nullptr};
}
PyMethodDef kMethods[] = {
    fast<&pb_quantize_pack, kQuantizePack, In, Int, Int, Int, Bytes, Out>(),
    fast<&pb_quantize_pack_desc, kQuantizePackDesc, In, Desc, Bytes, Out>(),
    fast<&pb_quantize_pack_mode, kQuantizePackMode, In, Desc, Int, Bytes, Out>(),
    fast<&pb_unpack, kUnpack, Bytes, Desc, Ints>(),
    fast<&pb_matmul, kMatmul, Bytes, In, Desc, Int, In, Int, Out, Bytes>(),
    fast<&pb_matmul_static, kMatmulStatic, Bytes, In, Desc, Int, In, Int, Out>(),
    fast<&pb_matmul_bias_act, kMatmulBiasAct, Bytes, In, Desc, Int, In, Int, InOrNone, Int, Out, Bytes>(),
    fast<&pb_matmul_acc, kMatmulAcc, Bytes, Desc, Int, In, Int, Longs, Bytes>(),
    fast<&pb_matmul_acc_pairs, kMatmulAccPairs, Bytes, Desc, Int, In, Int, Longs, Bytes>(),
    fast<&pb_act_prep, kActPrep, Desc, In, Int, Bytes>(),
    fast<&pb_matmul_prepared, kMatmulPrepared, Bytes, In, Desc, Int, Int, Out, Bytes>(),
    fast<&pb_fixed_point, kFixedPoint, Desc, In, Int, Ints, Bytes>(),
    fast<&pb_lstm_cell, kLstmCell, Bytes, In, Desc, Int, In, Int, In, In, InOrNone, Out, Out, Int, Bytes>(),
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&linear)), METH_FASTCALL, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {"set_slow", set_slow, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    s_rows = PyUnicode_InternFromString("rows");
    s_cols = PyUnicode_InternFromString("cols");
    s_bits = PyUnicode_InternFromString("bits");
    s_max_batch = PyUnicode_InternFromString("max_batch");
    s_desc = PyUnicode_InternFromString("desc");
    s_packed = PyUnicode_InternFromString("packed");
    s_scales = PyUnicode_InternFromString("scales");
    s_workspace = PyUnicode_InternFromString("workspace");
    s_home_stream = PyUnicode_InternFromString("home_stream");
    PyObject *m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", PB_BUILT_FOR) != 0) Py_CLEAR(m);   // (pb.py compares it)
    return m;
}
