// The Python binding's short way from torch tensors to the C ABI: a CPython
// module that checks the tensors of one call, collects their pointers and
// calls the library, for calls in the ordinary form -- plain device tensors
// on the current GPU, the current stream, builtin numbers.  Anything else
// (pinned host memory, another stream or device, a tensor the checks refuse)
// is left to the Python code of the package, which takes every form and
// raises the errors: call() then returns -1 and has done nothing.
//
// Why native: for W = 8 the call took 13.4 us, 7.7 of them the same checks in
// Python, against 2.4 us for a small kernel; it takes 4.0 us this way.
#include <torch/csrc/autograd/python_variable.h>

#include <Python.h>

#include <cstdint>
#include <limits>

#include "disdp.h"
#include "disdp_launch.h"

namespace {

// The library's entry points, as the package loaded them, and torch's queries
// of the current device and of a device's current stream.
decltype(&disdp_aggregate) lib_aggregate;
decltype(&disdp_adam_step) lib_adam_step;
decltype(&disdp_aggregate_adam) lib_aggregate_adam;
decltype(&disdp_aggregate_adam_dev) lib_aggregate_adam_dev;
decltype(&disdp_quantize) lib_quantize;
PyObject *current_device, *current_stream;

enum Op { kOpAggregate, kOpAdamStep, kOpFused, kOpFusedDev, kOpQuantize };

enum Kind { kF32, kHalf, kI32, kOther };  // kHalf: bf16, or its bits in 16-bit integers
Kind kind_of(const at::Tensor &t)
{
    switch (t.scalar_type()) {
    case at::kFloat: return kF32;
    case at::kBFloat16:
    case at::kShort:
    case at::kUInt16: return kHalf;
    case at::kInt: return kI32;
    default: return kOther;
    }
}

struct Held {
    PyObject *ref = nullptr;
    ~Held() { Py_XDECREF(ref); }
};

// What the tensors of one call have in common.
struct Common {
    int64_t n = -1;
    int device = -1;
};

// Dispatch keys of tensors that stand for others (tracing, vmap, function
// transforms).
const c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::Functionalize,
                                    c10::DispatchKey::FuncTorchBatched,
                                    c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::BatchedNestedTensor,
                                    c10::DispatchKey::ZeroTensor});

// The address of a tensor of `n` elements and the wanted kind, or false when
// it is not such a tensor in the ordinary form: exactly a Tensor or Parameter,
// with storage of its own.
bool address(PyObject *obj, Kind want, int64_t n, Common &c, void *&p)
{
    if (!THPVariable_CheckExact(obj))
        return false;
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided ||
        t.key_set().has_any(kWrapped) || kind_of(t) != want || t.numel() != n ||
        !t.is_contiguous())
        return false;
    const int device = t.get_device();
    if (c.device >= 0 && device != c.device)
        return false;
    c.device = device;
    p = t.data_ptr();
    return true;
}

bool optional_address(PyObject *obj, Kind want, int64_t n, Common &c, void *&p)
{
    p = nullptr;
    return obj == Py_None || address(obj, want, n, c, p);
}

bool number(PyObject *obj, float &x)
{
    const double d = PyFloat_AsDouble(obj);
    if (d == -1.0 && PyErr_Occurred())
        return false;
    x = static_cast<float>(d);
    return true;
}

bool integer(PyObject *obj, int64_t lo, int64_t hi, int64_t &x)
{
    if (!PyLong_CheckExact(obj))
        return false;
    x = PyLong_AsLongLong(obj);
    if (x == -1 && PyErr_Occurred())
        return false;
    return x >= lo && x <= hi;
}

// An integer from a torch query that takes `arg` (or nothing).
bool asked(PyObject *fn, PyObject *arg, unsigned long long &x)
{
    PyObject *r = arg ? PyObject_CallFunctionObjArgs(fn, arg, nullptr)
                      : PyObject_CallFunctionObjArgs(fn, nullptr);
    if (!r)
        return false;
    x = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// call(op, grads, param, m, v, param_bf16, agg_f32, agg_i32, scalars, mode,
// frac_bits, lr, beta1, beta2, eps, weight_decay, step, grad_scale) ->
// status, or -1.  Arguments an operation does not take are None; a None where
// the operation takes one is the caller's, and left to the Python code.
enum { A_OP, A_GRADS, A_P, A_M, A_V, A_P16, A_AGG_F32, A_AGG_I32, A_SCALARS, A_MODE, A_FRAC,
       A_LR, A_BETA1, A_BETA2, A_EPS, A_WD, A_STEP, A_GRAD_SCALE, A_COUNT };

// The status, or -1 with or without a Python error set (the caller clears it).
int ordinary_call(PyObject *const *a)
{
    int64_t op, mode = 0, frac = 0;
    if (!lib_aggregate || !integer(a[A_OP], 0, kOpQuantize, op))
        return -1;
    constexpr int64_t kIntMin = std::numeric_limits<int>::min();
    constexpr int64_t kIntMax = std::numeric_limits<int>::max();
    const bool sums = op == kOpAggregate || op == kOpFused || op == kOpFusedDev;
    if (sums) {
        if (PyUnicode_CheckExact(a[A_MODE])) {
            if (PyUnicode_CompareWithASCIIString(a[A_MODE], "fp32") == 0)
                mode = DISDP_AGG_FP32;
            else if (PyUnicode_CompareWithASCIIString(a[A_MODE], "fixed") == 0)
                mode = DISDP_AGG_FIXED;
            else
                return -1;
        } else if (!integer(a[A_MODE], DISDP_AGG_FP32, DISDP_AGG_FIXED, mode)) {
            return -1;
        }
    }
    if ((sums || op == kOpQuantize) && !integer(a[A_FRAC], kIntMin, kIntMax, frac))
        return -1;
    const bool adam = op == kOpAdamStep || op == kOpFused || op == kOpFusedDev;
    disdp_adamw_hparams_t hp{};
    if (op == kOpAdamStep || op == kOpFused) {
        int64_t step;
        if (!number(a[A_LR], hp.lr) || !number(a[A_BETA1], hp.beta1) ||
            !number(a[A_BETA2], hp.beta2) || !number(a[A_EPS], hp.eps) ||
            !number(a[A_WD], hp.weight_decay) || !number(a[A_GRAD_SCALE], hp.grad_scale) ||
            !integer(a[A_STEP], std::numeric_limits<int64_t>::min(),
                     std::numeric_limits<int64_t>::max(), step))
            return -1;
        hp.step = step;
    }

    // the contributions: a list or tuple, or the one gradient of an operation
    // that takes one
    const void *g[disdp::kMaxW];
    PyObject *const *items = &a[A_GRADS];
    Py_ssize_t W = 1;
    Held held;   // a list may change while the library runs without the lock
    if (sums) {
        if (PyList_CheckExact(a[A_GRADS]))
            held.ref = PyList_AsTuple(a[A_GRADS]);
        else if (PyTuple_CheckExact(a[A_GRADS]))
            held.ref = Py_NewRef(a[A_GRADS]);
        if (!held.ref)
            return -1;
        items = PySequence_Fast_ITEMS(held.ref);
        W = PyTuple_GET_SIZE(held.ref);
    }
    if (W < 1 || W > disdp::kMaxW || !THPVariable_CheckExact(items[0]))
        return -1;
    Common c;
    const at::Tensor &first = THPVariable_Unpack(items[0]);
    const Kind kind = kind_of(first);
    // the length is the weight's for the optimizer step alone, else the
    // contributions'
    if (op == kOpAdamStep) {
        if (!THPVariable_CheckExact(a[A_P]))
            return -1;
        c.n = THPVariable_Unpack(a[A_P]).numel();
    } else {
        c.n = first.numel();
    }
    if (kind == kOther || (op == kOpAdamStep && kind != kF32) ||
        (op == kOpQuantize && kind == kI32))
        return -1;
    const disdp_dtype_t gdtype = kind == kF32    ? DISDP_DT_F32
                                 : kind == kHalf ? DISDP_DT_BF16
                                                 : DISDP_DT_I32;
    for (Py_ssize_t w = 0; w < W; ++w) {
        void *p;
        if (!address(items[w], kind, c.n, c, p))
            return -1;
        g[w] = p;
    }
    void *p = nullptr, *m = nullptr, *v = nullptr, *p16, *agg_f32, *agg_i32, *scalars = nullptr;
    if (adam && (!address(a[A_P], kF32, c.n, c, p) || !address(a[A_M], kF32, c.n, c, m) ||
                 !address(a[A_V], kF32, c.n, c, v)))
        return -1;
    constexpr int64_t kScalars = sizeof(disdp_step_scalars_t) / sizeof(float);
    if (op == kOpFusedDev && !address(a[A_SCALARS], kF32, kScalars, c, scalars))
        return -1;
    if (!optional_address(a[A_P16], kHalf, c.n, c, p16) ||
        !optional_address(a[A_AGG_F32], kF32, c.n, c, agg_f32) ||
        !optional_address(a[A_AGG_I32], kI32, c.n, c, agg_i32) ||
        (op == kOpQuantize && a[A_AGG_I32] == Py_None))
        return -1;

    unsigned long long device, handle;
    if (!asked(current_device, nullptr, device) || static_cast<int>(device) != c.device)
        return -1;
    PyObject *index = PyLong_FromLong(c.device);
    const bool have = index && asked(current_stream, index, handle);
    Py_XDECREF(index);
    if (!have)
        return -1;
    const hipStream_t stream = reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(handle));
    const auto f = [](void *x) { return static_cast<float *>(x); };
    const auto h = [](void *x) { return static_cast<uint16_t *>(x); };
    const auto i = [](void *x) { return static_cast<int32_t *>(x); };
    const disdp_agg_mode_t md = static_cast<disdp_agg_mode_t>(mode);
    const int k = static_cast<int>(frac), Wn = static_cast<int>(W);
    disdp_status_t st = DISDP_OK;
    Py_BEGIN_ALLOW_THREADS
    switch (op) {
    case kOpAggregate:
        st = lib_aggregate(g, Wn, gdtype, c.n, md, k, f(agg_f32), i(agg_i32), stream);
        break;
    case kOpAdamStep:
        st = lib_adam_step(static_cast<const float *>(g[0]), f(p), f(m), f(v), h(p16), c.n, &hp,
                           stream);
        break;
    case kOpFused:
        st = lib_aggregate_adam(g, Wn, gdtype, c.n, md, k, f(p), f(m), f(v), h(p16), f(agg_f32),
                                i(agg_i32), &hp, stream);
        break;
    case kOpFusedDev:
        st = lib_aggregate_adam_dev(g, Wn, gdtype, c.n, md, k, f(p), f(m), f(v), h(p16),
                                    f(agg_f32), i(agg_i32),
                                    static_cast<const disdp_step_scalars_t *>(scalars), stream);
        break;
    default:
        st = lib_quantize(g[0], gdtype, c.n, k, i(agg_i32), stream);
        break;
    }
    Py_END_ALLOW_THREADS
    return static_cast<int>(st);
}

PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t count)
{
    if (count != A_COUNT) {
        PyErr_Format(PyExc_TypeError, "call takes %d arguments", static_cast<int>(A_COUNT));
        return nullptr;
    }
    int st = -1;
    try {
        st = ordinary_call(args);
    } catch (const std::exception &) {
        st = -1;  // torch refused a query: the Python code makes it again
    }
    if (st < 0)
        PyErr_Clear();
    return PyLong_FromLong(st);
}

// bind(aggregate, adam_step, aggregate_adam, aggregate_adam_dev, quantize,
// current_device, current_stream): the addresses of the library's functions
// and torch's queries.
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long f[5];
    PyObject *device, *stream;
    if (!PyArg_ParseTuple(args, "KKKKKOO", &f[0], &f[1], &f[2], &f[3], &f[4], &device, &stream))
        return nullptr;
    Py_INCREF(device);
    Py_INCREF(stream);
    Py_XDECREF(current_device);
    Py_XDECREF(current_stream);
    current_device = device;
    current_stream = stream;
    lib_aggregate = reinterpret_cast<decltype(lib_aggregate)>(f[0]);
    lib_adam_step = reinterpret_cast<decltype(lib_adam_step)>(f[1]);
    lib_aggregate_adam = reinterpret_cast<decltype(lib_aggregate_adam)>(f[2]);
    lib_aggregate_adam_dev = reinterpret_cast<decltype(lib_aggregate_adam_dev)>(f[3]);
    lib_quantize = reinterpret_cast<decltype(lib_quantize)>(f[4]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL,
     "One call of the library, or -1 when it is not in the ordinary form."},
    {"bind", bind, METH_VARARGS, "Sets the library's functions and torch's queries."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    return PyModule_Create(&module);
}
