// xred_torch.cpp -- marshalling of torch tensors into the xred_* C ABI.
//
// A small call's kernel takes 2-3 us; checking and collecting its tensors one
// attribute at a time from Python took 6-30 us, and 1.1 ms for a batch of 256
// items of 8 sources.  These functions make the same checks on the tensors
// themselves and call the library with the interpreter lock released
// (allreduce of 8 x 8 KiB bf16 11.0 -> 4.0 us a call, that batch 1209 -> 97 us).
//
// Each returns the call's xred_status, or None, with nothing done, for
// anything but plain torch.Tensor / Parameter arguments that pass every check:
// the binding's Python code then handles the call, or raises its error.  No
// argument is kept, no result of a check is remembered.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstring>
#include <exception>
#include <vector>

#include "../../include/xred.h"

namespace {

// The library's entry points (addresses handed over by bind()) and torch's
// function that gives the current stream of a device.
decltype(&xred_allreduce_local) f_allreduce;
decltype(&xred_reduce_scatter_local) f_scatter;
decltype(&xred_reduce_copy_step) f_step;
decltype(&xred_acc_cast) f_cast;
decltype(&xred_batched_reduce) f_batched;
decltype(&xred_ring_reduce) f_ring;
decltype(&xred_allreduce_sim) f_sim;
PyObject *current_raw_stream;

// Raised to leave a call to the Python code.
struct Decline {};

struct Type {
    xred_dtype code;
    size_t size, acc;
};

bool text_is(PyObject *o, const char *s)
{
    return PyUnicode_Check(o) && PyUnicode_CompareWithASCIIString(o, s) == 0;
}

Type type_named(PyObject *name)
{
    static const struct {
        const char *name;
        Type t;
    } table[] = {
        {"f32", {XRED_FLOAT32, 4, 4}}, {"bf16", {XRED_BFLOAT16, 2, 4}},
        {"f16", {XRED_FLOAT16, 2, 4}}, {"i32", {XRED_INT32, 4, 4}},
        {"u32", {XRED_UINT32, 4, 4}}, {"i64", {XRED_INT64, 8, 8}},
        {"u64", {XRED_UINT64, 8, 8}}, {"e4m3", {XRED_FP8_E4M3, 1, 4}},
        {"e5m2", {XRED_FP8_E5M2, 1, 4}}, {"f64", {XRED_FLOAT64, 8, 8}},
        {"i8", {XRED_INT8, 1, 4}}, {"u8", {XRED_UINT8, 1, 4}}};
    for (const auto &e : table)
        if (text_is(name, e.name)) return e.t;
    throw Decline{};
}

Type type_of(const at::Tensor &t, PyObject *name)
{
    if (name != Py_None) return type_named(name);
    switch (t.scalar_type()) {
    case at::kFloat: return {XRED_FLOAT32, 4, 4};
    case at::kBFloat16: return {XRED_BFLOAT16, 2, 4};
    case at::kHalf: return {XRED_FLOAT16, 2, 4};
    case at::kInt: return {XRED_INT32, 4, 4};
    case at::kUInt32: return {XRED_UINT32, 4, 4};
    case at::kLong: return {XRED_INT64, 8, 8};
    case at::kUInt64: return {XRED_UINT64, 8, 8};
    case at::kFloat8_e4m3fn: return {XRED_FP8_E4M3, 1, 4};
    case at::kFloat8_e5m2: return {XRED_FP8_E5M2, 1, 4};
    case at::kDouble: return {XRED_FLOAT64, 8, 8};
    case at::kChar: return {XRED_INT8, 1, 4};
    case at::kByte: return {XRED_UINT8, 1, 4};
    default: throw Decline{};
    }
}

xred_op op_named(PyObject *o)
{
    if (text_is(o, "sum")) return XRED_SUM;
    if (text_is(o, "avg")) return XRED_AVG;
    if (text_is(o, "max")) return XRED_MAX;
    if (text_is(o, "min")) return XRED_MIN;
    if (text_is(o, "prod")) return XRED_PROD;
    throw Decline{};
}

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw Decline{};
    return THPVariable_Unpack(o);
}

// The data pointer of a contiguous tensor of n elements of `size` bytes on dev.
void *data_of(const at::Tensor &t, c10::Device dev, int64_t n, size_t size)
{
    if (!t.is_cuda() || t.device() != dev || !t.is_contiguous() ||
        t.element_size() != (int64_t)size || t.numel() != n)
        throw Decline{};
    return t.data_ptr();
}

// Flags or a status word: the same, or pinned host memory, of at least n words.
void *words_of(PyObject *o, c10::Device dev, int64_t n)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o);
    if (t.is_cuda() ? t.device() != dev : !t.is_pinned()) throw Decline{};
    if (!t.is_contiguous() || t.element_size() != 4 || t.numel() < n) throw Decline{};
    return t.data_ptr();
}

// A list or tuple of 1..XRED_MAX_SRC tensors.
struct Sources {
    void *p[XRED_MAX_SRC];
    int n;
    Sources(PyObject *seq, c10::Device dev, int64_t numel, size_t size)
    {
        if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) throw Decline{};
        const Py_ssize_t len = PySequence_Fast_GET_SIZE(seq);
        if (len < 1 || len > XRED_MAX_SRC) throw Decline{};
        n = (int)len;
        PyObject **o = PySequence_Fast_ITEMS(seq);
        for (int i = 0; i < n; ++i) p[i] = data_of(tensor(o[i]), dev, numel, size);
    }
};

// The stream argument: None (the device's current stream), a stream object or a handle.
void *stream_of(PyObject *o, c10::Device dev)
{
    PyObject *h;
    if (o == Py_None) {
        PyObject *index = PyLong_FromLong(dev.index());
        h = index ? PyObject_CallOneArg(current_raw_stream, index) : nullptr;
        Py_XDECREF(index);
    } else if (PyLong_CheckExact(o)) {
        h = o;
        Py_INCREF(h);
    } else {
        h = PyObject_GetAttrString(o, "cuda_stream");
    }
    void *s = h ? PyLong_AsVoidPtr(h) : nullptr;
    Py_XDECREF(h);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Decline{};
    }
    return s;
}

template <class F>
int unlocked(F &&call)
{
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = (int)call();
    Py_END_ALLOW_THREADS
    return st;
}

// The body of every function: `want` arguments; f() gives a status, and
// whatever it throws leaves the call to the Python code.
template <class F>
PyObject *entry(Py_ssize_t nargs, Py_ssize_t want, F &&f)
{
    if (nargs != want || f_allreduce == nullptr) Py_RETURN_NONE;
    try {
        return PyLong_FromLong(f());
    } catch (const Decline &) {
    } catch (const std::exception &) {
    }
    Py_RETURN_NONE;
}

// allreduce(srcs, out, op, dtype, stream)
PyObject *allreduce(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 5, [&] {
        const at::Tensor &out = tensor(a[1]);
        const c10::Device dev = out.device();
        const Type t = type_of(out, a[3]);
        const int64_t n = out.numel();
        void *dst = data_of(out, dev, n, t.size);
        const Sources s(a[0], dev, n, t.size);
        const xred_op op = op_named(a[2]);
        void *stream = stream_of(a[4], dev);
        return unlocked([&] { return f_allreduce(s.p, s.n, dst, (size_t)n, t.code, op, stream); });
    });
}

// scatter(srcs, rank, out, op, dtype, stream)
PyObject *scatter(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 6, [&] {
        const at::Tensor &out = tensor(a[2]);
        const c10::Device dev = out.device();
        const Type t = type_of(out, a[4]);
        const int64_t n = out.numel();
        void *dst = data_of(out, dev, n, t.size);
        if (!PyList_CheckExact(a[0]) && !PyTuple_CheckExact(a[0])) throw Decline{};
        if (!PyLong_CheckExact(a[1])) throw Decline{};
        int over = 0;
        const long rank = PyLong_AsLongAndOverflow(a[1], &over);
        if (over || rank != (int)rank) throw Decline{};
        const Sources s(a[0], dev, n * (int64_t)PySequence_Fast_GET_SIZE(a[0]), t.size);
        const xred_op op = op_named(a[3]);
        void *stream = stream_of(a[5], dev);
        return unlocked([&] {
            return f_scatter(s.p, s.n, (int)rank, dst, (size_t)n, t.code, op, stream);
        });
    });
}

// step(in, acc, out, op, flags, dtype, stream)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 7, [&] {
        const at::Tensor &in = tensor(a[0]);
        const c10::Device dev = in.device();
        const Type t = type_of(in, a[5]);
        const int64_t n = in.numel();
        const unsigned flags = (unsigned)PyLong_AsUnsignedLong(a[4]);
        void *src = data_of(in, dev, n, t.size), *acc = nullptr, *dst = nullptr;
        // what the flags do not use is passed on unchecked, as the library takes it
        if (flags != (XRED_STEP_INIT | XRED_STEP_FINAL))
            acc = data_of(tensor(a[1]), dev, n, t.acc);
        else if (a[1] != Py_None)
            acc = tensor(a[1]).data_ptr();
        if (flags & XRED_STEP_FINAL) dst = data_of(tensor(a[2]), dev, n, t.size);
        else if (a[2] != Py_None) dst = tensor(a[2]).data_ptr();
        const xred_op op = op_named(a[3]);
        void *stream = stream_of(a[6], dev);
        return unlocked([&] { return f_step(src, acc, dst, (size_t)n, t.code, op, flags, stream); });
    });
}

// cast(acc, out, dtype, stream)
PyObject *cast(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 4, [&] {
        const at::Tensor &out = tensor(a[1]);
        const c10::Device dev = out.device();
        const Type t = type_of(out, a[2]);
        const int64_t n = out.numel();
        void *dst = data_of(out, dev, n, t.size);
        void *acc = data_of(tensor(a[0]), dev, n, t.acc);
        void *stream = stream_of(a[3], dev);
        return unlocked([&] { return f_cast(acc, dst, (size_t)n, t.code, stream); });
    });
}

// batched(items, op, dtype, stream): a list of (sources, out) pairs
PyObject *batched(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 4, [&] {
        if (!PyList_CheckExact(a[0]) || PyList_GET_SIZE(a[0]) < 1) throw Decline{};
        const Type t = type_named(a[2]);
        const xred_op op = op_named(a[1]);
        const Py_ssize_t k = PyList_GET_SIZE(a[0]);
        if (k != (int)k) throw Decline{};
        std::vector<xred_item> items((size_t)k);
        std::vector<void *> ptrs;
        ptrs.reserve((size_t)k * 8);
        std::vector<size_t> first((size_t)k);
        c10::Device dev(c10::kCPU);
        for (Py_ssize_t i = 0; i < k; ++i) {
            PyObject *pair = PyList_GET_ITEM(a[0], i);
            if (!PyTuple_CheckExact(pair) || PyTuple_GET_SIZE(pair) != 2) throw Decline{};
            const at::Tensor &out = tensor(PyTuple_GET_ITEM(pair, 1));
            if (i == 0) dev = out.device();
            const int64_t n = out.numel();
            items[i].dst = data_of(out, dev, n, t.size);
            const Sources s(PyTuple_GET_ITEM(pair, 0), dev, n, t.size);
            first[i] = ptrs.size();
            ptrs.insert(ptrs.end(), s.p, s.p + s.n);
            items[i].count = (uint64_t)n;
            items[i].nsrc = (uint32_t)s.n;
            items[i].reserved = 0;
        }
        for (Py_ssize_t i = 0; i < k; ++i) items[i].srcs = ptrs.data() + first[i];
        void *stream = stream_of(a[3], dev);
        return unlocked([&] { return f_batched(items.data(), (int)k, t.code, op, 0, stream); });
    });
}

// ring(chunks, out, op, ready, epoch, timeout_us, status, dtype, stream)
PyObject *ring(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 9, [&] {
        const at::Tensor &out = tensor(a[1]);
        const c10::Device dev = out.device();
        const Type t = type_of(out, a[7]);
        const int64_t n = out.numel();
        void *dst = data_of(out, dev, n, t.size);
        const Sources s(a[0], dev, n, t.size);
        const xred_op op = op_named(a[2]);
        const uint32_t *ready = (const uint32_t *)words_of(a[3], dev, s.n);
        uint32_t *status = (uint32_t *)words_of(a[6], dev, 1);
        const unsigned long epoch = PyLong_AsUnsignedLongMask(a[4]);
        const unsigned long long timeout = PyLong_AsUnsignedLongLongMask(a[5]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            throw Decline{};
        }
        void *stream = stream_of(a[8], dev);
        return unlocked([&] {
            return f_ring(s.p, s.n, dst, (size_t)n, t.code, op, ready, (uint32_t)epoch, timeout,
                          status, stream);
        });
    });
}

// sim(sends, recvs, op, schedule, dtype, stream)
PyObject *sim(PyObject *, PyObject *const *a, Py_ssize_t nargs)
{
    return entry(nargs, 6, [&] {
        if ((!PyList_CheckExact(a[1]) && !PyTuple_CheckExact(a[1])) ||
            PySequence_Fast_GET_SIZE(a[1]) < 1)
            throw Decline{};
        const at::Tensor &out = tensor(PySequence_Fast_ITEMS(a[1])[0]);
        const c10::Device dev = out.device();
        const Type t = type_of(out, a[4]);
        const int64_t n = out.numel();
        const Sources recvs(a[1], dev, n, t.size), sends(a[0], dev, n, t.size);
        if (sends.n != recvs.n) throw Decline{};
        const xred_op op = op_named(a[2]);
        xred_schedule schedule;
        if (text_is(a[3], "ring")) schedule = XRED_SCHEDULE_RING;
        else if (text_is(a[3], "rhd")) schedule = XRED_SCHEDULE_RHD;
        else if (text_is(a[3], "ring1")) schedule = XRED_SCHEDULE_RING_ONE_LAUNCH;
        else if (text_is(a[3], "rhd1")) schedule = XRED_SCHEDULE_RHD_ONE_LAUNCH;
        else throw Decline{};
        void *stream = stream_of(a[5], dev);
        return unlocked([&] {
            return f_sim(sends.p, recvs.p, sends.n, (size_t)n, t.code, op, schedule, stream);
        });
    });
}

// bind(current_raw_stream, {name: address}): once, by the loader.
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *get, *addr;
    if (!PyArg_ParseTuple(args, "OO!", &get, &PyDict_Type, &addr)) return nullptr;
    auto take = [&](const char *name, auto &f) {
        PyObject *v = PyDict_GetItemString(addr, name);
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;
        f = (std::remove_reference_t<decltype(f)>)p;
        if (p == nullptr && !PyErr_Occurred())
            PyErr_Format(PyExc_ValueError, "no address for %s", name);
        return p != nullptr;
    };
    decltype(f_allreduce) all = nullptr;
    if (!take("xred_reduce_scatter_local", f_scatter) || !take("xred_reduce_copy_step", f_step) ||
        !take("xred_acc_cast", f_cast) || !take("xred_batched_reduce", f_batched) ||
        !take("xred_ring_reduce", f_ring) || !take("xred_allreduce_sim", f_sim) ||
        !take("xred_allreduce_local", all))
        return nullptr;
    Py_INCREF(get);
    Py_XSETREF(current_raw_stream, get);
    f_allreduce = all;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"allreduce", (PyCFunction)(void *)allreduce, METH_FASTCALL, nullptr},
    {"scatter", (PyCFunction)(void *)scatter, METH_FASTCALL, nullptr},
    {"step", (PyCFunction)(void *)step, METH_FASTCALL, nullptr},
    {"cast", (PyCFunction)(void *)cast, METH_FASTCALL, nullptr},
    {"batched", (PyCFunction)(void *)batched, METH_FASTCALL, nullptr},
    {"ring", (PyCFunction)(void *)ring, METH_FASTCALL, nullptr},
    {"sim", (PyCFunction)(void *)sim, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_xred_torch",
                      "Marshalling of torch tensors into the xred_* C ABI.", -1, methods};

}  // namespace

#define XRED_TEXT_(x) #x
#define XRED_TEXT(x) XRED_TEXT_(x)

// `python` and `torch`: what the module was compiled against, for the loader.
PyMODINIT_FUNC PyInit__xred_torch()
{
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr &&
        (PyModule_AddStringConstant(
             m, "python", XRED_TEXT(PY_MAJOR_VERSION) "." XRED_TEXT(PY_MINOR_VERSION)) < 0 ||
         PyModule_AddStringConstant(m, "torch",
                                    XRED_TEXT(TORCH_VERSION_MAJOR) "." XRED_TEXT(
                                        TORCH_VERSION_MINOR) "." XRED_TEXT(TORCH_VERSION_PATCH)) < 0)) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
