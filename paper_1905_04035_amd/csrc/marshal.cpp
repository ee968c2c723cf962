// Marshalling of the binding's calls: PyTorch tensors in, the C ABI's pointers and sizes out.  A Python extension module
// of its own, because in Python the checks and conversions cost 5.5 us for a call on one buffer and 15.6 us for one on
// thirteen, more than the launches: the host needed 12.3 and 22.4 us for a whole call, now 7.1 and 7.1 (a gather of three
// gradients, one launch, 13.6 and 6.3), while the GPU needs 8-15 us for the smallest.
// Every function gets the address of the library's entry point first, checks what the entry point cannot see (device,
// type, contiguity, lengths: AssertionError), and returns the entry point's status.
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "ts_densify.h"

namespace {

PyObject* g_current_device = nullptr;       // torch._C._cuda_getDevice()
PyObject* g_current_stream = nullptr;       // torch._C._cuda_getCurrentRawStream(device)

struct Failed {};       // a Python error is set

void require(bool ok)
{
    if (ok) return;
    PyErr_SetNone(PyExc_AssertionError);
    throw Failed();
}

const at::Tensor& tensor(PyObject* o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
        throw Failed();
    }
    return THPVariable_Unpack(o);
}

int64_t integer(PyObject* o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failed();
    return v;
}

// An argument of the C ABI that is 32 bits wide.
int32_t integer32(PyObject* o)
{
    const int64_t v = integer(o);
    if (v != (int32_t)v) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit 32 bits");
        throw Failed();
    }
    return (int32_t)v;
}

void* address(PyObject* o)
{
    void* const p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Failed();
    return p;
}

void* stream_of(PyObject* stream)
{
    PyObject* raw;
    if (stream == Py_None) {
        PyObject* const device = PyObject_CallNoArgs(g_current_device);
        if (!device) throw Failed();
        raw = PyObject_CallOneArg(g_current_stream, device);
        Py_DECREF(device);
    } else {
        raw = PyObject_GetAttrString(stream, "cuda_stream");
    }
    if (!raw) throw Failed();
    void* const p = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    if (!p && PyErr_Occurred()) throw Failed();
    return p;
}

bool fp32_on_gpu(const at::Tensor& t) { return t.is_cuda() && t.scalar_type() == at::kFloat && t.is_contiguous(); }

float* dense(PyObject* o, int64_t V, int64_t d)
{
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    require(fp32_on_gpu(t) && t.dim() == 2 && t.size(0) == V && t.size(1) == d);
    return static_cast<float*>(t.data_ptr());
}

// ids and value rows of one contribution: elem 4 (float32) or 2 (any 2-byte type that holds bf16 bits).
struct Pair {
    const int32_t* ids;
    const void* rows;
    int64_t n;
};

Pair pair(PyObject* ids_o, PyObject* rows_o, int64_t d, int elem, bool any_type)
{
    const at::Tensor &ids = tensor(ids_o), &rows = tensor(rows_o);
    require(ids.is_cuda() && ids.scalar_type() == at::kInt && ids.is_contiguous());
    require(rows.is_cuda() && rows.is_contiguous() && (any_type ? (int)rows.element_size() == elem : rows.scalar_type() == at::kFloat));
    const int64_t n = ids.numel();
    require(rows.numel() == n * d);
    return Pair{static_cast<const int32_t*>(ids.data_ptr()), rows.data_ptr(), n};
}

// The items of something that has a length (an iterator, whose items nobody else holds, has none: TypeError).  New reference.
PyObject* items(PyObject* o, const char* otherwise)
{
    if (PyObject_Size(o) < 0) throw Failed();
    PyObject* const list = PySequence_Fast(o, otherwise);
    if (!list) throw Failed();
    return list;
}

struct Shards {
    std::vector<const int32_t*> ids;
    std::vector<const void*> rows;
    std::vector<int64_t> n;
    int32_t k;

    Shards(PyObject* ids_k, PyObject* rows_k, int32_t row_dtype, int64_t d)
    {
        PyObject* const i = items(ids_k, "ids_k is not a sequence");
        PyObject* r = nullptr;
        try {
            r = items(rows_k, "rows_k is not a sequence");
            const Py_ssize_t m = PySequence_Fast_GET_SIZE(i);
            require(m == PySequence_Fast_GET_SIZE(r) && m == (int32_t)m);
            k = (int32_t)m;
            ids.resize(m + 1);
            rows.resize(m + 1);
            n.resize(m + 1);
            for (Py_ssize_t j = 0; j < m; ++j) {
                const Pair p = pair(PySequence_Fast_GET_ITEM(i, j), PySequence_Fast_GET_ITEM(r, j), d, row_dtype == TS_ROW_BF16 ? 2 : 4, true);
                ids[j] = p.ids;
                rows[j] = p.rows;
                n[j] = p.n;
            }
        } catch (...) {
            Py_DECREF(i);
            Py_XDECREF(r);
            throw;
        }
        Py_DECREF(i);
        Py_DECREF(r);
    }
};

// Runs f with the interpreter's lock given back and returns its status.
template <typename F>
PyObject* status(F&& f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// No C++ exception leaves the module.
template <typename F>
PyObject* guarded(Py_ssize_t nargs, Py_ssize_t want, F&& f)
{
    if (nargs != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", nargs, want);
        return nullptr;
    }
    try {
        return f();
    } catch (const Failed&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// densify(entry, elem, ids, rows, d, V, dense_in, dense_out, stream)
PyObject* densify(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    return guarded(nargs, 9, [&] {
        const auto fn = reinterpret_cast<decltype(&ts_densify)>(address(a[0]));
        const int elem = (int)integer(a[1]);
        const int32_t d = integer32(a[4]), V = integer32(a[5]);
        const Pair p = pair(a[2], a[3], d, elem, elem == 2);
        require(a[7] != Py_None);
        float* const out = dense(a[7], V, d);
        const float* const in = dense(a[6], V, d);
        void* const stream = stream_of(a[8]);
        // (ts_densify, ts_densify_static and ts_densify_bf16 differ in the type that rows points to only)
        return status([&] { return fn(p.ids, static_cast<const float*>(p.rows), p.n, d, V, in, out, stream); });
    });
}

// multi(entry, ids_k, rows_k, row_dtype, d, V, dense_in, dense_out, stream)
PyObject* multi(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    return guarded(nargs, 9, [&] {
        const auto fn = reinterpret_cast<decltype(&ts_densify_multi)>(address(a[0]));
        const int32_t row_dtype = integer32(a[3]), d = integer32(a[4]), V = integer32(a[5]);
        const Shards s(a[1], a[2], row_dtype, d);
        require(a[7] != Py_None);
        float* const out = dense(a[7], V, d);
        const float* const in = dense(a[6], V, d);
        void* const stream = stream_of(a[8]);
        return status([&] { return fn(s.ids.data(), s.rows.data(), s.n.data(), s.k, row_dtype, d, V, in, out, stream); });
    });
}

// scaled(entry, ids_k, rows_k, row_dtype, d, V, dense_in, out, scale, stream)
PyObject* scaled(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    return guarded(nargs, 10, [&] {
        const auto fn = reinterpret_cast<decltype(&ts_densify_scaled)>(address(a[0]));
        const int32_t row_dtype = integer32(a[3]), d = integer32(a[4]), V = integer32(a[5]);
        const Shards s(a[1], a[2], row_dtype, d);
        const at::Tensor& out = tensor(a[7]);
        require(out.is_cuda() && out.is_contiguous() && out.numel() == (int64_t)V * d);
        require(out.scalar_type() == at::kFloat || out.element_size() == 2);
        const float* const in = dense(a[6], V, d);
        const double scale = PyFloat_AsDouble(a[8]);
        if (scale == -1.0 && PyErr_Occurred()) throw Failed();
        void* const stream = stream_of(a[9]);
        void* const to = out.data_ptr();
        const int32_t out_dtype = out.scalar_type() == at::kFloat ? TS_OUT_FP32 : TS_OUT_BF16;
        return status([&] {
            return fn(s.ids.data(), s.rows.data(), s.n.data(), s.k, row_dtype, d, V, in, to, out_dtype, (float)scale, stream);
        });
    });
}

// range(entry, ids_k, rows_k, row_dtype, d, V, v_begin, v_end, dense_in, dense_out, stream)
PyObject* range(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    return guarded(nargs, 11, [&] {
        const auto fn = reinterpret_cast<decltype(&ts_densify_range)>(address(a[0]));
        const int32_t row_dtype = integer32(a[3]), d = integer32(a[4]), V = integer32(a[5]), v0 = integer32(a[6]), v1 = integer32(a[7]);
        const Shards s(a[1], a[2], row_dtype, d);
        require(a[9] != Py_None);
        float* const out = dense(a[9], (int64_t)v1 - v0, d);
        const float* const in = dense(a[8], (int64_t)v1 - v0, d);
        void* const stream = stream_of(a[10]);
        return status([&] { return fn(s.ids.data(), s.rows.data(), s.n.data(), s.k, row_dtype, d, V, v0, v1, in, out, stream); });
    });
}

// accumulate(entry, strategy entry, grads, rule, d, V, dense_out, ids_out, rows_out, stream) -> (status, strategy, slices)
// grads: ("dense", tensor) or ("slices", ids, rows).  Gradients and the outputs that the rule's branch writes hold at least
// what the call reads and writes (flat and longer buffers are fine); outputs that it does not write are not looked at, but for
// rows_out, which holds what ids_out has room for.
PyObject* accumulate(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    return guarded(nargs, 10, [&]() -> PyObject* {
        const auto fn = reinterpret_cast<decltype(&ts_accumulate)>(address(a[0]));
        const auto strategy_fn = reinterpret_cast<decltype(&ts_accumulate_strategy)>(address(a[1]));
        const int32_t rule = integer32(a[3]), d = integer32(a[4]), V = integer32(a[5]);
        const bool shape_ok = V > 0 && d > 0 && d % 4 == 0;             // (else the entry point refuses the call)
        const int64_t vd = shape_ok ? (int64_t)V * d : 0;
        std::vector<ts_grad> grads;
        PyObject* const list = items(a[2], "grads is not a sequence");
        try {
            const Py_ssize_t m = PySequence_Fast_GET_SIZE(list);
            require(m == (int32_t)m);
            grads.resize(m + 1);
            for (Py_ssize_t j = 0; j < m; ++j) {
                PyObject* const one = items(PySequence_Fast_GET_ITEM(list, j), "a gradient is not a sequence");
                try {
                    ts_grad g{};
                    const Py_ssize_t parts = PySequence_Fast_GET_SIZE(one);
                    require(parts > 0);
                    PyObject* const kind = PySequence_Fast_GET_ITEM(one, 0);
                    const bool is_dense = PyUnicode_Check(kind) && PyUnicode_CompareWithASCIIString(kind, "dense") == 0;
                    require(parts >= (is_dense ? 2 : 3));
                    if (is_dense) {
                        const at::Tensor& t = tensor(PySequence_Fast_GET_ITEM(one, 1));
                        require(fp32_on_gpu(t) && t.numel() >= vd);
                        g.kind = TS_GRAD_DENSE;
                        g.values = static_cast<const float*>(t.data_ptr());
                    } else {
                        const at::Tensor &ids = tensor(PySequence_Fast_GET_ITEM(one, 1)), &rows = tensor(PySequence_Fast_GET_ITEM(one, 2));
                        require(ids.is_cuda() && ids.scalar_type() == at::kInt && ids.is_contiguous());
                        require(fp32_on_gpu(rows) && (!shape_ok || rows.numel() / d >= ids.numel()));
                        g.kind = TS_GRAD_SLICES;
                        g.ids = static_cast<const int32_t*>(ids.data_ptr());
                        g.values = static_cast<const float*>(rows.data_ptr());
                        g.n = ids.numel();
                    }
                    grads[j] = g;
                } catch (...) {
                    Py_DECREF(one);
                    throw;
                }
                Py_DECREF(one);
            }
        } catch (...) {
            Py_DECREF(list);
            throw;
        }
        Py_DECREF(list);
        const int32_t m = (int32_t)grads.size() - 1;
        int32_t branch = -1;
        const bool known = strategy_fn(grads.data(), m, rule, &branch) == TS_OK;
        const bool to_dense = known && (branch == TS_ACC_REDUCE || branch == TS_ACC_DENSIFY_REDUCE ||
                                        (branch == TS_ACC_PASS_THROUGH && grads[0].kind == TS_GRAD_DENSE));
        int64_t capacity = 0;
        int32_t* ids_out = nullptr;
        float *rows_out = nullptr, *dense_out = nullptr;
        if (a[7] != Py_None) {
            const at::Tensor& t = tensor(a[7]);
            require(!known || to_dense || (t.is_cuda() && t.scalar_type() == at::kInt && t.is_contiguous()));
            capacity = t.numel();
            ids_out = static_cast<int32_t*>(t.data_ptr());
        }
        if (a[8] != Py_None) {
            const at::Tensor& t = tensor(a[8]);
            require(t.is_cuda() && t.scalar_type() == at::kFloat && t.numel() >= capacity * d);
            require(!known || to_dense || t.is_contiguous());
            rows_out = static_cast<float*>(t.data_ptr());
        }
        if (a[6] != Py_None) {
            const at::Tensor& t = tensor(a[6]);
            require(!to_dense || (fp32_on_gpu(t) && t.numel() >= vd));
            dense_out = static_cast<float*>(t.data_ptr());
        }
        void* const stream = stream_of(a[9]);
        int64_t slices = -1;
        int32_t strategy = -1;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = fn(grads.data(), m, rule, d, V, dense_out, ids_out, rows_out, capacity, &slices, &strategy, stream);
        Py_END_ALLOW_THREADS
        return Py_BuildValue("iiL", rc, (int)strategy, (long long)slices);
    });
}

PyMethodDef methods[] = {
    {"densify", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(densify)), METH_FASTCALL, nullptr},
    {"multi", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(multi)), METH_FASTCALL, nullptr},
    {"scaled", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(scaled)), METH_FASTCALL, nullptr},
    {"range", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(range)), METH_FASTCALL, nullptr},
    {"accumulate", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(accumulate)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* const c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_current_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_current_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    Py_DECREF(c);
    if (!g_current_device || !g_current_stream) return nullptr;
    return PyModule_Create(&module);
}
