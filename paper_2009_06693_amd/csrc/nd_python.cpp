// The sampling calls as Python functions (module _nd_call): they check tensors, collect their addresses and call the
// library.  A walk of 100 steps hands over 100 output arrays; checked and collected tensor by tensor through Python
// attributes and ctypes they cost the host 35 us for a sampling and a gathering call, more than the GPU works on 4,096
// walks, and a k-hop call 4 us.  The library's entry points come as addresses (init), so the module is
// independent of which library binding.py has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>
#include <vector>

#include "../../include/nd.h"

namespace {

using SampleFn = int (*)(const void*, int, const void*, const int32_t*, int64_t, uint64_t, int32_t* const*, void*, size_t,
                         void*);
using StaticFn = int (*)(const void*, int, const void*, const int32_t*, int64_t, uint64_t, int32_t* const*, uint32_t*,
                         void*);
using PackFn = int (*)(const int32_t* const*, int32_t, const int64_t*, int64_t, int32_t*, void*);
SampleFn g_sample = nullptr;
StaticFn g_static = nullptr;
PackFn g_pack = nullptr;

// An address or handle given as an integer, None for null.
bool as_address(PyObject* o, void** out) {
    *out = nullptr;
    if (o == Py_None) return true;
    *out = PyLong_AsVoidPtr(o);
    return !(*out == nullptr && PyErr_Occurred());
}

const at::Tensor* as_tensor(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) {
        PyErr_SetString(PyExc_TypeError, what);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

bool is_array(const at::Tensor& t) {
    return t.scalar_type() == at::kInt && t.is_cuda() && t.is_contiguous();
}

// Memory that a kernel reaches at the tensor's address: the GPU's, or pinned on the host.
bool is_reachable(const at::Tensor& t) { return t.is_cuda() || t.is_pinned(); }

// The tensors of a sequence: contiguous int32 arrays on a GPU.
struct Arrays {
    std::vector<int32_t*> ptr;
    std::vector<int64_t> len;
    bool take(PyObject* seq, const char* complaint, int64_t at_least = 0) {
        PyObject* fast = PySequence_Fast(seq, complaint);
        if (!fast) return false;
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
        if (n < at_least) {
            PyErr_Format(PyExc_ValueError, "%zd arrays for %lld steps", n, (long long)at_least);
            Py_DECREF(fast);
            return false;
        }
        ptr.reserve((size_t)n);
        len.reserve((size_t)n);
        bool ok = true;
        for (Py_ssize_t i = 0; ok && i < n; ++i) {
            const at::Tensor* t = as_tensor(PySequence_Fast_GET_ITEM(fast, i), complaint);
            ok = t != nullptr;
            if (ok && !is_array(*t)) {
                PyErr_SetString(PyExc_TypeError, complaint);
                ok = false;
            }
            if (ok) {
                ptr.push_back((int32_t*)t->data_ptr());
                len.push_back(t->numel());
            }
        }
        Py_DECREF(fast);
        return ok;
    }
};

constexpr const char* kRoots = "roots must be a contiguous int32 CUDA tensor";
constexpr const char* kOutputs = "outputs must be contiguous int32 CUDA tensors";
constexpr const char* kSteps = "step arrays must be contiguous int32 CUDA tensors";

// What both sampling calls take: handle, app, params, roots, seed, outputs.
struct Call {
    void* handle = nullptr;
    int app = 0;
    Py_buffer params{};
    const int32_t* roots = nullptr;
    int64_t num_roots = 0;
    uint64_t seed = 0;
    Arrays out;
    ~Call() {
        if (params.obj) PyBuffer_Release(&params);
    }
    bool take(PyObject* const* a) {
        if (!as_address(a[0], &handle)) return false;
        app = (int)PyLong_AsUnsignedLongMask(a[1]);  // what has __index__ counts as an integer, NumPy's integers too
        if (PyErr_Occurred()) return false;
        seed = PyLong_AsUnsignedLongLongMask(a[4]);
        if (PyErr_Occurred()) return false;
        if (PyObject_GetBuffer(a[2], &params, PyBUF_SIMPLE) != 0) return false;  // the ctypes structure itself
        if (params.len != (Py_ssize_t)sizeof(nd_params)) {
            PyErr_SetString(PyExc_TypeError, "params must be an nd_params");
            return false;
        }
        const at::Tensor* r = as_tensor(a[3], kRoots);
        if (!r) return false;
        if (!is_array(*r)) {
            PyErr_SetString(PyExc_TypeError, kRoots);
            return false;
        }
        num_roots = r->numel();
        // the library reads an address per step and has no count of them
        nd_params p;
        std::memcpy(&p, params.buf, sizeof p);
        const int64_t steps = p.num_steps <= ND_MAX_WALK_STEPS ? p.num_steps : 0;  // more than that it refuses
        if (!out.take(a[5], kOutputs, num_roots > 0 ? steps : 0)) return false;
        if ((int64_t)out.ptr.size() < steps) out.ptr.resize((size_t)steps, nullptr);
        roots = (const int32_t*)r->data_ptr();
        return true;
    }
};

bool expects(Py_ssize_t got, Py_ssize_t want) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, expected %zd", got, want);
    return false;
}

PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void *s, *t, *p;
    if (!expects(n, 4) || !as_address(a[0], &s) || !as_address(a[1], &t) || !as_address(a[2], &p)) return nullptr;
    const Py_ssize_t params_size = PyLong_AsSsize_t(a[3]);
    if (params_size < 0 && PyErr_Occurred()) return nullptr;
    if (params_size != (Py_ssize_t)sizeof(nd_params)) {
        PyErr_Format(PyExc_TypeError, "nd_params of %zd bytes, expected %zu", params_size, sizeof(nd_params));
        return nullptr;
    }
    g_sample = (SampleFn)s;
    g_static = (StaticFn)t;
    g_pack = (PackFn)p;
    Py_RETURN_NONE;
}

// sample(handle, app, params, roots, seed, outputs, workspace, stream) -> code
PyObject* sample(PyObject*, PyObject* const* a, Py_ssize_t n) try {
    Call c;
    void* stream;
    if (!expects(n, 8) || !c.take(a) || !as_address(a[7], &stream)) return nullptr;
    constexpr const char* kWorkspace = "workspace must be a CUDA tensor without gaps";
    const at::Tensor* w = as_tensor(a[6], kWorkspace);
    if (!w) return nullptr;
    if (!is_reachable(*w) || !w->is_non_overlapping_and_dense()) {
        PyErr_SetString(PyExc_TypeError, kWorkspace);
        return nullptr;
    }
    void* ws = w->data_ptr();
    const size_t bytes = (size_t)w->numel() * (size_t)w->element_size();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_sample(c.handle, c.app, c.params.buf, c.roots, c.num_roots, c.seed, c.out.ptr.data(), ws, bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
} catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
}

// sample_static(handle, app, params, roots, seed, outputs, status or None, stream) -> code
PyObject* sample_static(PyObject*, PyObject* const* a, Py_ssize_t n) try {
    Call c;
    void* stream;
    if (!expects(n, 8) || !c.take(a) || !as_address(a[7], &stream)) return nullptr;
    uint32_t* status = nullptr;
    if (a[6] != Py_None) {
        constexpr const char* kStatus = "status must be a CUDA tensor of one 32-bit element";
        const at::Tensor* s = as_tensor(a[6], kStatus);
        if (!s) return nullptr;
        const bool holds = s->numel() > 0 && (size_t)s->numel() * (size_t)s->element_size() >= sizeof(uint32_t);
        if (!holds || !is_reachable(*s) || !s->is_non_overlapping_and_dense()) {
            PyErr_SetString(PyExc_TypeError, kStatus);
            return nullptr;
        }
        status = (uint32_t*)s->data_ptr();
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_static(c.handle, c.app, c.params.buf, c.roots, c.num_roots, c.seed, c.out.ptr.data(), status, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
} catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
}

// Entries of one record.
int64_t record_of(const Arrays& steps, int64_t num_samples) {
    int64_t length = 0;
    if (num_samples > 0)
        for (int64_t len : steps.len) length += len / num_samples;
    return length;
}

// pack(step arrays, samples, records, stream) -> code
PyObject* pack(PyObject*, PyObject* const* a, Py_ssize_t n) try {
    Arrays steps;
    void* stream;
    if (!expects(n, 4) || !steps.take(a[0], kSteps)) return nullptr;
    const int64_t num_samples = PyLong_AsLongLong(a[1]);
    if (PyErr_Occurred()) return nullptr;
    constexpr const char* kRecords = "samples must be a contiguous int32 CUDA tensor of num_samples * record entries";
    const at::Tensor* r = as_tensor(a[2], kRecords);
    if (!r || !as_address(a[3], &stream)) return nullptr;
    if (r->scalar_type() != at::kInt || r->numel() < num_samples * record_of(steps, num_samples) || !r->is_contiguous() ||
        (r->numel() > 0 && !is_reachable(*r))) {
        PyErr_SetString(PyExc_TypeError, kRecords);
        return nullptr;
    }
    int32_t* records = r->numel() > 0 ? (int32_t*)r->data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_pack(steps.ptr.data(), (int32_t)steps.ptr.size(), steps.len.data(), num_samples, records, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
} catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
}

// record_length(step arrays, samples): entries of one record, after the same check of the arrays
PyObject* record_length(PyObject*, PyObject* const* a, Py_ssize_t n) try {
    Arrays steps;
    if (!expects(n, 2) || !steps.take(a[0], kSteps)) return nullptr;
    const int64_t num_samples = PyLong_AsLongLong(a[1]);
    if (PyErr_Occurred()) return nullptr;
    return PyLong_FromLongLong(record_of(steps, num_samples));
} catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)(void (*)())init, METH_FASTCALL, nullptr},
    {"sample", (PyCFunction)(void (*)())sample, METH_FASTCALL, nullptr},
    {"sample_static", (PyCFunction)(void (*)())sample_static, METH_FASTCALL, nullptr},
    {"pack", (PyCFunction)(void (*)())pack, METH_FASTCALL, nullptr},
    {"record_length", (PyCFunction)(void (*)())record_length, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nd_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nd_call(void) { return PyModule_Create(&module); }
