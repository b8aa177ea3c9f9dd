// The host side of a product call from Python: argument checks, the output tensor, the current stream and the call into the C
// ABI, without a Python-level step in between.  From Python the same takes about 5 us more per call (tensor attributes
// read one by one, torch.empty, a Stream object, ctypes), more than the kernel of a small projection: 1024 x 4096 with one
// request, called over and over, 9.1 -> 4.4 us a call (its kernel 2.8), the four calls of a Llama-3-8B block's linear layers with four
// requests 53 -> 30 us.
//
// Every function takes the call only if everything about it is as it should be (plain tensors, ints, lists, dicts; several matrices only with
// new results), and returns None otherwise: the Python code behind it then makes the same checks again and makes the call, or raises what it always raised.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bcq.h"

namespace {

decltype(&bcq_gemv_offset) g_gemv = nullptr;
decltype(&bcq_gemv_multi) g_multi = nullptr;
decltype(&bcq_gemm_mixed) g_mixed = nullptr;
decltype(&bcq_gemm_mixed_offset) g_mixed_offset = nullptr;
PyObject *g_error = nullptr;            // the exception class: (status, where)

// A plain tensor on the GPU, contiguous, of this type; nullptr otherwise.  (Subclasses, wrappers and tensors without storage go the Python way.)
const at::Tensor *gpu_tensor(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous()) return nullptr;
    return &t;
}

bool whole(PyObject *o, long &v)
{
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return v >= 0 && v <= (1L << 30);
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// other Python threads run while memory is allocated and kernels are launched, as they do during torch.empty and a ctypes call
struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

at::Tensor output(const at::Tensor &x, int64_t batch, int64_t m)
{
    WithoutGil released;
    return at::empty({batch, m}, at::TensorOptions().dtype(at::kHalf).device(x.device()));
}

template <typename F, typename... Args>
int launch(F f, Args... args)
{
    WithoutGil released;
    return f(args...);
}

// the result object, or the library's error
PyObject *finish(int status, const char *where, PyObject *y)
{
    if (status == 0) return y;
    Py_DECREF(y);
    if (PyObject *e = PyObject_CallFunction(g_error, "is", status, where)) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// planes [>= p][m][n/32], int32
const at::Tensor *planes_of(PyObject *o, int64_t &m, int64_t &n)
{
    const at::Tensor *t = gpu_tensor(o, at::kInt);
    if (!t || t->dim() != 3) return nullptr;
    m = t->size(1);
    n = t->size(2) * 32;
    return t;
}

bool scales_fit(const at::Tensor *t, int64_t p, int64_t m, int64_t ngroups)
{
    return t && t->dim() == 3 && t->size(0) == p && t->size(1) == m && t->size(2) == ngroups;
}

bool matrix_fits(const at::Tensor *t, int64_t rows, int64_t cols) { return t && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols; }

const bcq_half *half(const at::Tensor *t) { return static_cast<const bcq_half *>(t->const_data_ptr()); }

// y: the caller's tensor, or a new one; nullptr where the caller's does not fit
PyObject *result(PyObject *given, const at::Tensor &x, int64_t batch, int64_t m, bcq_half *&ptr)
{
    if (given == Py_None) {
        at::Tensor y = output(x, batch, m);
        ptr = static_cast<bcq_half *>(y.mutable_data_ptr());
        return THPVariable_Wrap(std::move(y));
    }
    const at::Tensor *y = gpu_tensor(given, at::kHalf);
    if (!matrix_fits(y, batch, m)) return nullptr;
    ptr = static_cast<bcq_half *>(y->mutable_data_ptr());
    Py_INCREF(given);
    return given;
}

// what the Python code would not get either: fall back to it and let it say so
template <typename F>
PyObject *guarded(F f)
{
    try {
        if (at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        return f();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// gemv(planes, scales_p, p, x, y, group, offsets)
PyObject *gemv(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    if (count != 7 || !g_gemv) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        long p, group;
        int64_t m, n;
        const at::Tensor *planes = planes_of(a[0], m, n), *scales = gpu_tensor(a[1], at::kHalf), *x = gpu_tensor(a[3], at::kHalf);
        if (!planes || !x || x->dim() != 2 || !whole(a[2], p) || !whole(a[5], group) || group == 0) Py_RETURN_NONE;
        const int64_t batch = x->size(0);
        if (x->size(1) != n || batch > (1 << 30) || !scales_fit(scales, p, m, n / group) || planes->size(0) < p) Py_RETURN_NONE;
        const at::Tensor *offsets = nullptr;
        if (a[6] != Py_None) {
            offsets = gpu_tensor(a[6], at::kHalf);
            if (!matrix_fits(offsets, m, n / group)) Py_RETURN_NONE;
        }
        bcq_half *to = nullptr;
        PyObject *y = result(a[4], *x, batch, m, to);
        if (!y) Py_RETURN_NONE;
        const int status = launch(g_gemv, static_cast<const uint32_t *>(planes->const_data_ptr()), half(scales), offsets ? half(offsets) : nullptr, (int)p,
                                  half(x), to, m, n, (int)batch, (int)group, stream());
        return finish(status, offsets ? "bcq_gemv_offset" : "bcq_gemv", y);
    });
}

// gemv_multi(planes, scales_p, p, x, group): lists of the matrices, new outputs
PyObject *gemv_multi(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    if (count != 5 || !g_multi) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        long p, group;
        const at::Tensor *x = gpu_tensor(a[3], at::kHalf);
        if (!PyList_CheckExact(a[0]) || !PyList_CheckExact(a[1]) || !x || x->dim() != 2 || !whole(a[2], p) || !whole(a[4], group) || group == 0)
            Py_RETURN_NONE;
        const Py_ssize_t k = PyList_GET_SIZE(a[0]);
        if (k < 1 || k > BCQ_MAX_MULTI || PyList_GET_SIZE(a[1]) != k) Py_RETURN_NONE;
        const int64_t batch = x->size(0), n = x->size(1);
        if (batch > (1 << 30)) Py_RETURN_NONE;
        const uint32_t *planes[BCQ_MAX_MULTI];
        const bcq_half *scales[BCQ_MAX_MULTI];
        int64_t ms[BCQ_MAX_MULTI];
        for (Py_ssize_t i = 0; i < k; ++i) {
            int64_t wide;
            const at::Tensor *w = planes_of(PyList_GET_ITEM(a[0], i), ms[i], wide), *s = gpu_tensor(PyList_GET_ITEM(a[1], i), at::kHalf);
            if (!w || wide != n || w->size(0) < p || !scales_fit(s, p, ms[i], n / group)) Py_RETURN_NONE;
            planes[i] = static_cast<const uint32_t *>(w->const_data_ptr());
            scales[i] = half(s);
        }
        PyObject *ys = PyList_New(k);
        if (!ys) return nullptr;
        bcq_half *to[BCQ_MAX_MULTI];
        for (Py_ssize_t i = 0; i < k; ++i) {
            PyObject *y = nullptr;
            try {
                y = result(Py_None, *x, batch, ms[i], to[i]);
            } catch (...) {
            }
            if (!y) {
                PyErr_Clear();
                Py_DECREF(ys);
                Py_RETURN_NONE;
            }
            PyList_SET_ITEM(ys, i, y);
        }
        return finish(launch(g_multi, (int)k, planes, scales, ms, to, (int)p, half(x), n, (int)batch, (int)group, stream()), "bcq_gemv_multi", ys);
    });
}

// sets by precision: a dict of whole numbers to tensors, their pointers in by_p[1 .. p_max]
template <typename Fits>
bool sets_of(PyObject *dict, int64_t p_max, const bcq_half **by_p, Fits fits)
{
    PyObject *key, *value;
    Py_ssize_t pos = 0;
    while (PyDict_Next(dict, &pos, &key, &value)) {
        long q;
        if (!whole(key, q) || q < 1 || q > p_max) return false;
        const at::Tensor *t = gpu_tensor(value, at::kHalf);
        if (!fits(t, q)) return false;
        by_p[q] = half(t);
    }
    return true;
}

// gemm_mixed(planes, scales_by_p, p_req, x, y, group, offsets_by_p)
PyObject *gemm_mixed(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    if (count != 7 || !g_mixed) Py_RETURN_NONE;
    return guarded([&]() -> PyObject * {
        long group;
        int64_t m, n;
        const at::Tensor *planes = planes_of(a[0], m, n), *p_req = gpu_tensor(a[2], at::kInt), *x = gpu_tensor(a[3], at::kHalf);
        if (!planes || !p_req || !x || x->dim() != 2 || !PyDict_CheckExact(a[1]) || !whole(a[5], group) || group == 0) Py_RETURN_NONE;
        const int64_t p_max = planes->size(0), batch = x->size(0);
        if (p_max < 1 || p_max > BCQ_MAX_PLANES || batch > (1 << 30) || x->size(1) != n || p_req->dim() != 1 || p_req->size(0) != batch) Py_RETURN_NONE;
        const bcq_half *scales[BCQ_MAX_PLANES + 1] = {}, *offsets[BCQ_MAX_PLANES + 1] = {};
        const int64_t ngroups = n / group;
        if (!sets_of(a[1], p_max, scales, [&](const at::Tensor *t, long q) { return scales_fit(t, q, m, ngroups); })) Py_RETURN_NONE;
        bool with_offsets = false;
        if (a[6] != Py_None) {
            if (!PyDict_CheckExact(a[6])) Py_RETURN_NONE;
            with_offsets = PyDict_Size(a[6]) > 0;
            if (!sets_of(a[6], p_max, offsets, [&](const at::Tensor *t, long) { return matrix_fits(t, m, ngroups); })) Py_RETURN_NONE;
        }
        bcq_half *to = nullptr;
        PyObject *y = result(a[4], *x, batch, m, to);
        if (!y) Py_RETURN_NONE;
        const uint32_t *w = static_cast<const uint32_t *>(planes->const_data_ptr());
        const int32_t *req = static_cast<const int32_t *>(p_req->const_data_ptr());
        if (with_offsets)
            return finish(launch(g_mixed_offset, w, scales, offsets, req, (int)p_max, half(x), to, m, n, (int)batch, (int)group, stream()),
                          "bcq_gemm_mixed_offset", y);
        return finish(launch(g_mixed, w, scales, req, (int)p_max, half(x), to, m, n, (int)batch, (int)group, stream()), "bcq_gemm_mixed", y);
    });
}

// bind(gemv_offset, gemv_multi, gemm_mixed, gemm_mixed_offset, error): addresses of the C ABI's functions in the library that is loaded
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long f[4];
    PyObject *error;
    if (!PyArg_ParseTuple(args, "KKKKO", &f[0], &f[1], &f[2], &f[3], &error)) return nullptr;
    g_gemv = reinterpret_cast<decltype(g_gemv)>(f[0]);
    g_multi = reinterpret_cast<decltype(g_multi)>(f[1]);
    g_mixed = reinterpret_cast<decltype(g_mixed)>(f[2]);
    g_mixed_offset = reinterpret_cast<decltype(g_mixed_offset)>(f[3]);
    Py_INCREF(error);
    Py_XSETREF(g_error, error);
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"gemv", (PyCFunction)(void (*)(void))gemv, METH_FASTCALL, nullptr},
                           {"gemv_multi", (PyCFunction)(void (*)(void))gemv_multi, METH_FASTCALL, nullptr},
                           {"gemm_mixed", (PyCFunction)(void (*)(void))gemm_mixed, METH_FASTCALL, nullptr},
                           {"bind", bind, METH_VARARGS, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_bcq_host", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// the torch this was built against, as torch.__version__ has it: another one's tensors may be laid out differently
constexpr char kBuiltFor[] = "built for torch " BCQ_TORCH_VERSION;

PyMODINIT_FUNC PyInit__bcq_host(void)
{
    PyObject *module = PyModule_Create(&g_module);
    if (module && PyModule_AddStringConstant(module, "torch_version", kBuiltFor + sizeof "built for torch " - 1) != 0) Py_CLEAR(module);
    return module;
}
