// Python extension module `_call`: the device calls of binding.py without ctypes.  A short call is
// bound by its host time: one image's softmax is a kernel of 2.3 us (in a graph) and cost 5.1 us per call
// through ctypes, 3.7 here; its GELU 4.6 and 3.2.  The launch itself is 2.5 to 3 of those.  So the ordinary
// case is checked and converted here.
//
// Every function takes the arguments of its namesake in binding.py and returns the library's return
// code, or None if any of them is not what this path takes (another type, too few elements, an
// integer that does not fit): nothing has been called then, and the caller goes the long way, which
// raises what it always raised.  It calls the library through the addresses it was given.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/iptq.h"

namespace {

// bound by bind(): entry points of the loaded library and the parameter classes of binding.py
struct Bound {
    decltype(&iptq_requant) requant;
    decltype(&iptq_softmax_i32) softmax_i32;
    decltype(&iptq_softmax_i32_windowed) windowed;
    decltype(&iptq_softmax_i32_windowed_bits) windowed_bits;
    decltype(&iptq_gelu_i8) gelu_i8;
    decltype(&iptq_gelu_i32) gelu_i32;
    decltype(&iptq_softmax_i32_layers) softmax_layers;
    decltype(&iptq_gelu_i8_layers) gelu_layers;
    PyTypeObject *softmax_params, *gelu_params, *dyadic;
} g = {};

// A contiguous tensor of that type on the GPU, of class torch.Tensor itself: its address.
bool tensor(PyObject *o, at::ScalarType type, int64_t least, void **p)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || t.numel() < least) return false;
    *p = t.data_ptr();
    return true;
}

bool integer(PyObject *o, int64_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool integer(PyObject *o, int32_t *v)
{
    int64_t w = 0;
    if (!integer(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
    *v = (int32_t)w;
    return true;
}

// rows x cols, or -1 where that is no element count (left to the long way)
int64_t elements(int64_t rows, int64_t cols)
{
    int64_t n = 0;
    return rows < 0 || cols < 0 || __builtin_mul_overflow(rows, cols, &n) ? -1 : n;
}

// A copy of a parameter structure of exactly that class.
template <typename T>
bool structure(PyObject *o, PyTypeObject *type, T *out)
{
    if (Py_TYPE(o) != type) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = view.len == (Py_ssize_t)sizeof(T);
    if (ok) memcpy(out, view.buf, sizeof(T));
    PyBuffer_Release(&view);
    return ok;
}
template <typename T>
bool structures(PyObject *o, PyTypeObject *type, int32_t n, std::vector<T> *out)
{
    if (!(PyList_CheckExact(o) || PyTuple_CheckExact(o)) || n < 1 || PySequence_Fast_GET_SIZE(o) != n) return false;
    out->resize(n);
    for (int32_t i = 0; i < n; ++i)
        if (!structure(PySequence_Fast_GET_ITEM(o, i), type, &(*out)[i])) return false;
    return true;
}

// Runs the call on torch's current stream without the interpreter's lock, as ctypes does.
template <typename F>
PyObject *enqueue(F call)
{
    void *const stream = c10::hip::getCurrentHIPStream().stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// Anything torch throws (a tensor without storage, say) is left to the long way.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        PyObject *r = F(a, n);
        if (r != nullptr) return r;
    } catch (...) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

at::ScalarType byte_type(int is_signed) { return is_signed ? at::kChar : at::kByte; }

PyObject *requant(PyObject *const *a, Py_ssize_t n_args)
{
    void *in, *out;
    int64_t n;
    int32_t is_signed;
    iptq_dyadic_t p;
    if (n_args != 5 || g.requant == nullptr || !integer(a[2], &n) || n < 0 || !integer(a[3], &is_signed) ||
        !tensor(a[0], at::kInt, n, &in) || !tensor(a[1], byte_type(is_signed), n, &out) || !structure(a[4], g.dyadic, &p))
        return nullptr;
    return enqueue([&](void *s) { return g.requant((const int32_t *)in, out, n, is_signed, &p, s); });
}

// scores, bias, period, then `skip` arguments of the mask, out, rows, cols, params
struct SoftmaxArguments {
    void *scores, *bias, *out;
    int64_t period, rows;
    int32_t cols;
    iptq_softmax_params_t p;
    bool take(PyObject *const *a, int skip)
    {
        PyObject *const *b = a + 3 + skip;
        bias = nullptr;
        if (!integer(b[1], &rows) || !integer(b[2], &cols) || !integer(a[2], &period) ||
            !structure(b[3], g.softmax_params, &p))
            return false;
        const int64_t n = elements(rows, cols);
        if (n < 0 || !tensor(a[0], at::kInt, n, &scores) || !tensor(b[0], byte_type(p.out_is_signed), n, &out)) return false;
        if (a[1] == Py_None) return true;
        const int64_t table = elements(period, cols);
        return table >= 0 && tensor(a[1], at::kInt, table, &bias);
    }
};

PyObject *softmax_i32(PyObject *const *a, Py_ssize_t n_args)
{
    SoftmaxArguments s;
    if (n_args != 7 || g.softmax_i32 == nullptr || !s.take(a, 0)) return nullptr;
    return enqueue([&](void *st) {
        return g.softmax_i32((const int32_t *)s.scores, (const int32_t *)s.bias, s.period, s.out, s.rows, s.cols, &s.p, st);
    });
}

template <bool BITS>
PyObject *windowed(PyObject *const *a, Py_ssize_t n_args)
{
    SoftmaxArguments s;
    int32_t windows, heads;
    void *mask = nullptr;
    if (n_args != 10 || g.windowed == nullptr || !integer(a[4], &windows) || !integer(a[5], &heads) || !s.take(a, 3)) return nullptr;
    if (a[3] != Py_None) {
        const int64_t queries = elements(windows, s.cols);
        const int64_t n = queries < 0 ? -1 : elements(queries, BITS ? ((int64_t)s.cols + 63) / 64 : s.cols);
        if (n < 0 || !tensor(a[3], BITS ? at::kLong : at::kInt, n, &mask)) return nullptr;
    }
    return enqueue([&](void *st) {
        if (BITS)
            return g.windowed_bits((const int32_t *)s.scores, (const int32_t *)s.bias, s.period, (const uint64_t *)mask, windows,
                                   heads, s.out, s.rows, s.cols, &s.p, st);
        return g.windowed((const int32_t *)s.scores, (const int32_t *)s.bias, s.period, (const int32_t *)mask, windows, heads,
                          s.out, s.rows, s.cols, &s.p, st);
    });
}

template <bool FROM_I8>
PyObject *gelu(PyObject *const *a, Py_ssize_t n_args)
{
    void *in, *out;
    int64_t n;
    iptq_gelu_params_t p;
    if (n_args != 4 || g.gelu_i8 == nullptr || !integer(a[2], &n) || n < 0 || !tensor(a[0], FROM_I8 ? at::kChar : at::kInt, n, &in) ||
        !tensor(a[1], at::kChar, n, &out) || !structure(a[3], g.gelu_params, &p))
        return nullptr;
    return enqueue([&](void *s) {
        return FROM_I8 ? g.gelu_i8((const int8_t *)in, (int8_t *)out, n, &p, s)
                       : g.gelu_i32((const int32_t *)in, (int8_t *)out, n, &p, s);
    });
}

// (n - 1) stride + size, or -1
int64_t extent(int32_t n, int64_t stride, int64_t size)
{
    int64_t e = 0;
    return stride < 0 || size < 0 || __builtin_mul_overflow((int64_t)(n - 1), stride, &e) || __builtin_add_overflow(e, size, &e) ? -1 : e;
}

PyObject *softmax_layers(PyObject *const *a, Py_ssize_t n_args)
{
    void *in, *out;
    int64_t in_stride, out_stride, rows;
    int32_t cols, n;
    std::vector<iptq_softmax_params_t> p;
    if (n_args != 8 || g.softmax_layers == nullptr || !integer(a[1], &in_stride) || !integer(a[3], &out_stride) ||
        !integer(a[4], &rows) || !integer(a[5], &cols) || !integer(a[6], &n) || !structures(a[7], g.softmax_params, n, &p))
        return nullptr;
    const int64_t size = elements(rows, cols);
    const int64_t read = extent(n, in_stride, size), written = extent(n, out_stride, size);
    if (size < 0 || read < 0 || written < 0 || !tensor(a[0], at::kInt, read, &in) ||
        !tensor(a[2], byte_type(p[0].out_is_signed), written, &out))
        return nullptr;
    return enqueue([&](void *s) {
        return g.softmax_layers((const int32_t *)in, in_stride, out, out_stride, rows, cols, n, p.data(), s);
    });
}

PyObject *gelu_layers(PyObject *const *a, Py_ssize_t n_args)
{
    void *in, *out;
    int64_t in_stride, out_stride, size;
    int32_t n;
    std::vector<iptq_gelu_params_t> p;
    if (n_args != 7 || g.gelu_layers == nullptr || !integer(a[1], &in_stride) || !integer(a[3], &out_stride) ||
        !integer(a[4], &size) || !integer(a[5], &n) || !structures(a[6], g.gelu_params, n, &p))
        return nullptr;
    const int64_t read = extent(n, in_stride, size), written = extent(n, out_stride, size);
    if (read < 0 || written < 0 || !tensor(a[0], at::kChar, read, &in) || !tensor(a[2], at::kChar, written, &out)) return nullptr;
    return enqueue([&](void *s) { return g.gelu_layers((const int8_t *)in, in_stride, (int8_t *)out, out_stride, size, n, p.data(), s); });
}

// bind(addresses of the eight entry points in the order of Bound, SoftmaxParams, GeluParams, Dyadic)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    if (n_args != 11) {
        PyErr_SetString(PyExc_TypeError, "bind takes eight addresses and three classes");
        return nullptr;
    }
    void *at[8];
    for (int i = 0; i < 8; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i]);
        if (at[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: an entry point is missing");
            return nullptr;
        }
    }
    for (int i = 8; i < 11; ++i)
        if (!PyType_Check(a[i])) {
            PyErr_SetString(PyExc_TypeError, "bind takes eight addresses and three classes");
            return nullptr;
        }
    g.requant = reinterpret_cast<decltype(g.requant)>(at[0]);
    g.softmax_i32 = reinterpret_cast<decltype(g.softmax_i32)>(at[1]);
    g.windowed = reinterpret_cast<decltype(g.windowed)>(at[2]);
    g.windowed_bits = reinterpret_cast<decltype(g.windowed_bits)>(at[3]);
    g.gelu_i8 = reinterpret_cast<decltype(g.gelu_i8)>(at[4]);
    g.gelu_i32 = reinterpret_cast<decltype(g.gelu_i32)>(at[5]);
    g.softmax_layers = reinterpret_cast<decltype(g.softmax_layers)>(at[6]);
    g.gelu_layers = reinterpret_cast<decltype(g.gelu_layers)>(at[7]);
    PyTypeObject **types[3] = {&g.softmax_params, &g.gelu_params, &g.dyadic};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[8 + i]);                          // kept for the life of the process, as the module is
        *types[i] = reinterpret_cast<PyTypeObject *>(a[8 + i]);
    }
    Py_RETURN_NONE;
}

#define IPTQ_METHOD(NAME, FN) {NAME, (PyCFunction)(void (*)(void))(FN), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    IPTQ_METHOD("bind", bind),
    IPTQ_METHOD("requant", guarded<requant>),
    IPTQ_METHOD("softmax_i32", guarded<softmax_i32>),
    IPTQ_METHOD("softmax_i32_windowed", guarded<windowed<false>>),
    IPTQ_METHOD("softmax_i32_windowed_bits", guarded<windowed<true>>),
    IPTQ_METHOD("gelu_i8", guarded<gelu<true>>),
    IPTQ_METHOD("gelu_i32", guarded<gelu<false>>),
    IPTQ_METHOD("softmax_i32_layers", guarded<softmax_layers>),
    IPTQ_METHOD("gelu_i8_layers", guarded<gelu_layers>),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
