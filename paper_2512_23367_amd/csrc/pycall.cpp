// Argument marshalling of the calls that a program makes per layer, in native code (Python module _qlcall): what binding.py
// checks and passes on through ctypes costs 2 to 3 us of Python per call, as long as the smallest call runs on the GPU.
//
// Each function takes the arguments of the function of binding.py that it stands for, and one to ask for the stream, and returns
// the library's status -- or None, without having called the library, for whatever is not plainly in order (an argument of another
// type, a size that does not fit, a tensor that is a view of the world of its own: subclass, batched, traced,
// without storage): binding.py then goes its own way and says what is wrong.  So every check here is one that binding.py makes as
// well, and nothing is reported from here.  One token through 1536 x 1536: 6.1 us a call through ctypes, 4.0 here.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <climits>
#include <cstdint>
#include <cstring>

#include "qlinear.h"

namespace {

struct Library {
    decltype(&ql_weight_bytes) weight_bytes;
    decltype(&ql_act_kernel_bytes) act_kernel_bytes;
    decltype(&ql_w8a8_linear) w8a8_linear;
    decltype(&ql_w4a8_linear) w4a8_linear;
    decltype(&ql_w8a8_gemm) w8a8_gemm;
    decltype(&ql_w4a8_gemm) w4a8_gemm;
    decltype(&ql_quant_act_per_token) quant_act;
    decltype(&ql_quant_act_rmsnorm) quant_rmsnorm;
    decltype(&ql_quant_act_swiglu) quant_swiglu;
    decltype(&ql_quant_act_per_token_transformed) quant_transformed;
} lib;

// An argument that is not in order: the caller returns None.
struct NotPlain {};
// A Python exception on its way (a keyboard interrupt may arrive wherever Python code runs): the caller passes it on.
struct Raised {};

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw NotPlain();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || at::isTensorSubclassLike(t)) throw NotPlain();
    return t;
}

const at::Tensor &tensor(PyObject *o, at::ScalarType type)
{
    const at::Tensor &t = tensor(o);
    if (t.scalar_type() != type) throw NotPlain();
    return t;
}

int as_int(int64_t v)
{
    if (v < INT_MIN || v > INT_MAX) throw NotPlain();
    return (int)v;
}

int as_int(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw NotPlain();
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow) throw NotPlain();
    return as_int((int64_t)v);
}

float as_float(PyObject *o)
{
    if (!PyFloat_CheckExact(o)) throw NotPlain();
    return (float)PyFloat_AS_DOUBLE(o);
}

// the stream is asked for (binding.py's function) when all else is in order
void *stream_from(PyObject *ask)
{
    PyObject *o = PyObject_CallNoArgs(ask);
    if (!o) throw Raised();
    void *p = PyLong_Check(o) ? PyLong_AsVoidPtr(o) : nullptr;
    const bool failed = !PyLong_Check(o) || PyErr_Occurred();
    Py_DECREF(o);
    if (failed) throw NotPlain();   // (binding.py asks again and reports what is wrong)
    return p;
}

// any device tensor or None
template <typename T>
T *pointer(PyObject *o)
{
    return o == Py_None ? nullptr : static_cast<T *>(tensor(o).data_ptr());
}

// fp16 [rows, columns] with unit inner stride and at least one row
struct Matrix {
    void *p;
    int rows, columns;
    int64_t ld;
    explicit Matrix(PyObject *o)
    {
        const at::Tensor &t = tensor(o, at::kHalf);
        if (t.dim() != 2 || t.size(0) < 1 || t.stride(1) != 1) throw NotPlain();
        p = t.data_ptr(), rows = as_int(t.size(0)), columns = as_int(t.size(1)), ld = t.stride(0);
    }
};

struct Workspace {
    void *p = nullptr;
    size_t bytes = 0;
    explicit Workspace(PyObject *o)
    {
        if (o == Py_None) return;
        const at::Tensor &t = tensor(o);
        p = t.data_ptr(), bytes = t.nbytes();
    }
};

const void *blob(PyObject *o, int N, int K, int bits, int group)
{
    size_t need = 0;
    const at::Tensor &t = tensor(o);
    if (lib.weight_bytes(N, K, bits, group, nullptr, nullptr, &need) != QL_OK || t.nbytes() < need) throw NotPlain();
    return t.data_ptr();
}

const float *floats(PyObject *o, int64_t n)
{
    const at::Tensor &t = tensor(o, at::kFloat);
    if (t.numel() < n) throw NotPlain();
    return static_cast<const float *>(t.data_ptr());
}

const void *bias_of(PyObject *o, int N)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, at::kHalf);
    if (t.numel() < N) throw NotPlain();
    return t.data_ptr();
}

Matrix output(PyObject *o, int M, int N)
{
    const Matrix y(o);
    if (y.rows != M || y.columns != N) throw NotPlain();
    return y;
}

const int8_t *codes(PyObject *o, int M, int K)
{
    size_t need = 0;
    const at::Tensor &t = tensor(o);
    if (lib.act_kernel_bytes(M, K, &need) != QL_OK || t.nbytes() < need) throw NotPlain();
    return static_cast<const int8_t *>(t.data_ptr());
}

// The call itself, without the interpreter's lock (as ctypes makes it); None if an argument was not plain.
template <typename Prepare>
PyObject *call(Py_ssize_t given, Py_ssize_t wanted, Prepare prepare)
{
    if (given != wanted || !lib.weight_bytes) Py_RETURN_NONE;
    int status;
    try {
        auto launch = prepare();
        PyThreadState *state = PyEval_SaveThread();
        status = launch();
        PyEval_RestoreThread(state);
    } catch (const Raised &) {
        return nullptr;
    } catch (...) {   // NotPlain, or what a tensor throws when it is asked for its storage
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

using Args = PyObject *const *;

PyObject *w8a8_linear(PyObject *, Args a, Py_ssize_t n)   // x, wq_kernel, sw, bias, N, y, ws, stream
{
    return call(n, 8, [&] {
        const Matrix x(a[0]);
        const int N = as_int(a[4]);
        const void *w = blob(a[1], N, x.columns, 8, 0), *b = bias_of(a[3], N);
        const float *sw = floats(a[2], N);
        const Matrix y = output(a[5], x.rows, N);
        const Workspace ws(a[6]);
        void *st = stream_from(a[7]);
        return [=] { return lib.w8a8_linear(x.p, x.ld, x.rows, x.columns, w, sw, b, N, y.p, y.ld, ws.p, ws.bytes, st); };
    });
}

PyObject *w4a8_linear(PyObject *, Args a, Py_ssize_t n)   // x, w4_kernel, group, bias, N, y, ws, stream
{
    return call(n, 8, [&] {
        const Matrix x(a[0]);
        const int group = as_int(a[2]), N = as_int(a[4]);
        const void *w = blob(a[1], N, x.columns, 4, group), *b = bias_of(a[3], N);
        const Matrix y = output(a[5], x.rows, N);
        const Workspace ws(a[6]);
        void *st = stream_from(a[7]);
        return [=] { return lib.w4a8_linear(x.p, x.ld, x.rows, x.columns, w, group, b, N, y.p, y.ld, ws.p, ws.bytes, st); };
    });
}

PyObject *w8a8_gemm(PyObject *, Args a, Py_ssize_t n)   // xq_kernel, sx, M, K, wq_kernel, sw, bias, N, y, ws, stream
{
    return call(n, 11, [&] {
        const int M = as_int(a[2]), K = as_int(a[3]), N = as_int(a[7]);
        const int8_t *xq = codes(a[0], M, K);
        const float *sx = floats(a[1], M), *sw = floats(a[5], N);
        const void *w = blob(a[4], N, K, 8, 0), *b = bias_of(a[6], N);
        const Matrix y = output(a[8], M, N);
        const Workspace ws(a[9]);
        void *st = stream_from(a[10]);
        return [=] { return lib.w8a8_gemm(xq, sx, M, K, w, sw, b, N, y.p, y.ld, ws.p, ws.bytes, st); };
    });
}

PyObject *w4a8_gemm(PyObject *, Args a, Py_ssize_t n)   // xq_kernel, sx, M, K, w4_kernel, group, bias, N, y, ws, stream
{
    return call(n, 11, [&] {
        const int M = as_int(a[2]), K = as_int(a[3]), group = as_int(a[5]), N = as_int(a[7]);
        const int8_t *xq = codes(a[0], M, K);
        const float *sx = floats(a[1], M);
        const void *w = blob(a[4], N, K, 4, group), *b = bias_of(a[6], N);
        const Matrix y = output(a[8], M, N);
        const Workspace ws(a[9]);
        void *st = stream_from(a[10]);
        return [=] { return lib.w4a8_gemm(xq, sx, M, K, w, group, b, N, y.p, y.ld, ws.p, ws.bytes, st); };
    });
}

PyObject *quant_act(PyObject *, Args a, Py_ssize_t n)   // x, xq_rowmajor, xq_kernel, sx, stream
{
    return call(n, 5, [&] {
        const Matrix x(a[0]);
        int8_t *rm = pointer<int8_t>(a[1]), *kl = pointer<int8_t>(a[2]);
        float *sx = pointer<float>(a[3]);
        void *st = stream_from(a[4]);
        return [=] { return lib.quant_act(x.p, x.ld, x.rows, x.columns, rm, kl, sx, st); };
    });
}

PyObject *quant_rmsnorm(PyObject *, Args a, Py_ssize_t n)   // x, gamma, eps, xq_rowmajor, xq_kernel, sx, stream
{
    return call(n, 7, [&] {
        const Matrix x(a[0]);
        const void *gamma = tensor(a[1], at::kHalf).data_ptr();
        const float eps = as_float(a[2]);
        int8_t *rm = pointer<int8_t>(a[3]), *kl = pointer<int8_t>(a[4]);
        float *sx = pointer<float>(a[5]);
        void *st = stream_from(a[6]);
        return [=] { return lib.quant_rmsnorm(x.p, x.ld, x.rows, x.columns, gamma, eps, rm, kl, sx, st); };
    });
}

PyObject *quant_swiglu(PyObject *, Args a, Py_ssize_t n)   // gate_up, xq_rowmajor, xq_kernel, sx, stream
{
    return call(n, 5, [&] {
        const Matrix x(a[0]);
        if (x.columns % 2) throw NotPlain();
        int8_t *rm = pointer<int8_t>(a[1]), *kl = pointer<int8_t>(a[2]);
        float *sx = pointer<float>(a[3]);
        void *st = stream_from(a[4]);
        return [=] { return lib.quant_swiglu(x.p, x.ld, x.rows, x.columns / 2, rm, kl, sx, st); };
    });
}

PyObject *quant_transformed(PyObject *, Args a, Py_ssize_t n)   // x, inv_smooth, hadamard_block, xq_rowmajor, xq_kernel, sx, stream
{
    return call(n, 7, [&] {
        const Matrix x(a[0]);
        const float *inv = pointer<float>(a[1]);
        const int block = as_int(a[2]);
        int8_t *rm = pointer<int8_t>(a[3]), *kl = pointer<int8_t>(a[4]);
        float *sx = pointer<float>(a[5]);
        void *st = stream_from(a[6]);
        return [=] { return lib.quant_transformed(x.p, x.ld, x.rows, x.columns, inv, block, rm, kl, sx, st); };
    });
}

// bind(addresses): the entry points of the library that binding.py has loaded, in the order of struct Library
PyObject *bind(PyObject *, PyObject *addresses)
{
    constexpr Py_ssize_t COUNT = sizeof(Library) / sizeof(void *);
    if (!PyTuple_CheckExact(addresses) || PyTuple_GET_SIZE(addresses) != COUNT) {
        PyErr_SetString(PyExc_TypeError, "bind takes a tuple of addresses");
        return nullptr;
    }
    void *p[COUNT];
    for (Py_ssize_t i = 0; i < COUNT; ++i) {
        p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
        if (PyErr_Occurred()) return nullptr;
    }
    static_assert(sizeof(lib) == sizeof(p), "pointers only");
    memcpy(&lib, p, sizeof(lib));
    Py_RETURN_NONE;
}

#define QL_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {QL_METHOD(w8a8_linear), QL_METHOD(w4a8_linear), QL_METHOD(w8a8_gemm), QL_METHOD(w4a8_gemm), QL_METHOD(quant_act),
                         QL_METHOD(quant_rmsnorm), QL_METHOD(quant_swiglu), QL_METHOD(quant_transformed),
                         {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qlcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qlcall() { return PyModule_Create(&module); }
