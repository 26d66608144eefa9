// Python entry points of the compute calls: argument marshalling from Python objects to the C ABI without ctypes.
//
// The smallest calls are bound by it: a kernel of 4 us behind 7 us of host time, most of it ctypes converting ten arguments,
// a Python frame for every address, and torch.cuda.current_stream().  Functions of the library are called through
// addresses that binding.py hands over (bind), so that it alone chooses the library.
// lora_delta of 64 tokens, 256 -> 256, fp32, one call among others: 7.3 us of host time by ctypes, 3.5 here (0.5 without the launch).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <pthread.h>

#include <cstddef>
#include <cstdint>

#include "../../include/lora_abi.h"

namespace {

struct library {
    decltype(&lora_plan_upload) plan_upload;
    decltype(&lora_shrink) shrink;
    decltype(&lora_expand) expand;
    decltype(&lora_delta) delta;
    decltype(&lora_delta_static) delta_static;
    decltype(&lora_base_gemm) base_gemm;
    decltype(&lora_fused_forward) fused_forward;
    decltype(&lora_merge) merge;
} lib;

PyObject* check = nullptr;                 // check(status, name) raises
PyObject* first_stream = nullptr;          // torch.cuda.current_stream() by itself: initialises torch's side
PyObject *get_device = nullptr, *get_stream = nullptr;
bool torch_ready = false;                  // first_stream has returned once in this process
PyObject *s_h = nullptr, *s_data_ptr = nullptr, *s_cuda_stream = nullptr;

void forked() { torch_ready = false; }     // (a child has to be refused by torch's own check)

// device or host address: None, an int, or what has data_ptr()
bool address(PyObject* o, void** out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    PyObject* n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (n && !PyLong_Check(n)) {
        PyObject* i = PyNumber_Long(n);
        Py_DECREF(n);
        n = i;
    }
    if (!n) return false;
    *out = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(n));
    Py_DECREF(n);
    return !PyErr_Occurred();
}

bool integer(PyObject* o, int64_t* out)
{
    PyObject* n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyNumber_Long(o);
    if (!n) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}

bool real(PyObject* o, float* out)
{
    PyObject* f = PyFloat_Check(o) ? (Py_INCREF(o), o) : PyNumber_Float(o);
    if (!f) return false;
    *out = (float)PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return true;
}

bool handle(PyObject* plan, lora_plan** out)
{
    PyObject* h = PyObject_GetAttr(plan, s_h);
    if (!h) return false;
    void* p = nullptr;
    const bool ok = address(h, &p);
    Py_DECREF(h);
    *out = static_cast<lora_plan*>(p);
    return ok;
}

// a stream object, its handle, or None: torch's current stream of the current device
bool stream_of(PyObject* o, void** out)
{
    if (o && o != Py_None) {
        if (PyLong_Check(o)) return address(o, out);
        PyObject* h = PyObject_GetAttr(o, s_cuda_stream);
        if (!h) return false;
        const bool ok = address(h, out);
        Py_DECREF(h);
        return ok;
    }
    PyObject* h = nullptr;
    if (!torch_ready) {
        h = PyObject_CallNoArgs(first_stream);               // (a pair of functions beside the handle)
        if (!h) return false;
        PyObject *n, *device, *stream;
        if (!PyArg_ParseTuple(h, "OOO", &n, &device, &stream)) {
            Py_DECREF(h);
            return false;
        }
        Py_INCREF(device);
        Py_INCREF(stream);
        Py_XSETREF(get_device, device);
        Py_XSETREF(get_stream, stream);
        torch_ready = true;
        const bool ok = address(n, out);
        Py_DECREF(h);
        return ok;
    }
    PyObject* device = PyObject_CallNoArgs(get_device);
    if (!device) return false;
    h = PyObject_CallOneArg(get_stream, device);
    Py_DECREF(device);
    if (!h) return false;
    const bool ok = address(h, out);
    Py_DECREF(h);
    return ok;
}

// arguments by position and name; those from `required` on may be missing (null)
bool arguments(const char* function, const char* const* names, int count, int required, PyObject* const* args, Py_ssize_t nargs,
               PyObject* kwnames, PyObject** out)
{
    if (nargs > count) {
        PyErr_Format(PyExc_TypeError, "%s() takes %d arguments but %zd were given", function, count, nargs);
        return false;
    }
    uint32_t given = (1u << nargs) - 1;
    for (Py_ssize_t i = 0; i < nargs; ++i) out[i] = args[i];
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t q = 0; q < nkw; ++q) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, q);
        int i = 0;
        while (i < count && PyUnicode_CompareWithASCIIString(name, names[i]) != 0) ++i;
        if (i == count || (given >> i & 1)) {
            PyErr_Format(PyExc_TypeError, i == count ? "%s() got an unexpected keyword argument '%U'" : "%s() got multiple values for argument '%U'",
                         function, name);
            return false;
        }
        out[i] = args[nargs + q];
        given |= 1u << i;
    }
    for (int i = 0; i < required; ++i)
        if (!(given >> i & 1)) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", function, names[i]);
            return false;
        }
    return true;
}

PyObject* result(lora_status status, const char* function)
{
    if (status == LORA_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(check, "is", (int)status, function);
}

#define ARGS(REQUIRED, ...)                                                                                                     \
    static const char* const names[] = {__VA_ARGS__};                                                                          \
    constexpr int count = sizeof(names) / sizeof(names[0]);                                                                    \
    PyObject* a[count];                                                                                                        \
    for (PyObject*& o : a) o = nullptr;                                                                                        \
    if (!arguments(__func__, names, count, REQUIRED, args, nargs, kwnames, a)) return nullptr;
#define SIGNATURE(NAME) PyObject* NAME(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
#define CALL(EXPRESSION)                                                                                                        \
    lora_status status;                                                                                                        \
    Py_BEGIN_ALLOW_THREADS                                                                                                     \
    status = lib.EXPRESSION;                                                                                                   \
    Py_END_ALLOW_THREADS                                                                                                       \
    return result(status, __func__);

const void* const* table(void* p) { return static_cast<const void* const*>(p); }

SIGNATURE(lora_plan_upload)
{
    ARGS(1, "plan", "stream")
    lora_plan* plan;
    void* stream;
    if (!handle(a[0], &plan) || !stream_of(a[1], &stream)) return nullptr;
    CALL(plan_upload(plan, stream))
}

SIGNATURE(lora_shrink)
{
    ARGS(5, "plan", "x", "ldx", "d_At_ptrs", "v", "stream")
    lora_plan* plan;
    void *x, *At, *v, *stream;
    int64_t ldx;
    if (!handle(a[0], &plan) || !address(a[1], &x) || !integer(a[2], &ldx) || !address(a[3], &At) || !address(a[4], &v) || !stream_of(a[5], &stream))
        return nullptr;
    CALL(shrink(plan, x, ldx, table(At), static_cast<float*>(v), stream))
}

SIGNATURE(lora_expand)
{
    ARGS(5, "plan", "v", "d_Bt_ptrs", "y", "ldy", "beta", "stream")
    lora_plan* plan;
    void *v, *Bt, *y, *stream;
    int64_t ldy;
    float beta = 1.f;
    if (!handle(a[0], &plan) || !address(a[1], &v) || !address(a[2], &Bt) || !address(a[3], &y) || !integer(a[4], &ldy) ||
        (a[5] && !real(a[5], &beta)) || !stream_of(a[6], &stream))
        return nullptr;
    CALL(expand(plan, static_cast<const float*>(v), table(Bt), y, ldy, beta, stream))
}

SIGNATURE(lora_delta)
{
    ARGS(8, "plan", "x", "ldx", "d_At_ptrs", "d_Bt_ptrs", "v", "y", "ldy", "beta", "stream")
    lora_plan* plan;
    void *x, *At, *Bt, *v, *y, *stream;
    int64_t ldx, ldy;
    float beta = 1.f;
    if (!handle(a[0], &plan) || !address(a[1], &x) || !integer(a[2], &ldx) || !address(a[3], &At) || !address(a[4], &Bt) || !address(a[5], &v) ||
        !address(a[6], &y) || !integer(a[7], &ldy) || (a[8] && !real(a[8], &beta)) || !stream_of(a[9], &stream))
        return nullptr;
    CALL(delta(plan, x, ldx, table(At), table(Bt), static_cast<float*>(v), y, ldy, beta, stream))
}

SIGNATURE(lora_delta_static)
{
    ARGS(7, "plan", "x", "ldx", "d_At_ptrs", "d_Bt_ptrs", "y", "ldy", "beta", "stream")
    lora_plan* plan;
    void *x, *At, *Bt, *y, *stream;
    int64_t ldx, ldy;
    float beta = 1.f;
    if (!handle(a[0], &plan) || !address(a[1], &x) || !integer(a[2], &ldx) || !address(a[3], &At) || !address(a[4], &Bt) || !address(a[5], &y) ||
        !integer(a[6], &ldy) || (a[7] && !real(a[7], &beta)) || !stream_of(a[8], &stream))
        return nullptr;
    CALL(delta_static(plan, x, ldx, table(At), table(Bt), y, ldy, beta, stream))
}

SIGNATURE(lora_base_gemm)
{
    ARGS(10, "num_tokens", "k", "n", "dtype", "x", "ldx", "Wt", "ldw", "y", "ldy", "stream")
    int64_t num_tokens, k, n, dtype, ldx, ldw, ldy;
    void *x, *Wt, *y, *stream;
    if (!integer(a[0], &num_tokens) || !integer(a[1], &k) || !integer(a[2], &n) || !integer(a[3], &dtype) || !address(a[4], &x) ||
        !integer(a[5], &ldx) || !address(a[6], &Wt) || !integer(a[7], &ldw) || !address(a[8], &y) || !integer(a[9], &ldy) || !stream_of(a[10], &stream))
        return nullptr;
    CALL(base_gemm((int32_t)num_tokens, (int32_t)k, (int32_t)n, (int32_t)dtype, x, ldx, Wt, ldw, y, ldy, stream))
}

SIGNATURE(lora_merge)
{
    ARGS(10, "num_layers", "n", "k", "rank", "scale", "dtype", "d_Wt_ptrs", "ldw", "d_At_ptrs", "d_Bt_ptrs", "variant", "stream")
    int64_t num_layers, n, k, rank, dtype, ldw, variant = LORA_VARIANT_AUTO;
    float scale;
    void *Wt, *At, *Bt, *stream;
    if (!integer(a[0], &num_layers) || !integer(a[1], &n) || !integer(a[2], &k) || !integer(a[3], &rank) || !real(a[4], &scale) ||
        !integer(a[5], &dtype) || !address(a[6], &Wt) || !integer(a[7], &ldw) || !address(a[8], &At) || !address(a[9], &Bt) ||
        (a[10] && !integer(a[10], &variant)) || !stream_of(a[11], &stream))
        return nullptr;
    CALL(merge((int32_t)num_layers, (int32_t)n, (int32_t)k, (int32_t)rank, scale, (int32_t)dtype, (int32_t)variant, static_cast<void* const*>(Wt), ldw,
               table(At), table(Bt), stream))
}

SIGNATURE(lora_fused_forward)
{
    ARGS(11, "plan", "x", "ldx", "Wt", "ldw", "d_At_ptrs", "d_Bt_ptrs", "y", "ldy", "workspace", "workspace_bytes", "stream")
    lora_plan* plan;
    void *x, *Wt, *At, *Bt, *y, *workspace, *stream;
    int64_t ldx, ldw, ldy, bytes;
    if (!handle(a[0], &plan) || !address(a[1], &x) || !integer(a[2], &ldx) || !address(a[3], &Wt) || !integer(a[4], &ldw) || !address(a[5], &At) ||
        !address(a[6], &Bt) || !address(a[7], &y) || !integer(a[8], &ldy) || !address(a[9], &workspace) || !integer(a[10], &bytes) ||
        !stream_of(a[11], &stream))
        return nullptr;
    CALL(fused_forward(plan, x, ldx, Wt, ldw, table(At), table(Bt), y, ldy, workspace, (size_t)bytes, stream))
}

// bind(check, first_stream, addresses of the library's functions in the order of `library`)
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *c, *f;
    unsigned long long p[8];
    if (!PyArg_ParseTuple(args, "OOKKKKKKKK", &c, &f, &p[0], &p[1], &p[2], &p[3], &p[4], &p[5], &p[6], &p[7])) return nullptr;
    Py_INCREF(c);
    Py_INCREF(f);
    Py_XSETREF(check, c);
    Py_XSETREF(first_stream, f);
    torch_ready = false;
    lib = library{reinterpret_cast<decltype(library::plan_upload)>(p[0]),   reinterpret_cast<decltype(library::shrink)>(p[1]),
                  reinterpret_cast<decltype(library::expand)>(p[2]),        reinterpret_cast<decltype(library::delta)>(p[3]),
                  reinterpret_cast<decltype(library::delta_static)>(p[4]),  reinterpret_cast<decltype(library::base_gemm)>(p[5]),
                  reinterpret_cast<decltype(library::fused_forward)>(p[6]), reinterpret_cast<decltype(library::merge)>(p[7])};
    Py_RETURN_NONE;
}

#define METHOD(NAME, SIGNATURE_)                                                                                                \
    {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL | METH_KEYWORDS, #NAME SIGNATURE_ "\n--\n\n"}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    METHOD(lora_plan_upload, "(plan, stream=None)"),
    METHOD(lora_shrink, "(plan, x, ldx, d_At_ptrs, v, stream=None)"),
    METHOD(lora_expand, "(plan, v, d_Bt_ptrs, y, ldy, beta=1.0, stream=None)"),
    METHOD(lora_delta, "(plan, x, ldx, d_At_ptrs, d_Bt_ptrs, v, y, ldy, beta=1.0, stream=None)"),
    METHOD(lora_delta_static, "(plan, x, ldx, d_At_ptrs, d_Bt_ptrs, y, ldy, beta=1.0, stream=None)"),
    METHOD(lora_base_gemm, "(num_tokens, k, n, dtype, x, ldx, Wt, ldw, y, ldy, stream=None)"),
    METHOD(lora_merge, "(num_layers, n, k, rank, scale, dtype, d_Wt_ptrs, ldw, d_At_ptrs, d_Bt_ptrs, variant=0, stream=None)"),
    METHOD(lora_fused_forward, "(plan, x, ldx, Wt, ldw, d_At_ptrs, d_Bt_ptrs, y, ldy, workspace, workspace_bytes, stream=None)"),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls()
{
    s_h = PyUnicode_InternFromString("handle");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_h || !s_data_ptr || !s_cuda_stream || pthread_atfork(nullptr, nullptr, forked) != 0) return nullptr;
    return PyModule_Create(&module);
}
