// The hot calls of binding.py in native code: tensors to pointers, torch's current stream, the call.  A decode step of one sequence
// takes 4 us on the GPU and took 5.4 on the host, 3 of them in looking at nine tensors through their Python attributes and in ctypes.
// Through these calls one after the other take 3.6 to 4.4 us (6.0), about the rate at which launches follow each other on the GPU; a
// call that is waited for gains the same 2 us of about 18.  16 heads of fp32 attention decode 6.4 -> 4.4.
// Every function returns the library's status, or None for arguments that are anything but contiguous GPU tensors and plain
// numbers: the caller then goes the general way, which says what is wrong with them.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "dsla.h"

namespace {

PyObject *g_device, *g_raw_stream, *g_parameter, *g_desc;   // torch._C._cuda_getDevice, _cuda_getCurrentRawStream; torch.nn.Parameter, binding.DslaDesc
struct Entries {
    decltype(&dsla_decode) decode;
    decltype(&dsla_decode_slots) decode_slots;
    decltype(&dsla_prefill) prefill;
    decltype(&dsla_prefill_varlen) prefill_varlen;
    decltype(&dsla_attention_decode) attention_decode;
    decltype(&dsla_attention_prefill) attention_prefill;
    decltype(&dsla_project) project;
} g_entry;

// A tensor whose memory can be handed over; other subclasses answer for themselves in Python.
const at::Tensor *gpu_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o) && reinterpret_cast<PyObject *>(Py_TYPE(o)) != g_parameter) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

struct Args {
    PyObject *const *o;
    bool ok = true;
    explicit Args(PyObject *const *args) : o(args) {}
    void *pointer(int i, bool optional = false)
    {
        if (optional && o[i] == Py_None) return nullptr;
        const at::Tensor *t = gpu_tensor(o[i]);
        if (!t) ok = false;
        return t ? t->data_ptr() : nullptr;
    }
    void *buffer(int i, size_t *bytes)
    {
        *bytes = 0;
        if (o[i] == Py_None) return nullptr;
        const at::Tensor *t = gpu_tensor(o[i]);
        if (!t) {
            ok = false;
            return nullptr;
        }
        *bytes = static_cast<size_t>(t->numel()) * t->element_size();
        return t->data_ptr();
    }
    dsla_desc desc(int i)   // (a copy: the caller's structure may change while the call runs without the interpreter's lock)
    {
        dsla_desc d;
        std::memset(&d, 0, sizeof(d));
        Py_buffer view;
        if (reinterpret_cast<PyObject *>(Py_TYPE(o[i])) != g_desc) {   // (bytes of that size have a buffer too)
            ok = false;
            return d;
        }
        if (PyObject_GetBuffer(o[i], &view, PyBUF_SIMPLE) != 0) {
            ok = false;
            return d;
        }
        if (view.len == static_cast<Py_ssize_t>(sizeof(d))) std::memcpy(&d, view.buf, sizeof(d));
        else ok = false;
        PyBuffer_Release(&view);
        return d;
    }
    int64_t integer(int i)
    {
        if (!PyLong_CheckExact(o[i])) {
            ok = false;
            return 0;
        }
        const int64_t x = PyLong_AsLongLong(o[i]);
        if (x == -1 && PyErr_Occurred()) ok = false;
        return x;
    }
    float real(int i)
    {
        if (!PyFloat_CheckExact(o[i])) ok = false;
        return ok ? static_cast<float>(PyFloat_AS_DOUBLE(o[i])) : 0.f;
    }
    void *stream()
    {
        if (!ok) return nullptr;
        PyObject *device = PyObject_CallNoArgs(g_device), *s = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
        Py_XDECREF(device);
        void *p = s ? PyLong_AsVoidPtr(s) : nullptr;
        Py_XDECREF(s);
        if (PyErr_Occurred()) ok = false;
        return p;
    }
};

// [B][T][H][d] of a bf16 or fp32 tensor
bool shape_of(PyObject *o, int32_t (&dims)[3], int64_t *T, int32_t *dtype)
{
    const at::Tensor *t = gpu_tensor(o);
    if (!t || t->dim() != 4) return false;
    const auto s = t->sizes();
    for (int i = 0; i < 4; ++i)
        if (s[i] > 0x7fffffff) return false;
    dims[0] = static_cast<int32_t>(s[0]);
    *T = s[1];
    dims[1] = static_cast<int32_t>(s[2]);
    dims[2] = static_cast<int32_t>(s[3]);
    if (t->scalar_type() == at::kBFloat16) *dtype = DSLA_BF16;
    else if (t->scalar_type() == at::kFloat) *dtype = DSLA_F32;
    else return false;
    return true;
}

// Runs f(args) -> status without the interpreter's lock; None where the arguments were not what it takes.
template <class F>
PyObject *guarded(PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want, F &&f)
{
    if (nargs == want) {
        try {
            Args a(args);
            const int status = f(a);
            if (a.ok) return PyLong_FromLong(status);
        } catch (const std::exception &) {
        }
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}
#define CALL(status, a, ...)                                                                                       \
    do {                                                                                                           \
        if (!(a).ok) return 0;                                                                                     \
        Py_BEGIN_ALLOW_THREADS                                                                                     \
        status = __VA_ARGS__;                                                                                      \
        Py_END_ALLOW_THREADS                                                                                       \
    } while (0)

PyObject *decode(PyObject *, PyObject *const *args, Py_ssize_t n)   // desc, q, k, v, g1, g2, S1, S2, o
{
    return guarded(args, n, 9, [](Args &a) -> int {
        const dsla_desc d = a.desc(0);
        void *p[9];
        for (int i = 1; i < 9; ++i) p[i] = a.pointer(i);
        void *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.decode(&d, p[1], p[2], p[3], p[4], p[5], static_cast<float *>(p[6]), static_cast<float *>(p[7]), p[8], s));
        return status;
    });
}

PyObject *decode_slots(PyObject *, PyObject *const *args, Py_ssize_t n)   // desc, q, k, v, g1, g2, row_index, state_slot, S1, S2, o
{
    return guarded(args, n, 11, [](Args &a) -> int {
        const dsla_desc d = a.desc(0);
        void *p[11];
        for (int i = 1; i < 11; ++i) p[i] = a.pointer(i, i == 6 || i == 7);
        void *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.decode_slots(&d, p[1], p[2], p[3], p[4], p[5], static_cast<int32_t *>(p[6]), static_cast<int32_t *>(p[7]),
                                             static_cast<float *>(p[8]), static_cast<float *>(p[9]), p[10], s));
        return status;
    });
}

PyObject *prefill(PyObject *, PyObject *const *args, Py_ssize_t n)   // desc, T, q, k, v, g1, g2, S1, S2, o, workspace
{
    return guarded(args, n, 11, [](Args &a) -> int {
        const dsla_desc d = a.desc(0);
        const int64_t T = a.integer(1);
        void *p[10];
        for (int i = 2; i < 10; ++i) p[i] = a.pointer(i);
        size_t bytes;
        void *ws = a.buffer(10, &bytes), *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.prefill(&d, T, p[2], p[3], p[4], p[5], p[6], static_cast<float *>(p[7]), static_cast<float *>(p[8]), p[9], ws, bytes, s));
        return status;
    });
}

// desc, total_T, max_T, cu_seqlens, seq_index, state_slot, q, k, v, g1, g2, S1, S2, o, workspace
PyObject *prefill_varlen(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 15, [](Args &a) -> int {
        const dsla_desc d = a.desc(0);
        const int64_t total = a.integer(1), longest = a.integer(2);
        void *p[14];
        for (int i = 3; i < 14; ++i) p[i] = a.pointer(i, i == 4 || i == 5);
        size_t bytes;
        void *ws = a.buffer(14, &bytes), *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.prefill_varlen(&d, total, longest, static_cast<int32_t *>(p[3]), static_cast<int32_t *>(p[4]), static_cast<int32_t *>(p[5]),
                                               p[6], p[7], p[8], p[9], p[10], static_cast<float *>(p[11]), static_cast<float *>(p[12]), p[13], ws, bytes, s));
        return status;
    });
}

PyObject *attention_decode(PyObject *, PyObject *const *args, Py_ssize_t n)   // q, k, v, o, scale, workspace, seq_lens
{
    return guarded(args, n, 7, [](Args &a) -> int {
        int32_t dims[3] = {}, dtype = 0;
        int64_t T = 0;
        if (!shape_of(a.o[1], dims, &T, &dtype)) a.ok = false;
        void *q = a.pointer(0), *k = a.pointer(1), *v = a.pointer(2), *o = a.pointer(3);
        const float scale = a.real(4);
        size_t bytes;
        void *ws = a.buffer(5, &bytes), *lens = a.pointer(6, true), *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.attention_decode(dims[0], dims[1], dims[2], T, dtype, scale, q, k, v, static_cast<int32_t *>(lens), o, ws, bytes, s));
        return status;
    });
}

PyObject *attention_prefill(PyObject *, PyObject *const *args, Py_ssize_t n)   // q, k, v, o, scale
{
    return guarded(args, n, 5, [](Args &a) -> int {
        int32_t dims[3] = {}, dtype = 0;
        int64_t T = 0;
        if (!shape_of(a.o[0], dims, &T, &dtype)) a.ok = false;
        void *q = a.pointer(0), *k = a.pointer(1), *v = a.pointer(2), *o = a.pointer(3);
        const float scale = a.real(4);
        void *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.attention_prefill(dims[0], dims[1], dims[2], T, dtype, scale, q, k, v, o, s));
        return status;
    });
}

PyObject *project(PyObject *, PyObject *const *args, Py_ssize_t n)   // x, W, outs, bias
{
    return guarded(args, n, 4, [](Args &a) -> int {
        constexpr int kMost = 16;
        void *po[kMost];
        const at::Tensor *x = gpu_tensor(a.o[0]), *w = gpu_tensor(a.o[1]);
        if (!x || !w || !PyList_CheckExact(a.o[2]) || x->dim() != 2 || w->dim() != 2) {
            a.ok = false;
            return 0;
        }
        const int64_t M = x->size(0), K = x->size(1), n_out = PyList_GET_SIZE(a.o[2]);
        if (n_out < 1 || n_out > kMost || w->size(0) > 0x7fffffff || K > 0x7fffffff || w->size(0) % n_out != 0 || w->size(1) != K) {
            a.ok = false;
            return 0;
        }
        const int64_t width = w->size(0) / n_out;
        for (int64_t i = 0; i < n_out; ++i) {
            const at::Tensor *t = gpu_tensor(PyList_GET_ITEM(a.o[2], i));
            if (!t || t->numel() != M * width) {
                a.ok = false;
                return 0;
            }
            po[i] = t->data_ptr();
        }
        void *px = a.pointer(0), *pw = a.pointer(1), *bias = a.pointer(3, true), *s = a.stream();
        int status = 0;
        CALL(status, a, g_entry.project(M, static_cast<int32_t>(K), static_cast<int32_t>(n_out), static_cast<int32_t>(width), px, pw,
                                        static_cast<float *>(bias), po, s));
        return status;
    });
}

// device, raw_stream, parameter type, descriptor type, addresses of the entry points in the order of Entries
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    constexpr int kEntries = sizeof(Entries) / sizeof(void *);
    constexpr int kObjects = 4;
    if (n != kObjects + kEntries) {
        PyErr_SetString(PyExc_TypeError, "bind: number of arguments");
        return nullptr;
    }
    void *p[kEntries];
    for (int i = 0; i < kEntries; ++i) {
        p[i] = PyLong_AsVoidPtr(args[kObjects + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    std::memcpy(&g_entry, p, sizeof(p));
    PyObject **to[kObjects] = {&g_device, &g_raw_stream, &g_parameter, &g_desc};
    for (int i = 0; i < kObjects; ++i) {
        Py_INCREF(args[i]);
        Py_XDECREF(*to[i]);
        *to[i] = args[i];
    }
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {METHOD(bind), METHOD(decode), METHOD(decode_slots), METHOD(prefill), METHOD(prefill_varlen), METHOD(attention_decode),
                           METHOD(attention_prefill), METHOD(project), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&g_module);
    if (m && PyModule_AddStringConstant(m, "built_for", DSLA_BUILT_FOR) != 0) Py_CLEAR(m);   // (build.py: marshal_stamp)
    return m;
}
