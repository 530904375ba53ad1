// Argument marshalling of binding.py in native code.
//
// Small layers wait for the host: checking a call's three to seven tensors, asking PyTorch for the
// current stream and passing a dozen arguments through ctypes took 5 of the 7.5 us of a call.  Each
// function here takes the arguments of the binding function of the same name in its order and
// either calls the library and returns the status, or returns None, having done nothing, where an
// argument is not of the plain form that it knows: then the binding takes its general path, which
// converts the argument or refuses it.  Plain are: device tensors of the right dtype, contiguous, of
// type torch.Tensor or Parameter and not wrapped by a transform; int, float and bool objects;
// None or an int address where the general path takes one; a dsq_conv_desc.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/hip/HIPStream.h>

#include <limits.h>
#include <string.h>

#include "../../include/dsqconv.h"

namespace {

decltype(&dsq_quantize_act) f_quantize_act;
decltype(&dsq_conv2d) f_conv2d;
decltype(&dsq_conv2d_requant) f_conv2d_requant;
decltype(&dsq_conv2d_wq) f_conv2d_wq;
decltype(&dsq_soft_quantize_fwd) f_soft_fwd;
decltype(&dsq_soft_quantize_bwd) f_soft_bwd;
PyTypeObject *desc_type;

// Reads arguments one after the other; `plain` turns false at the first that is not.
struct Args {
    PyObject *const *at;
    bool plain;

    Args(PyObject *const *args, Py_ssize_t given, Py_ssize_t expected)
        : at(args), plain(given == expected && f_quantize_act && !at::impl::torch_function_mode_enabled())
    {
    }
    long long number()
    {
        PyObject *o = *at++;
        if (!plain || !(PyLong_CheckExact(o) || PyBool_Check(o))) { plain = false; return 0; }
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow || v < INT_MIN || v > INT_MAX) plain = false;
        return v;
    }
    int integer() { return (int)number(); }
    float real()
    {
        PyObject *o = *at;
        if (plain && PyFloat_CheckExact(o)) { ++at; return (float)PyFloat_AS_DOUBLE(o); }
        return (float)number();
    }
    int truth()
    {
        PyObject *o = *at++;
        if (o != Py_True && o != Py_False) plain = false;
        return o == Py_True;
    }
    void *tensor(at::ScalarType type, bool may_be_none = false, size_t *numel = nullptr)
    {
        PyObject *o = *at++;
        if (!plain) return nullptr;
        if (may_be_none && o == Py_None) return nullptr;
        if (numel == nullptr && PyLong_CheckExact(o)) {                       // a raw device address
            void *p = PyLong_AsVoidPtr(o);
            if (PyErr_Occurred()) { PyErr_Clear(); plain = false; }
            return p;
        }
        plain = false;
        if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || at::isTensorSubclassLike(t) || !t.has_storage() || !t.is_cuda() || t.scalar_type() != type ||
            !t.is_contiguous())
            return nullptr;
        plain = true;
        if (numel) *numel = (size_t)t.numel();
        return t.data_ptr();
    }
    const dsq_conv_desc *desc(dsq_conv_desc &d)
    {
        PyObject *o = *at++;
        Py_buffer view;
        if (!plain || Py_TYPE(o) != desc_type || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            plain = false;
            return nullptr;
        }
        if (view.len == (Py_ssize_t)sizeof d) memcpy(&d, view.buf, sizeof d);
        else plain = false;
        PyBuffer_Release(&view);
        return &d;
    }
    void *stream()
    {
        PyObject *o = *at++;
        if (!plain) return nullptr;
        if (o == Py_None) return (void *)c10::hip::getCurrentHIPStream().stream();
        if (!PyLong_CheckExact(o)) { plain = false; return nullptr; }
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) { PyErr_Clear(); plain = false; }
        return p;
    }
};

// (a C++ exception, from a tensor without memory of its own for instance, is left to the general path)
template <class F>
PyObject *guarded(F body)
{
    try {
        return body();
    } catch (...) {
        Py_RETURN_NONE;
    }
}

template <class F>
PyObject *call(const Args &a, F f)
{
    if (!a.plain) Py_RETURN_NONE;
    dsq_status status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)status);
}

PyObject *quantize_act(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 12);
        if (!a.plain) Py_RETURN_NONE;
        const float *x = (const float *)a.tensor(at::kFloat);
        const dsq_layout layout = (dsq_layout)a.integer();
        const int N = a.integer(), C = a.integer(), H = a.integer(), W = a.integer();
        const float l = a.real(), u = a.real();
        const int bits = a.integer();
        size_t bytes = 0;
        void *codes = a.tensor(at::kByte, false, &bytes);
        int32_t *sums = (int32_t *)a.tensor(at::kInt);
        void *stream = a.stream();
        return call(a, [=] { return f_quantize_act(x, layout, N, C, H, W, l, u, bits, codes, bytes, sums, stream); });
    });
}

PyObject *conv2d(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 11);
        if (!a.plain) Py_RETURN_NONE;
        dsq_conv_desc d;
        a.desc(d);
        const void *act = a.tensor(at::kByte);
        const int32_t *sums = (const int32_t *)a.tensor(at::kInt);
        const float l = a.real(), u = a.real();
        const void *w = a.tensor(at::kByte), *aux = a.tensor(at::kByte);
        float *out = (float *)a.tensor(at::kFloat);
        const dsq_layout layout = (dsq_layout)a.integer();
        int32_t *acc = (int32_t *)a.tensor(at::kInt, true);
        void *stream = a.stream();
        return call(a, [=, &d] { return f_conv2d(&d, act, sums, l, u, w, aux, out, layout, acc, stream); });
    });
}

PyObject *conv2d_requant(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 16);
        if (!a.plain) Py_RETURN_NONE;
        dsq_conv_desc d;
        a.desc(d);
        const void *act = a.tensor(at::kByte);
        const int32_t *sums = (const int32_t *)a.tensor(at::kInt);
        const float l = a.real(), u = a.real();
        const void *w = a.tensor(at::kByte), *aux = a.tensor(at::kByte);
        const float *scale = (const float *)a.tensor(at::kFloat, true), *shift = (const float *)a.tensor(at::kFloat, true);
        const int relu = a.truth();
        const float l_next = a.real(), u_next = a.real();
        const int bits_next = a.integer();
        size_t bytes = 0;
        void *codes = a.tensor(at::kByte, false, &bytes);
        int32_t *sums_next = (int32_t *)a.tensor(at::kInt);
        void *stream = a.stream();
        return call(a, [=, &d] {
            return f_conv2d_requant(&d, act, sums, l, u, w, aux, scale, shift, relu, l_next, u_next, bits_next, codes, bytes,
                                    sums_next, stream);
        });
    });
}

PyObject *conv2d_wq(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 8);
        if (!a.plain) Py_RETURN_NONE;
        dsq_conv_desc d;
        a.desc(d);
        const float *x = (const float *)a.tensor(at::kFloat);
        const dsq_layout x_layout = (dsq_layout)a.integer();
        const void *w = a.tensor(at::kByte), *aux = a.tensor(at::kByte);
        float *out = (float *)a.tensor(at::kFloat);
        const dsq_layout out_layout = (dsq_layout)a.integer();
        void *stream = a.stream();
        return call(a, [=, &d] { return f_conv2d_wq(&d, x, x_layout, w, aux, out, out_layout, stream); });
    });
}

PyObject *soft_quantize_fwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 7);
        if (!a.plain) Py_RETURN_NONE;
        size_t count = 0;
        const float *x = (const float *)a.tensor(at::kFloat, false, &count);
        const float l = a.real(), u = a.real(), alpha = a.real();
        const int bits = a.integer();
        float *y = (float *)a.tensor(at::kFloat);
        void *stream = a.stream();
        return call(a, [=] { return f_soft_fwd(x, count, l, u, alpha, bits, y, stream); });
    });
}

PyObject *soft_quantize_bwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&] {
        Args a(args, n, 9);
        if (!a.plain) Py_RETURN_NONE;
        size_t count = 0;
        const float *x = (const float *)a.tensor(at::kFloat, false, &count);
        const float *gy = (const float *)a.tensor(at::kFloat);
        const float l = a.real(), u = a.real(), alpha = a.real();
        const int bits = a.integer();
        float *gx = (float *)a.tensor(at::kFloat);
        double *sums = (double *)a.tensor(at::kDouble);
        void *stream = a.stream();
        return call(a, [=] { return f_soft_bwd(x, gy, count, l, u, alpha, bits, gx, sums, stream); });
    });
}

// init(desc_type, addresses of the six entry points, in the order below)
PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 7 || !PyType_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "init(desc_type, six addresses)");
        return nullptr;
    }
    void *p[6];
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(args[1 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(args[0]);
    Py_XDECREF((PyObject *)desc_type);
    desc_type = (PyTypeObject *)args[0];
    f_conv2d = (decltype(f_conv2d))p[1];
    f_conv2d_requant = (decltype(f_conv2d_requant))p[2];
    f_conv2d_wq = (decltype(f_conv2d_wq))p[3];
    f_soft_fwd = (decltype(f_soft_fwd))p[4];
    f_soft_bwd = (decltype(f_soft_bwd))p[5];
    f_quantize_act = (decltype(f_quantize_act))p[0];
    Py_RETURN_NONE;
}

#define METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(init), METHOD(quantize_act), METHOD(conv2d), METHOD(conv2d_requant), METHOD(conv2d_wq),
                         METHOD(soft_quantize_fwd), METHOD(soft_quantize_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module_def); }
