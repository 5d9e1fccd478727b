// The linear calls of binding.py in one native step: checks on the tensors, the output, the current stream and the library
// call.  One token through a 512 -> 512 linear, called eagerly, is bound by the host: in Python the same steps took 3.4 us beside
// the 3.3 of the call itself (the output alone 1.7, the checks of rows and strides 0.5, the stream's handle 0.4).
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "paro.h"

namespace {

// The ctypes classes of the two structures (binding.py hands them over once).
PyObject *g_rotation, *g_weight;

// A ctypes structure of class `type` through the buffer protocol; NULL with an exception set if it is anything else.
template <class T>
const T *structure(PyObject *o, PyObject *type)
{
    if (!type || !PyObject_TypeCheck(o, (PyTypeObject *)type)) {
        PyErr_SetString(PyExc_TypeError, "not the structure that this call takes");
        return nullptr;
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return nullptr;
    const void *p = view.buf;
    PyBuffer_Release(&view);                          // the caller's reference keeps the structure
    return (const T *)p;
}

PyObject *types(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 2 || !PyType_Check(a[0]) || !PyType_Check(a[1])) { PyErr_SetString(PyExc_TypeError, "types takes two classes"); return nullptr; }
    Py_INCREF(a[0]); Py_INCREF(a[1]);
    Py_XDECREF(g_rotation); Py_XDECREF(g_weight);
    g_rotation = a[0]; g_weight = a[1];
    Py_RETURN_NONE;
}

const at::Tensor *tensor(PyObject *o)
{
    if (THPVariable_Check(o)) return &THPVariable_Unpack(o);
    PyErr_SetString(PyExc_TypeError, "expected a tensor");
    return nullptr;
}

// fp16 rows; false with an exception set for anything else
bool rows(const at::Tensor &t)
{
    if (t.scalar_type() == at::kHalf && t.dim() == 2 && t.stride(1) == 1) return true;
    PyErr_SetString(PyExc_AssertionError, "expected a 2-D float16 tensor with contiguous rows");
    return false;
}

// X, Y or None -> the output; undefined with an exception set on failure
at::Tensor output(const at::Tensor &x, PyObject *y, int64_t width)
{
    if (y == Py_None) return at::empty({x.size(0), width}, x.options().requires_grad(false));
    const at::Tensor *t = tensor(y);
    return t && rows(*t) ? *t : at::Tensor();
}

// The result: the output, or the status of a call that was refused.
PyObject *result(paro_status st, PyObject *y, at::Tensor &&out)
{
    if (st != PARO_OK) return PyLong_FromLong(st);
    if (y != Py_None) { Py_INCREF(y); return y; }
    return THPVariable_Wrap(std::move(out));
}

// linear(rotation or None, weight, c_out, X, Y or None, workspace or None, bytes)
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "linear takes 7 arguments"); return nullptr; }
    const paro_rotation *rot = a[0] == Py_None ? nullptr : structure<paro_rotation>(a[0], g_rotation);
    if (!rot && a[0] != Py_None) return nullptr;
    const paro_w4_weight *w = structure<paro_w4_weight>(a[1], g_weight);
    if (!w) return nullptr;
    const int64_t c_out = PyLong_AsLongLong(a[2]);
    const at::Tensor *x = tensor(a[3]);
    if (!x || !rows(*x)) return nullptr;
    const at::Tensor *ws = a[5] == Py_None ? nullptr : tensor(a[5]);
    if (!ws && a[5] != Py_None) return nullptr;
    const size_t bytes = PyLong_AsSize_t(a[6]);
    if (PyErr_Occurred()) return nullptr;
    at::Tensor out = output(*x, a[4], c_out);
    if (!out.defined()) return nullptr;
    const paro_half_t *xp = (const paro_half_t *)x->data_ptr();
    paro_half_t *yp = (paro_half_t *)out.data_ptr();
    void *wp = ws ? ws->data_ptr() : nullptr, *stream = (void *)c10::hip::getCurrentHIPStream().stream();
    const int64_t ldx = x->stride(0), ldy = out.stride(0);
    const int32_t T = (int32_t)x->size(0);
    paro_status st;
    Py_BEGIN_ALLOW_THREADS
    st = rot ? paro_rotated_linear(rot, w, xp, ldx, yp, ldy, T, wp, bytes, stream) : paro_w4a16_linear(w, xp, ldx, yp, ldy, T, wp, bytes, stream);
    Py_END_ALLOW_THREADS
    return result(st, a[4], std::move(out));
    END_HANDLE_TH_ERRORS
}

// rotate(rotation, c_in, X, Xr or None)
PyObject *rotate(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4) { PyErr_SetString(PyExc_TypeError, "rotate takes 4 arguments"); return nullptr; }
    const paro_rotation *rot = structure<paro_rotation>(a[0], g_rotation);
    if (!rot) return nullptr;
    const int64_t c_in = PyLong_AsLongLong(a[1]);
    const at::Tensor *x = tensor(a[2]);
    if (!x || !rows(*x) || PyErr_Occurred()) return nullptr;
    at::Tensor out = output(*x, a[3], c_in);
    if (!out.defined()) return nullptr;
    const paro_half_t *xp = (const paro_half_t *)x->data_ptr();
    paro_half_t *yp = (paro_half_t *)out.data_ptr();
    void *stream = (void *)c10::hip::getCurrentHIPStream().stream();
    const int64_t ldx = x->stride(0), ldy = out.stride(0);
    const int32_t T = (int32_t)x->size(0);
    paro_status st;
    Py_BEGIN_ALLOW_THREADS
    st = paro_rotate_scale(rot, xp, ldx, yp, ldy, T, stream);
    Py_END_ALLOW_THREADS
    return result(st, a[3], std::move(out));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"types", (PyCFunction)(void (*)(void))types, METH_FASTCALL, nullptr},
    {"linear", (PyCFunction)(void (*)(void))linear, METH_FASTCALL, nullptr},
    {"rotate", (PyCFunction)(void (*)(void))rotate, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "paro_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_paro_host(void) { return PyModule_Create(&module); }
