// The calls that a program makes once per layer, from torch tensors without a trip through ctypes:
// nvq.gemv_w4a16 and its like spend 2.8 us in Python on shapes, types and the stream (2048 x 2048 at one
// token: 6.4 us a call, of which the launch takes 3.6 and the kernel 2.7).
//
// Only the ordinary case is served here: tensors (no subclasses, which may say themselves where their
// data is) of the expected types on a device, contiguous, with fitting shapes and room for what is
// written and read.  For everything else a function returns None and the caller takes its own way, which
// names what is wrong.  The library's entry points are handed over by address (bind); a call returns their
// status.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "nvq.h"

namespace {

decltype(&nvq_gemv_w4a16) g_gemv_w4a16;
decltype(&nvq_gemv_w4a8) g_gemv_w4a8;
decltype(&nvq_quant_act_i8) g_quant_act_i8;
decltype(&nvq_gemm_w4a16) g_gemm_w4a16;

// A contiguous device tensor of that type; dims < 0: any shape.
const at::Tensor *device_tensor(PyObject *o, at::ScalarType type, int64_t dims) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) return nullptr;
    if (dims >= 0 && t.dim() != dims) return nullptr;
    return &t;
}

// The same with room for n values.
const at::Tensor *device_room(PyObject *o, at::ScalarType type, int64_t n) {
    const at::Tensor *const t = device_tensor(o, type, -1);
    return t && t->numel() >= n ? t : nullptr;
}

// The output of a product (n results), and its type for the library.
const at::Tensor *output_tensor(PyObject *o, int64_t n, int *y_dtype) {
    if (const at::Tensor *t = device_room(o, at::kFloat, n)) {
        *y_dtype = NVQ_F32;
        return t;
    }
    *y_dtype = NVQ_BF16;
    return device_room(o, at::kBFloat16, n);
}

struct Weights {
    const uint8_t *q;
    const uint16_t *s;
    int64_t N, K;
};
bool weights(PyObject *qweight, PyObject *scales, Weights *w) {
    const at::Tensor *q = device_tensor(qweight, at::kByte, 2), *s = device_tensor(scales, at::kShort, 2);
    if (!q || !s) return false;
    w->N = q->size(0);
    w->K = q->size(1) * 2;
    if (s->size(0) != w->N || s->size(1) != w->K / 32 || w->N > INT32_MAX || w->K > INT32_MAX) return false;
    w->q = static_cast<const uint8_t *>(q->data_ptr());
    w->s = static_cast<const uint16_t *>(s->data_ptr());
    return true;
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject *none() { Py_RETURN_NONE; }

template <typename CALL>
PyObject *status_of(CALL call) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// (qweight, scales, x, y)
template <bool GEMM>
PyObject *product_w4a16(PyObject *const *a, Py_ssize_t n) {
    Weights w;
    int y_dtype;
    if (n != 4 || !weights(a[0], a[1], &w)) return none();
    const at::Tensor *const x = device_tensor(a[2], at::kBFloat16, 2);
    if (!x || x->size(1) != w.K || x->size(0) > INT32_MAX) return none();
    const int64_t M = x->size(0);
    const at::Tensor *const y = output_tensor(a[3], M * w.N, &y_dtype);
    if (!y) return none();
    const uint16_t *const xp = static_cast<const uint16_t *>(x->data_ptr());
    void *const yp = y->data_ptr(), *const st = current_stream();
    if (GEMM) return status_of([&] { return g_gemm_w4a16(w.q, w.s, w.N, w.K, xp, M, yp, y_dtype, st); });
    return status_of([&] { return g_gemv_w4a16(w.q, w.s, (int)w.N, (int)w.K, xp, (int)M, yp, y_dtype, st); });
}

PyObject *gemv_w4a16(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return product_w4a16<false>(a, n);
    END_HANDLE_TH_ERRORS
}

PyObject *gemm_w4a16(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return product_w4a16<true>(a, n);
    END_HANDLE_TH_ERRORS
}

// An int that fits the library's, or false (another type, too large).
bool small_int(PyObject *o, int *v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow;
    const long l = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || l < INT32_MIN || l > INT32_MAX) return false;
    *v = (int)l;
    return true;
}

// (qweight, scales, xq, xscale, xgsum, act_group, y)
PyObject *gemv_w4a8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Weights w;
    int y_dtype, group;
    if (n != 7 || !weights(a[0], a[1], &w) || !small_int(a[5], &group)) return none();
    const at::Tensor *const xq = device_tensor(a[2], at::kChar, 2);
    if (!xq || xq->size(1) != w.K || xq->size(0) > INT32_MAX) return none();
    const int M = (int)xq->size(0);
    const int64_t groups = M * (w.K / 32);
    const at::Tensor *const xs = device_room(a[3], at::kFloat, group == 32 ? groups : M),
                     *const gs = device_room(a[4], at::kInt, M <= 3 ? groups : 0),  // (read for up to three tokens)
                     *const y = output_tensor(a[6], M * w.N, &y_dtype);
    if (!xs || !gs || !y) return none();
    const int8_t *const xp = static_cast<const int8_t *>(xq->data_ptr());
    const float *const sp = static_cast<const float *>(xs->data_ptr());
    const int32_t *const gp = static_cast<const int32_t *>(gs->data_ptr());
    void *const yp = y->data_ptr(), *const st = current_stream();
    return status_of([&] {
        return g_gemv_w4a8(w.q, w.s, (int)w.N, (int)w.K, xp, sp, gp, group, M, yp, y_dtype, nullptr, st);
    });
    END_HANDLE_TH_ERRORS
}

// (x, act_group, xq, xscale, xgsum)
PyObject *quant_act_i8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int group;
    if (n != 5 || !small_int(a[1], &group)) return none();
    const at::Tensor *x = device_tensor(a[0], at::kBFloat16, 2);
    if (!x || x->size(0) > INT32_MAX || x->size(1) > INT32_MAX) return none();
    const int64_t M = x->size(0), groups = M * (x->size(1) / 32);
    const at::Tensor *const xq = device_room(a[2], at::kChar, M * x->size(1)),
                     *const xs = device_room(a[3], at::kFloat, group == 32 ? groups : M),
                     *const gs = device_room(a[4], at::kInt, groups);
    if (!xq || !xs || !gs) return none();
    const uint16_t *const xp = static_cast<const uint16_t *>(x->data_ptr());
    int8_t *const q = static_cast<int8_t *>(xq->data_ptr());
    float *const s = static_cast<float *>(xs->data_ptr());
    int32_t *const g = static_cast<int32_t *>(gs->data_ptr());
    void *const st = current_stream();
    return status_of([&] { return g_quant_act_i8(xp, (int)x->size(0), (int)x->size(1), group, q, s, g, st); });
    END_HANDLE_TH_ERRORS
}

// The addresses of gemv_w4a16, gemv_w4a8, quant_act_i8, gemm_w4a16 in the library.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    void *p[4];
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "four addresses");
        return nullptr;
    }
    for (int i = 0; i < 4; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    g_gemv_w4a16 = reinterpret_cast<decltype(g_gemv_w4a16)>(p[0]);
    g_gemv_w4a8 = reinterpret_cast<decltype(g_gemv_w4a8)>(p[1]);
    g_quant_act_i8 = reinterpret_cast<decltype(g_quant_act_i8)>(p[2]);
    g_gemm_w4a16 = reinterpret_cast<decltype(g_gemm_w4a16)>(p[3]);
    return none();
    END_HANDLE_TH_ERRORS
}

// The handle that the calls pass (for tests).
PyObject *stream_handle(PyObject *, PyObject *) {
    HANDLE_TH_ERRORS
    return PyLong_FromVoidPtr(current_stream());
    END_HANDLE_TH_ERRORS
}

#define NVQ_FAST(name_) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name_)), METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"bind", NVQ_FAST(bind)},
                         {"gemv_w4a16", NVQ_FAST(gemv_w4a16)},
                         {"gemv_w4a8", NVQ_FAST(gemv_w4a8)},
                         {"quant_act_i8", NVQ_FAST(quant_act_i8)},
                         {"gemm_w4a16", NVQ_FAST(gemm_w4a16)},
                         {"stream_handle", stream_handle, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    PyObject *const m = PyModule_Create(&module);
    // (the caller leaves a module alone that was built for another torch)
    if (m && PyModule_AddStringConstant(m, "torch_version", NVQ_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
