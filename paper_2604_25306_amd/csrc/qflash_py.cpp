// Native half of the Python binding: turns torch tensors into the pointers and extents of the C ABI
// and calls it.  A call on a small layer takes the GPU less time than ctypes takes to marshal its
// fifteen arguments: through ctypes and Python-level tensor checks a call cost the host 9.9 us
// (DeiT-Tiny, one image), of which 3 us are the HIP launch; the checks below are a few loads each.
// The module holds no device code and no state but the two types that constants come in; every function
// returns the error code of the C ABI, raises ValueError for tensors that do not have the type or shape the
// binding promises and TypeError for constants that are not a QFlashParams or an array of them.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "qflash.h"

namespace {

// One argument as a tensor, or nullptr after setting the Python error.
const at::Tensor* tensor_arg(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch tensor", what);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

bool dense(const at::Tensor& t, at::ScalarType type) {
    return t.scalar_type() == type && t.is_cuda() && t.is_contiguous();
}

// Q, K, V (of one type) and O (int8): contiguous CUDA tensors [B,H,N,d] of one shape.
struct Layer {
    const void *q, *k, *v;
    void* o;
    int B, H, N, d, device;
};

bool layer_args(PyObject* const* t, at::ScalarType type, const char* type_name, const char* const names[3], Layer* out) {
    const at::Tensor* x[4];
    for (int i = 0; i < 4; ++i) {
        const bool is_out = i == 3;
        if (!(x[i] = tensor_arg(t[i], is_out ? "O" : names[i]))) return false;
        if (!dense(*x[i], is_out ? at::kChar : type) || x[i]->dim() != 4) {
            PyErr_Format(PyExc_ValueError, "%s must be a contiguous %s CUDA tensor [B,H,N,d]", is_out ? "O" : names[i],
                         is_out ? "int8" : type_name);
            return false;
        }
        if (i > 0 && x[i]->sizes() != x[0]->sizes()) {
            PyErr_Format(PyExc_ValueError, "%s, %s, %s, O must share one shape", names[0], names[1], names[2]);
            return false;
        }
    }
    for (int i = 0; i < 4; ++i)
        if (x[0]->size(i) > INT32_MAX) {
            PyErr_SetString(PyExc_ValueError, "tensor extent too large");
            return false;
        }
    out->q = x[0]->data_ptr(); out->k = x[1]->data_ptr(); out->v = x[2]->data_ptr(); out->o = x[3]->data_ptr();
    out->B = (int)x[0]->size(0); out->H = (int)x[0]->size(1); out->N = (int)x[0]->size(2); out->d = (int)x[0]->size(3);
    out->device = x[0]->get_device();
    return true;
}

// An int argument (anything int() takes); false after setting the Python error.
bool int_arg(PyObject* o, int* out) {
    long v;
    if (PyLong_Check(o)) {
        v = PyLong_AsLong(o);
    } else {
        PyObject* i = PyNumber_Long(o);
        if (!i) return false;
        v = PyLong_AsLong(i);
        Py_DECREF(i);
    }
    if (v == -1 && PyErr_Occurred()) return false;
    if (v < INT32_MIN || v > INT32_MAX) {
        PyErr_SetString(PyExc_ValueError, "integer argument out of range");
        return false;
    }
    *out = (int)v;
    return true;
}
bool ctx_arg(PyObject* o, qflash_ctx** out) {
    *out = nullptr;
    if (o == Py_None) return true;
    *out = (qflash_ctx*)PyLong_AsVoidPtr(o);
    return *out || !PyErr_Occurred();
}
// A raw stream handle, or None: torch's current stream on `device`.
bool stream_arg(PyObject* o, int device, void** out) {
    if (o == Py_None) {
        *out = (void*)c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
        return true;
    }
    *out = PyLong_AsVoidPtr(o);
    return *out || !PyErr_Occurred();
}

// The types constants come in, told by the binding when it loads this module (bind_types).
PyTypeObject* g_params_type = nullptr;     // QFlashParams
PyTypeObject* g_array_type = nullptr;      // ctypes.Array

// The qflash_params behind a QFlashParams or a ctypes array of them, through the buffer protocol.  The
// type is checked, not only the size: with any other count than the entry point takes, or with a buffer
// that merely is as long, the kernel would run on constants of another head or on none at all.
enum class Constants { one, array, either };
class Params {
public:
    ~Params() { if (held_) PyBuffer_Release(&buf_); }
    bool get(PyObject* o, Constants want) {
        if (!g_params_type || !g_array_type) {
            PyErr_SetString(PyExc_RuntimeError, "bind_types has not been called");
            return false;
        }
        const bool one = want != Constants::array && PyObject_TypeCheck(o, g_params_type);
        if (!one && (want == Constants::one || !is_array(o))) {
            if (!PyErr_Occurred())
                PyErr_Format(PyExc_TypeError, "params must be %s, not %.200s", want == Constants::one ? "one QFlashParams" :
                             want == Constants::array ? "an array of QFlashParams" : "one QFlashParams or an array of them",
                             Py_TYPE(o)->tp_name);
            return false;
        }
        if (PyObject_GetBuffer(o, &buf_, PyBUF_SIMPLE) != 0) return false;
        held_ = true;
        n_ = one ? 1 : (int)(buf_.len / (Py_ssize_t)sizeof(qflash_params));
        if (n_ < 1 || (!one && buf_.itemsize != (Py_ssize_t)sizeof(qflash_params)) || buf_.len < (Py_ssize_t)sizeof(qflash_params)) {
            PyErr_SetString(PyExc_ValueError, "params must hold at least one QFlashParams");
            return false;
        }
        return true;
    }
    const qflash_params* p() const { return (const qflash_params*)buf_.buf; }
    int n() const { return n_; }

private:
    // A ctypes array whose elements are QFlashParams.
    static bool is_array(PyObject* o) {
        if (!PyObject_TypeCheck(o, g_array_type)) return false;
        PyObject* t = PyObject_GetAttrString((PyObject*)Py_TYPE(o), "_type_");
        if (!t) return false;
        const bool ok = PyType_Check(t) && PyType_IsSubtype((PyTypeObject*)t, g_params_type);
        Py_DECREF(t);
        return ok;
    }
    Py_buffer buf_;
    int n_ = 0;
    bool held_ = false;
};

const char* const kInt8Names[3] = {"Q", "K", "V"};
const char* const kFloatNames[3] = {"Qf", "Kf", "Vf"};

bool count_is(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

#define QF_TRY try {
#define QF_CATCH                                         \
    }                                                    \
    catch (const std::exception& e) {                    \
        PyErr_SetString(PyExc_RuntimeError, e.what());   \
        return nullptr;                                  \
    }

enum { kPerTensor = 0, kStatic = 1, kPerHead = 2 };

// attention(entry, ctx, Q, K, V, O, params, kv_tile, bias, stream)
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    QF_TRY
    int entry, tile;
    qflash_ctx* ctx;
    Layer L;
    Params p;
    void* stream;
    if (!count_is(n, 10) || !int_arg(a[0], &entry) || !ctx_arg(a[1], &ctx) ||
        !p.get(a[6], entry == kPerHead ? Constants::array : Constants::one) ||
        !layer_args(a + 2, at::kChar, "int8", kInt8Names, &L) || !int_arg(a[7], &tile))
        return nullptr;
    if (entry == kPerHead && p.n() != L.H) {
        PyErr_SetString(PyExc_ValueError, "need one QFlashParams per head");
        return nullptr;
    }
    const int32_t* bias = nullptr;
    int bias_B = 0, bias_H = 0;
    if (a[8] != Py_None) {
        const at::Tensor* t = tensor_arg(a[8], "bias");
        if (!t) return nullptr;
        if (!dense(*t, at::kInt) || t->dim() != 4 || t->size(2) != L.N || t->size(3) != L.N || t->size(0) > INT32_MAX ||
            t->size(1) > INT32_MAX) {
            PyErr_SetString(PyExc_ValueError, "bias must be a contiguous int32 CUDA tensor [bias_B,bias_H,N,N]");
            return nullptr;
        }
        bias = (const int32_t*)t->data_ptr();
        bias_B = (int)t->size(0);
        bias_H = (int)t->size(1);
    }
    if (!stream_arg(a[9], L.device, &stream)) return nullptr;
    const auto fn = entry == kStatic ? qflash_attention_static : entry == kPerHead ? qflash_attention_per_head : qflash_attention;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(ctx, (const int8_t*)L.q, (const int8_t*)L.k, (const int8_t*)L.v, (int8_t*)L.o, bias, bias_B, bias_H, L.B, L.H,
            L.N, L.d, tile, p.p(), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    QF_CATCH
}

// attention_packed_bias(ctx, Q, K, V, O, params, kv_tile, packed, bias_B, bias_H, stream)
PyObject* attention_packed_bias(PyObject*, PyObject* const* a, Py_ssize_t n) {
    QF_TRY
    int tile, bias_B, bias_H;
    qflash_ctx* ctx;
    Layer L;
    Params p;
    void* stream;
    if (!count_is(n, 11) || !ctx_arg(a[0], &ctx) || !p.get(a[5], Constants::either) ||
        !layer_args(a + 1, at::kChar, "int8", kInt8Names, &L) || !int_arg(a[6], &tile) || !int_arg(a[8], &bias_B) || !int_arg(a[9], &bias_H))
        return nullptr;
    const at::Tensor* t = tensor_arg(a[7], "packed");
    if (!t) return nullptr;
    if (!dense(*t, at::kInt)) {
        PyErr_SetString(PyExc_ValueError, "packed must be a contiguous int32 CUDA tensor");
        return nullptr;
    }
    const int64_t nb = ((int64_t)L.N + 31) / 32;
    if ((double)t->numel() < (double)bias_B * (double)bias_H * (double)(nb * nb) * 1024.0) {
        PyErr_SetString(PyExc_ValueError, "packed is smaller than qflash_packed_bias_bytes(bias_B, bias_H, N)");
        return nullptr;
    }
    const int32_t* packed = (const int32_t*)t->data_ptr();
    if (!stream_arg(a[10], L.device, &stream)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = qflash_attention_packed_bias(ctx, (const int8_t*)L.q, (const int8_t*)L.k, (const int8_t*)L.v, (int8_t*)L.o, packed,
                                      bias_B, bias_H, L.B, L.H, L.N, L.d, tile, p.p(), p.n(), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    QF_CATCH
}

// attention_dynamic(ctx, Qf, Kf, Vf, O, kv_tile, workspace, info, out_round, stream, bias_real, excluded)
PyObject* attention_dynamic(PyObject*, PyObject* const* a, Py_ssize_t n) {
    QF_TRY
    int tile, out_round;
    qflash_ctx* ctx;
    Layer L;
    void* stream;
    if (!count_is(n, 12) || !ctx_arg(a[0], &ctx) || !layer_args(a + 1, at::kFloat, "float32", kFloatNames, &L) ||
        !int_arg(a[5], &tile) || !int_arg(a[8], &out_round))
        return nullptr;
    const at::Tensor *ws = tensor_arg(a[6], "workspace"), *info = nullptr, *bias = nullptr, *mask = nullptr;
    if (!ws) return nullptr;
    if (!dense(*ws, at::kByte)) {
        PyErr_SetString(PyExc_ValueError, "workspace must be a contiguous uint8 CUDA tensor");
        return nullptr;
    }
    if (a[7] != Py_None) {
        if (!(info = tensor_arg(a[7], "info"))) return nullptr;
        if (info->scalar_type() != at::kByte || !info->is_cuda() || info->numel() < (int64_t)sizeof(qflash_dynamic_info)) {
            PyErr_SetString(PyExc_ValueError, "info must be a uint8 CUDA tensor of sizeof(DynamicInfo) bytes");
            return nullptr;
        }
    }
    if (a[10] != Py_None) {
        if (!(bias = tensor_arg(a[10], "bias_real"))) return nullptr;
        if (!dense(*bias, at::kFloat) || bias->dim() != 4) {
            PyErr_SetString(PyExc_ValueError, "bias_real must be a contiguous float32 CUDA tensor [bias_B,bias_H,N,N]");
            return nullptr;
        }
    }
    if (a[11] != Py_None) {
        if (!(mask = tensor_arg(a[11], "excluded"))) return nullptr;
        if (!dense(*mask, at::kByte) || (bias && mask->sizes() != bias->sizes())) {
            PyErr_SetString(PyExc_ValueError, "excluded must be a contiguous uint8 CUDA tensor of the bias shape");
            return nullptr;
        }
    }
    const at::Tensor* ref = bias ? bias : mask;
    if (ref && (ref->dim() != 4 || ref->size(2) != L.N || ref->size(3) != L.N || ref->size(0) > INT32_MAX || ref->size(1) > INT32_MAX)) {
        PyErr_SetString(PyExc_ValueError, "bias must be [bias_B,bias_H,N,N]");
        return nullptr;
    }
    if (!stream_arg(a[9], L.device, &stream)) return nullptr;
    qflash_dynamic_info* ip = info ? (qflash_dynamic_info*)info->data_ptr() : nullptr;
    void* wp = ws->data_ptr();
    const size_t wn = (size_t)ws->numel();
    const float* bp = bias ? (const float*)bias->data_ptr() : nullptr;
    const uint8_t* mp = mask ? (const uint8_t*)mask->data_ptr() : nullptr;
    const int rB = ref ? (int)ref->size(0) : 0, rH = ref ? (int)ref->size(1) : 0;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (ref)
        rc = qflash_attention_dynamic_bias(ctx, (const float*)L.q, (const float*)L.k, (const float*)L.v, (int8_t*)L.o, bp, mp,
                                           rB, rH, L.B, L.H, L.N, L.d, tile, out_round, ip, wp, wn, stream);
    else
        rc = qflash_attention_dynamic(ctx, (const float*)L.q, (const float*)L.k, (const float*)L.v, (int8_t*)L.o, L.B, L.H,
                                      L.N, L.d, tile, out_round, ip, wp, wn, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    QF_CATCH
}

// bind_types(QFlashParams, ctypes.Array)
PyObject* bind_types(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!count_is(n, 2)) return nullptr;
    if (!PyType_Check(a[0]) || !PyType_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "bind_types takes two types");
        return nullptr;
    }
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XDECREF((PyObject*)g_params_type);
    Py_XDECREF((PyObject*)g_array_type);
    g_params_type = (PyTypeObject*)a[0];
    g_array_type = (PyTypeObject*)a[1];
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind_types", (PyCFunction)(void (*)(void))bind_types, METH_FASTCALL,
     "bind_types(QFlashParams, ctypes.Array): the types that constants are accepted in"},
    {"attention", (PyCFunction)(void (*)(void))attention, METH_FASTCALL,
     "attention(entry, ctx, Q, K, V, O, params, kv_tile, bias, stream) -> error code; entry 0: per tensor, 1: static, 2: per head"},
    {"attention_packed_bias", (PyCFunction)(void (*)(void))attention_packed_bias, METH_FASTCALL,
     "attention_packed_bias(ctx, Q, K, V, O, params, kv_tile, packed, bias_B, bias_H, stream) -> error code"},
    {"attention_dynamic", (PyCFunction)(void (*)(void))attention_dynamic, METH_FASTCALL,
     "attention_dynamic(ctx, Qf, Kf, Vf, O, kv_tile, workspace, info, out_round, stream, bias_real, excluded) -> error code"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_qflash_native", "Argument marshalling of the C ABI for torch tensors.", -1,
                       kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qflash_native(void) { return PyModule_Create(&kModule); }
