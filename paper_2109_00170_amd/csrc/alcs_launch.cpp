// Python entry of the launches that a program makes once per layer and pass: reads the tensors'
// pointers, shapes and types through PyTorch's C++ interface, takes the current stream and calls the C
// ABI.  For small layers the call itself is the cost: one layer on one image takes the GPU about 3 us,
// while marshalling four tensors through ctypes (attribute look-ups, string comparisons of the type,
// pointer objects, the Python wrapper of the current stream) took 6 us of the call's 8.3; here it takes
// about 0.4.  No arithmetic and no state beyond the addresses of the C functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>
#include <new>

#include "alcs_internal.h"

namespace {

decltype(&alcs_sparse_conv) p_sparse = nullptr;
decltype(&alcs_sparse_conv_fused) p_fused = nullptr;
decltype(&alcs_sparse_conv_bf16) p_bf16 = nullptr;
decltype(&alcs_sparse_conv_bf16_mfma) p_mfma16 = nullptr;
decltype(&alcs_dense_conv) p_dense = nullptr;
decltype(&alcs_depthwise_conv) p_depthwise = nullptr;
decltype(&alcs_dw_sparse_conv_fused) p_dw = nullptr;
decltype(&alcs_block_scores) p_scores = nullptr;
decltype(&alcs_pack_network_device) p_pack_network = nullptr;
PyObject *g_error = nullptr;  // AlcsError(status, where)
PyObject *s_ptr = nullptr, *s_cuda_stream = nullptr;

// A tensor argument: a contiguous device tensor of the wanted type, or None where that is allowed.
struct Arg {
    void *p = nullptr;
    const at::Tensor *t = nullptr;
    int64_t dim(int i) const { return t->size(i); }
};
bool tensor(PyObject *o, const char *name, at::ScalarType type, bool none_ok, Arg &a) {
    if (o == Py_None && none_ok) return true;
    if (o == Py_None || !THPVariable_Check(o)) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous %s tensor on the GPU", name, c10::toString(type));
        return false;
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous %s tensor on the GPU", name, c10::toString(type));
        return false;
    }
    a.t = &t;
    a.p = t.data_ptr();
    return true;
}
bool shape(const Arg &a, const char *name, std::initializer_list<int64_t> want) {
    if (!a.t) return true;
    bool ok = a.t->dim() == (int64_t)want.size();
    int i = 0;
    for (int64_t w : want) ok = ok && a.t->size(i++) == w;
    if (!ok) PyErr_Format(PyExc_ValueError, "%s does not have the shape the call asks for", name);
    return ok;
}
// Four dimensions, each one that fits the C entries' int.
bool four(const Arg &a, const char *name) {
    if (a.t->dim() != 4) {
        PyErr_Format(PyExc_ValueError, "%s must have four dimensions", name);
        return false;
    }
    for (int i = 0; i < 4; ++i)
        if (a.dim(i) > INT32_MAX) {
            PyErr_Format(PyExc_ValueError, "%s: a dimension of %lld is more than the library takes", name, (long long)a.dim(i));
            return false;
        }
    return true;
}
// Weights [Cout, Cin, k, k].
bool filters(const Arg &a, const char *name) {
    if (!four(a, name)) return false;
    if (a.dim(2) == a.dim(3)) return true;
    PyErr_Format(PyExc_ValueError, "%s must be [Cout, Cin, k, k]", name);
    return false;
}
// A value for every channel (a bias may have more, and any shape).
bool per_channel(const Arg &a, const char *name, int64_t channels) {
    if (!a.t || a.t->numel() >= channels) return true;
    PyErr_Format(PyExc_ValueError, "%s must have %lld entries, got %lld", name, (long long)channels, (long long)a.t->numel());
    return false;
}
bool integer(PyObject *o, int &v) {
    PyObject *i = PyNumber_Long(o);
    if (!i) return false;
    const long x = PyLong_AsLong(i);
    Py_DECREF(i);
    if (x == -1 && PyErr_Occurred()) return false;
    if (x != (int)x) {
        PyErr_Format(PyExc_ValueError, "%ld is no 32-bit integer", x);
        return false;
    }
    v = (int)x;
    return true;
}
// None, "none", "relu", "relu6" or an alcs_activation integer.
bool activation(PyObject *o, int &v) {
    if (o == Py_None) { v = 0; return true; }
    if (PyUnicode_Check(o)) {
        const char *s = PyUnicode_AsUTF8(o);
        if (!s) return false;
        if (!std::strcmp(s, "relu")) v = 1;
        else if (!std::strcmp(s, "relu6")) v = 2;
        else if (!std::strcmp(s, "none")) v = 0;
        else { PyErr_SetObject(PyExc_KeyError, o); return false; }
        return true;
    }
    if (!PyLong_Check(o)) { PyErr_SetObject(PyExc_KeyError, o); return false; }
    return integer(o, v);
}
// None: PyTorch's current stream; a stream object; or a hipStream_t as an integer.
bool stream_of(PyObject *o, void *&st) {
    if (o == Py_None) {
        st = (void *)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    PyObject *v = PyObject_GetAttr(o, s_cuda_stream);
    if (!v) {
        PyErr_Clear();
        v = PyNumber_Long(o);
        if (!v) return false;
    }
    PyObject *i = PyNumber_Long(v);
    Py_DECREF(v);
    if (!i) return false;
    st = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return !PyErr_Occurred();
}
const alcs_packed *handle(PyObject *packed) {
    PyObject *v = PyObject_GetAttr(packed, s_ptr);
    if (!v) return nullptr;
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) return nullptr;
    if (!x) PyErr_SetString(PyExc_ValueError, "packed weights were freed");
    return (const alcs_packed *)(uintptr_t)x;
}
int64_t out_size(int64_t size, int k, int stride) {
    const int64_t span = size + 2 * ((k - 1) / 2) - k;
    // the floor of a negative span's quotient, as integer division in Python
    return stride > 0 ? (span >= 0 ? span / stride : -((-span + stride - 1) / stride)) + 1 : 0;
}
PyObject *done(int rc, const char *where) {
    if (rc == ALCS_OK) Py_RETURN_NONE;
    PyObject *args = Py_BuildValue("(is)", rc, where), *e = args ? PyObject_CallObject(g_error, args) : nullptr;
    Py_XDECREF(args);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}
bool count(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments wanted, got %zd", want, n);
    return false;
}

// packed, X, bias, residual, Y, stride, activation, stream - for the four convolutions through a handle
enum Kind { kPlain, kFused, kBf16, kMfma16 };
PyObject *conv(Kind kind, const char *where, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 8)) return nullptr;
    const alcs_packed *p = handle(a[0]);
    if (!p) return nullptr;
    const at::ScalarType io = kind >= kBf16 ? at::kBFloat16 : at::kFloat;
    Arg X, bias, R, Y;
    int stride = 1, act = 0;
    void *st = nullptr;
    if (!tensor(a[1], "X", io, false, X) || !four(X, "X") || !tensor(a[2], "bias", at::kFloat, true, bias) ||
        !tensor(a[3], "residual", io, true, R) || !tensor(a[4], "Y", io, false, Y) || !integer(a[5], stride) ||
        !activation(a[6], act))
        return nullptr;
    const int64_t N = X.dim(0), Cin = X.dim(1), H = X.dim(2), W = X.dim(3);
    if (stride == 0) { PyErr_SetString(PyExc_ZeroDivisionError, "stride is zero"); return nullptr; }
    const int64_t Ho = out_size(H, p->k, stride), Wo = out_size(W, p->k, stride);
    if (stride > 0 && (!shape(Y, "Y", {N, p->Cout, Ho, Wo}) || !shape(R, "residual", {N, p->Cout, Ho, Wo}))) return nullptr;
    if (!per_channel(bias, "bias", p->Cout) || !stream_of(a[7], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    switch (kind) {
        case kPlain:
            rc = p_sparse(p, (const float *)X.p, (const float *)bias.p, (float *)Y.p, (int)N, (int)Cin, p->Cout, (int)H, (int)W,
                          p->k, stride, st);
            break;
        case kFused:
            rc = p_fused(p, (const float *)X.p, (const float *)bias.p, (const float *)R.p, (float *)Y.p, (int)N, (int)Cin, p->Cout,
                         (int)H, (int)W, p->k, stride, act, st);
            break;
        default:
            rc = (kind == kBf16 ? p_bf16 : p_mfma16)(p, (const uint16_t *)X.p, (const float *)bias.p, (const uint16_t *)R.p,
                                                     (uint16_t *)Y.p, (int)N, (int)Cin, p->Cout, (int)H, (int)W, p->k, stride, act,
                                                     st);
    }
    Py_END_ALLOW_THREADS
    return done(rc, where);
}
PyObject *sparse_conv(PyObject *, PyObject *const *a, Py_ssize_t n) { return conv(kPlain, "alcs_sparse_conv", a, n); }
PyObject *sparse_conv_fused(PyObject *, PyObject *const *a, Py_ssize_t n) { return conv(kFused, "alcs_sparse_conv_fused", a, n); }
PyObject *sparse_conv_bf16(PyObject *, PyObject *const *a, Py_ssize_t n) { return conv(kBf16, "alcs_sparse_conv_bf16", a, n); }
PyObject *sparse_conv_bf16_mfma(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return conv(kMfma16, "alcs_sparse_conv_bf16_mfma", a, n);
}

// W, X, bias, Y, stride, stream
PyObject *dense_conv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 6)) return nullptr;
    Arg W, X, bias, Y;
    int stride = 1;
    void *st = nullptr;
    if (!tensor(a[0], "W", at::kFloat, false, W) || !filters(W, "W") || !tensor(a[1], "X", at::kFloat, false, X) || !four(X, "X") ||
        !tensor(a[2], "bias", at::kFloat, true, bias) || !tensor(a[3], "Y", at::kFloat, false, Y) || !integer(a[4], stride))
        return nullptr;
    const int64_t N = X.dim(0), Cin = X.dim(1), H = X.dim(2), Wd = X.dim(3), Cout = W.dim(0);
    const int k = (int)W.dim(2);
    if (W.dim(1) != Cin) { PyErr_SetString(PyExc_ValueError, "channel mismatch"); return nullptr; }
    if (stride == 0) { PyErr_SetString(PyExc_ZeroDivisionError, "stride is zero"); return nullptr; }
    if (stride > 0 && !shape(Y, "Y", {N, Cout, out_size(H, k, stride), out_size(Wd, k, stride)})) return nullptr;
    if (!per_channel(bias, "bias", Cout) || !stream_of(a[5], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p_dense((const float *)W.p, (const float *)X.p, (const float *)bias.p, (float *)Y.p, (int)N, (int)Cin, (int)Cout, (int)H,
                 (int)Wd, k, stride, st);
    Py_END_ALLOW_THREADS
    return done(rc, "alcs_dense_conv");
}

// D, X, bias, Y, stride, activation, stream
PyObject *depthwise_conv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 7)) return nullptr;
    Arg D, X, bias, Y;
    int stride = 1, act = 0;
    void *st = nullptr;
    if (!tensor(a[0], "dw_weights", at::kFloat, false, D) || !tensor(a[1], "X", at::kFloat, false, X) || !four(X, "X") ||
        !tensor(a[2], "bias", at::kFloat, true, bias) || !tensor(a[3], "Y", at::kFloat, false, Y) || !integer(a[4], stride) ||
        !activation(a[5], act))
        return nullptr;
    const int64_t N = X.dim(0), C = X.dim(1), H = X.dim(2), W = X.dim(3);
    if (!shape(D, "dw_weights", {C, 3, 3})) return nullptr;
    if (stride == 0) { PyErr_SetString(PyExc_ZeroDivisionError, "stride is zero"); return nullptr; }
    if (stride > 0 && !shape(Y, "Y", {N, C, out_size(H, 3, stride), out_size(W, 3, stride)})) return nullptr;
    if (!per_channel(bias, "bias", C) || !stream_of(a[6], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p_depthwise((const float *)D.p, (const float *)X.p, (const float *)bias.p, (float *)Y.p, (int)N, (int)C, (int)H, (int)W,
                     stride, act, st);
    Py_END_ALLOW_THREADS
    return done(rc, "alcs_depthwise_conv");
}

// packed, D, dw_bias, X, bias, residual, Y, dw_stride, dw_activation, activation, workspace, stream
PyObject *dw_sparse_conv_fused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 12)) return nullptr;
    const alcs_packed *p = handle(a[0]);
    if (!p) return nullptr;
    Arg D, db, X, bias, R, Y, ws;
    int stride = 1, dw_act = 0, act = 0;
    void *st = nullptr;
    if (!tensor(a[1], "dw_weights", at::kFloat, false, D) || !tensor(a[2], "dw_bias", at::kFloat, true, db) ||
        !tensor(a[3], "X", at::kFloat, false, X) || !four(X, "X") || !tensor(a[4], "bias", at::kFloat, true, bias) ||
        !tensor(a[5], "residual", at::kFloat, true, R) || !tensor(a[6], "Y", at::kFloat, false, Y) || !integer(a[7], stride) ||
        !activation(a[8], dw_act) || !activation(a[9], act) || !tensor(a[10], "workspace", at::kFloat, true, ws))
        return nullptr;
    const int64_t N = X.dim(0), C = X.dim(1), H = X.dim(2), W = X.dim(3);
    if (!shape(D, "dw_weights", {C, 3, 3})) return nullptr;
    if (stride == 0) { PyErr_SetString(PyExc_ZeroDivisionError, "stride is zero"); return nullptr; }
    if (stride > 0) {
        const int64_t Ho = out_size(H, 3, stride), Wo = out_size(W, 3, stride);
        if (!shape(Y, "Y", {N, p->Cout, Ho, Wo}) || !shape(R, "residual", {N, p->Cout, Ho, Wo}) ||
            !shape(ws, "workspace", {N, C, Ho, Wo}))
            return nullptr;
    }
    if (!per_channel(db, "dw_bias", C) || !per_channel(bias, "bias", p->Cout) || !stream_of(a[11], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p_dw(p, (const float *)D.p, (const float *)db.p, stride, dw_act, (const float *)X.p, (const float *)bias.p,
              (const float *)R.p, (float *)Y.p, (float *)ws.p, (int)N, (int)C, p->Cout, (int)H, (int)W, act, st);
    Py_END_ALLOW_THREADS
    return done(rc, "alcs_dw_sparse_conv_fused");
}

// W, V, scores, stream
PyObject *block_scores(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 4)) return nullptr;
    Arg W, S;
    int V = 0;
    void *st = nullptr;
    if (!tensor(a[0], "W", at::kFloat, false, W) || !filters(W, "W") || !integer(a[1], V) ||
        !tensor(a[2], "scores", at::kFloat, false, S))
        return nullptr;
    const int64_t Cout = W.dim(0), Cin = W.dim(1), k = W.dim(2);
    if (V <= 0) { PyErr_SetString(PyExc_ValueError, "the group size must be positive"); return nullptr; }
    if (!shape(S, "scores", {(Cout + V - 1) / V, Cin, k, k})) return nullptr;
    if (!stream_of(a[3], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p_scores((const float *)W.p, (int)Cout, (int)Cin, (int)k, V, (float *)S.p, st);
    Py_END_ALLOW_THREADS
    return done(rc, "alcs_block_scores");
}

// (G, K, nnzb) of a handle given by its address
PyObject *packed_info(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 1)) return nullptr;
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(a[0]);
    if (PyErr_Occurred()) return nullptr;
    if (!x) return done(ALCS_E_INVALID_ARG, "alcs_packed_info");
    const alcs_packed *p = (const alcs_packed *)(uintptr_t)x;
    return Py_BuildValue("(iiL)", p->G, p->K, (long long)p->nnzb);
}

// [W], [mask or None], [V], [address of alcs_options or 0], workspace or None, stream ->
// [(address, Cout, Cin, kernel, V)]
PyObject *pack_network(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 6)) return nullptr;
    const Py_ssize_t layers = PyList_Check(a[0]) ? PyList_GET_SIZE(a[0]) : -1;
    for (int i = 0; i < 4; ++i)
        if (!PyList_Check(a[i]) || PyList_GET_SIZE(a[i]) != layers) {
            PyErr_SetString(PyExc_ValueError, "one weight tensor, mask, group size and option per layer");
            return nullptr;
        }
    std::vector<alcs_layer_desc> desc((size_t)layers);
    std::vector<alcs_packed_t *> out((size_t)layers, nullptr);
    for (Py_ssize_t i = 0; i < layers; ++i) {
        Arg W, M;
        int V = 0;
        if (!tensor(PyList_GET_ITEM(a[0], i), "W", at::kFloat, false, W) || !filters(W, "W") ||
            !tensor(PyList_GET_ITEM(a[1], i), "mask", at::kByte, true, M) || !integer(PyList_GET_ITEM(a[2], i), V))
            return nullptr;
        const int64_t Cout = W.dim(0), Cin = W.dim(1), k = W.dim(2);
        if (V <= 0) { PyErr_SetString(PyExc_ValueError, "the group size must be positive"); return nullptr; }
        if (M.t && M.t->numel() != (Cout + V - 1) / V * Cin * k * k) {
            PyErr_Format(PyExc_ValueError, "mask %zd must have %lld entries", i, (long long)((Cout + V - 1) / V * Cin * k * k));
            return nullptr;
        }
        const unsigned long long opt = PyLong_AsUnsignedLongLongMask(PyList_GET_ITEM(a[3], i));
        if (PyErr_Occurred()) return nullptr;
        desc[(size_t)i] = alcs_layer_desc{(const float *)W.p, (const uint8_t *)M.p, (int)Cout, (int)Cin, (int)k, V,
                                          (const alcs_options *)(uintptr_t)opt};
    }
    Arg ws;
    void *st = nullptr;
    if (!tensor(a[4], "workspace", at::kByte, true, ws) || !stream_of(a[5], st)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = p_pack_network(desc.data(), (int)layers, ws.p, ws.t ? (long long)ws.t->numel() : 0, st, out.data());
    Py_END_ALLOW_THREADS
    if (rc != ALCS_OK) return done(rc, "alcs_pack_network_device");
    PyObject *list = PyList_New(layers);
    for (Py_ssize_t i = 0; list && i < layers; ++i) {
        const alcs_layer_desc &d = desc[(size_t)i];
        PyObject *t = Py_BuildValue("(Kiiii)", (unsigned long long)(uintptr_t)out[(size_t)i], d.Cout, d.Cin, d.kernel, d.V);
        if (!t) { Py_DECREF(list); return nullptr; }
        PyList_SET_ITEM(list, i, t);
    }
    return list;
}

// error class, {name: address}
PyObject *connect(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!count(n, 2)) return nullptr;
    auto get = [&](const char *name, auto &fn) {
        PyObject *v = PyDict_GetItemString(a[1], name);
        if (!v) { PyErr_Format(PyExc_KeyError, "%s", name); return false; }
        fn = (std::decay_t<decltype(fn)>)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
        return !PyErr_Occurred();
    };
    if (!get("alcs_sparse_conv", p_sparse) || !get("alcs_sparse_conv_fused", p_fused) || !get("alcs_sparse_conv_bf16", p_bf16) ||
        !get("alcs_sparse_conv_bf16_mfma", p_mfma16) || !get("alcs_dense_conv", p_dense) ||
        !get("alcs_depthwise_conv", p_depthwise) || !get("alcs_dw_sparse_conv_fused", p_dw) || !get("alcs_block_scores", p_scores) ||
        !get("alcs_pack_network_device", p_pack_network))
        return nullptr;
    Py_INCREF(a[0]);
    Py_XDECREF(g_error);
    g_error = a[0];
    Py_RETURN_NONE;
}

// Reading a tensor can throw (one without storage, as a tracer makes; a sparse one; no device): the
// interpreter's C frames must not see that.
typedef PyObject *(*Entry)(PyObject *, PyObject *const *, Py_ssize_t);
template <Entry F>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) noexcept {
    try {
        return F(self, a, n);
    } catch (const std::bad_alloc &) {
        return PyErr_NoMemory();
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(connect),        ENTRY(sparse_conv),          ENTRY(sparse_conv_fused),
                         ENTRY(sparse_conv_bf16), ENTRY(sparse_conv_bf16_mfma), ENTRY(dense_conv),
                         ENTRY(depthwise_conv), ENTRY(dw_sparse_conv_fused), ENTRY(block_scores),
                         ENTRY(packed_info),    ENTRY(pack_network),         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch(void) {
    s_ptr = PyUnicode_InternFromString("_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_ptr || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
