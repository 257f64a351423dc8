// Native argument marshalling of the Python binding (binding.py): the calls that programs make in earnest, device tensors
// in plain descriptions, go from here straight to the C ABI.  Everything else (no tensor, other tensor classes,
// descriptions that do not fit their tensors, integers of other types) returns -1 before anything is launched, and the
// binding marshals it itself, with its own checks and messages.
//
// Why: a call of a small product is bound by the host.  With the descriptors built in Python and ctypes the
// marshalling took 4 to 5 us of the 7 to 9 of a call of fg_gemm and 8 of the 11 to 12 of fg_contract; the launch itself takes 3.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <pthread.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/flexgemm.h"

namespace {

typedef fg_status (*GemmFn)(int64_t, int64_t, int64_t, float, const fg_matrix *, const fg_matrix *, float, const fg_matrix *, const fg_matrix *,
                            const fg_epilogue *, void *);
typedef fg_status (*GemmExFn)(int64_t, int64_t, int64_t, float, const fg_matrix *, const fg_matrix *, float, const fg_matrix *, const fg_matrix *,
                              const fg_epilogue *, const fg_load_transforms *, void *);
typedef fg_status (*DualFn)(int64_t, int64_t, int64_t, float, const fg_matrix *, const fg_matrix *, float, const fg_matrix *, const fg_matrix *, void *);
typedef fg_status (*ContractFn)(int32_t, const int32_t *, const int64_t *, const void *, int32_t, const int32_t *, const int64_t *, const void *, int32_t,
                                const int32_t *, const int64_t *, const float *, float *, int32_t, const int32_t *, const int64_t *, float, float, void *);

struct Entry { GemmFn gemm; GemmExFn ex, noalloc; DualFn dual; ContractFn contract; } g_entry;
PyObject *g_matrix_type, *g_raw_stream, *g_device;                 // binding.Matrix and how the current stream is asked for
PyObject *s_re, *s_im, *s_layout, *s_ld, *s_dtype;
bool g_forked;                                                    // a child of fork() cannot use the GPU: torch says so

// An integer that fits; anything else is left to the binding.
bool as_int(PyObject *o, int64_t &v) {
    if (!o || !PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool as_float(PyObject *o, float &v) {
    if (PyFloat_CheckExact(o)) { v = (float)PyFloat_AS_DOUBLE(o); return true; }
    int64_t i;
    if (!as_int(o, i) || i > (1 << 24) || i < -(1 << 24)) return false;
    v = (float)i;
    return true;
}

// Address and element count of a plain device tensor; what its dtype is called in the C ABI.
struct Device { void *ptr; int64_t numel; int dtype; bool is_complex; };
bool device_tensor(PyObject *o, Device &d) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) return false;
    d.ptr = t.data_ptr();
    d.numel = t.numel();
    d.is_complex = t.is_complex();
    switch (t.scalar_type()) {
        case at::kHalf: d.dtype = FG_F16; break;
        case at::kBFloat16: d.dtype = FG_BF16; break;
        case at::kFloat: d.dtype = FG_F32; break;
        case at::kComplexHalf: d.dtype = FG_CF16; break;
        case at::kComplexFloat: d.dtype = FG_CF32; break;
        default: return false;
    }
    return true;
}

// binding.Matrix -> fg_matrix, with the binding's check that the tensors hold the matrix.  present: false for None.
bool matrix(PyObject *o, int64_t rows, int64_t cols, fg_matrix &x, bool &present) {
    present = o != Py_None;
    if (!present) return true;
    if ((PyObject *)Py_TYPE(o) != g_matrix_type) return false;
    PyObject **dict = _PyObject_GetDictPtr(o);
    if (!dict || !*dict) return false;
    PyObject *re = PyDict_GetItemWithError(*dict, s_re), *im = PyDict_GetItemWithError(*dict, s_im), *dt = PyDict_GetItemWithError(*dict, s_dtype);
    int64_t layout, ld, dtype;
    if (!re || !im || !dt || !as_int(PyDict_GetItemWithError(*dict, s_layout), layout) || !as_int(PyDict_GetItemWithError(*dict, s_ld), ld)) return false;
    Device t[2];
    if (!device_tensor(re, t[0])) return false;
    const bool two = im != Py_None;
    if (two && !device_tensor(im, t[1])) return false;
    if (dt == Py_None) dtype = t[0].dtype;
    else if (!as_int(dt, dtype)) return false;
    if (layout < 0 || layout > FG_ZERO || dtype < 0 || dtype > FG_CF32 || ld < 0 || ld > (1ll << 31) || rows > (1 << 30) || cols > (1 << 30)) return false;
    const int64_t need = layout == FG_COL ? (ld >= rows ? (cols - 1) * ld + rows : 0) : layout == FG_ROW ? (ld >= cols ? (rows - 1) * ld + cols : 0)
                       : layout == FG_DIAG ? (rows < cols ? rows : cols) : 0;
    for (int k = 0; k < (two ? 2 : 1); ++k) {
        const int64_t per_entry = (dt != Py_None && (dtype == FG_CF16 || dtype == FG_CF32) && !t[k].is_complex) ? 2 : 1;
        if (need > t[k].numel / per_entry) return false;              // the binding raises
    }
    x.re = t[0].ptr;
    x.im = two ? t[1].ptr : nullptr;
    x.dtype = (int32_t)dtype;
    x.layout = (int32_t)layout;
    x.ld = ld;
    return true;
}

bool current_stream(PyObject *stream, void *&handle) {
    if (stream != Py_None) return false;
    PyObject *dev = PyObject_CallNoArgs(g_device);
    PyObject *raw = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
    Py_XDECREF(dev);
    handle = raw ? PyLong_AsVoidPtr(raw) : nullptr;
    Py_XDECREF(raw);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

PyObject *not_here() {
    PyErr_Clear();
    return PyLong_FromLong(-1);
}

// gemm(M, N, K, alpha, A, B, beta, C, D, bias, bias_dim, act, stream, a_add, b_add, c_act, noalloc) -> status
// dual(M, N, K, alpha, A, B, beta, C, D, stream) -> status
PyObject *product(PyObject *const *a, Py_ssize_t n, bool dual) {
    if (g_forked || n != (dual ? 10 : 17)) return not_here();
    try {
        int64_t M, N, K, bias_dim = 0, act = 0, c_act = 0;
        float alpha, beta, a_add = 0.f, b_add = 0.f;
        if (!as_int(a[0], M) || !as_int(a[1], N) || !as_int(a[2], K) || !as_float(a[3], alpha) || !as_float(a[6], beta) || M <= 0 || N <= 0 || K <= 0) return not_here();
        fg_matrix A, B, C, D;
        bool has_a, has_b, has_c, has_d;
        if (!matrix(a[4], M, K, A, has_a) || !matrix(a[5], K, N, B, has_b) || !matrix(a[7], M, N, C, has_c) || !matrix(a[8], M, N, D, has_d)) return not_here();
        if (!has_a || !has_b || !has_d) return not_here();
        fg_epilogue ep = {};
        bool has_ep = false, noalloc = false;
        if (!dual) {
            if (!as_int(a[10], bias_dim) || !as_int(a[11], act) || !as_float(a[13], a_add) || !as_float(a[14], b_add) || !as_int(a[15], c_act) ||
                (a[16] != Py_False && a[16] != Py_True)) return not_here();
            if (bias_dim < 0 || bias_dim > 1 || act < 0 || act > 1 || c_act < 0 || c_act > 1) return not_here();
            noalloc = a[16] == Py_True;
            if (a[9] != Py_None) {
                Device bias;
                if (!device_tensor(a[9], bias)) return not_here();
                ep.bias = (const float *)bias.ptr;
            }
            ep.bias_dim = (int32_t)bias_dim;
            ep.act = (int32_t)act;
            has_ep = ep.bias || act != FG_ACT_NONE || a[9] != Py_None;
        }
        void *stream;
        if (!current_stream(a[dual ? 9 : 12], stream)) return not_here();
        const fg_matrix *c = has_c ? &C : nullptr;
        const fg_epilogue *e = has_ep ? &ep : nullptr;
        const fg_load_transforms lt = {a_add, b_add, (int32_t)c_act};
        auto call = [&]() noexcept {
            if (dual) return g_entry.dual(M, N, K, alpha, &A, &B, beta, c, &D, stream);
            if (noalloc) return g_entry.noalloc(M, N, K, alpha, &A, &B, beta, c, &D, e, &lt, stream);
            if (a_add != 0.f || b_add != 0.f || c_act != FG_ACT_NONE) return g_entry.ex(M, N, K, alpha, &A, &B, beta, c, &D, e, &lt, stream);
            return g_entry.gemm(M, N, K, alpha, &A, &B, beta, c, &D, e, stream);
        };
        fg_status st;
        Py_BEGIN_ALLOW_THREADS
        st = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(st);
    } catch (...) {                                                  // a tensor without storage: the binding's own call says what is wrong
        return not_here();
    }
}
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n) { return product(args, n, false); }
PyObject *dual(PyObject *, PyObject *const *args, Py_ssize_t n) { return product(args, n, true); }

constexpr int kModes = 12, kLabels = 24;                              // what the library takes
struct Modes { int32_t n; int32_t label[kModes]; int64_t stride[kModes]; };
bool modes(PyObject *labels, PyObject *strides, Modes &m) {
    if (!(PyList_CheckExact(labels) || PyTuple_CheckExact(labels)) || !(PyList_CheckExact(strides) || PyTuple_CheckExact(strides))) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(labels);
    if (n > kModes || PySequence_Fast_GET_SIZE(strides) != n) return false;
    for (Py_ssize_t i = 0; i < n; ++i) {
        int64_t l, s;
        if (!as_int(PySequence_Fast_GET_ITEM(labels, i), l) || !as_int(PySequence_Fast_GET_ITEM(strides, i), s)) return false;
        if (l < INT32_MIN || l > INT32_MAX || s < 0 || s > (1ll << 40)) return false;
        m.label[i] = (int32_t)l;
        m.stride[i] = s;
    }
    m.n = (int32_t)n;
    return true;
}

// contract(modesA, stridesA, A, modesB, stridesB, B, modesC, stridesC, Cin, Cout, extents, alpha, beta, stream) -> status
PyObject *contract(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (g_forked || n != 14) return not_here();
    try {
        Modes mA, mB, mC;
        Device A, B, Cin = {}, Cout;
        float alpha, beta;
        if (!modes(a[0], a[1], mA) || !modes(a[3], a[4], mB) || !modes(a[6], a[7], mC) || !PyDict_CheckExact(a[10])) return not_here();
        if (!device_tensor(a[2], A) || !device_tensor(a[5], B) || !device_tensor(a[9], Cout)) return not_here();
        if (a[8] != Py_None && !device_tensor(a[8], Cin)) return not_here();
        if (!as_float(a[11], alpha) || !as_float(a[12], beta)) return not_here();
        int32_t labels[kLabels], count = 0;
        int64_t extents[kLabels];
        PyObject *key, *value;
        Py_ssize_t pos = 0;
        while (PyDict_Next(a[10], &pos, &key, &value)) {
            int64_t l, e;
            if (count == kLabels || !as_int(key, l) || !as_int(value, e) || l < INT32_MIN || l > INT32_MAX || e <= 0 || e > (1 << 30)) return not_here();
            labels[count] = (int32_t)l;
            extents[count++] = e;
        }
        // the last element that a description reaches must exist (a mode without an extent: the library refuses it)
        auto holds = [&](const Modes &m, const Device &t) {
            int64_t need = 1;
            for (int i = 0; i < m.n; ++i) {
                int64_t e = 0;
                for (int k = 0; k < count; ++k) if (labels[k] == m.label[i]) e = extents[k];
                if (e == 0) return false;
                if ((e - 1) > 0 && m.stride[i] > (1ll << 44) / (e - 1)) return false;
                need += (e - 1) * m.stride[i];
            }
            return need <= t.numel;
        };
        if (!holds(mA, A) || !holds(mB, B) || !holds(mC, Cout) || (a[8] != Py_None && !holds(mC, Cin))) return not_here();
        void *stream;
        if (!current_stream(a[13], stream)) return not_here();
        auto call = [&]() noexcept {
            return g_entry.contract(mA.n, mA.label, mA.stride, A.ptr, mB.n, mB.label, mB.stride, B.ptr, mC.n, mC.label, mC.stride, (const float *)Cin.ptr,
                                    (float *)Cout.ptr, count, labels, extents, alpha, beta, stream);
        };
        fg_status st;
        Py_BEGIN_ALLOW_THREADS
        st = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(st);
    } catch (...) {
        return not_here();
    }
}

// setup(Matrix, raw_stream, device, addresses of fg_gemm, fg_gemm_ex, fg_gemm_noalloc, fg_gemm_dual, fg_contract)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "setup takes 8 arguments"); return nullptr; }
    void *f[5];
    for (int i = 0; i < 5; ++i) {
        f[i] = PyLong_AsVoidPtr(a[3 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    g_entry = Entry{(GemmFn)f[0], (GemmExFn)f[1], (GemmExFn)f[2], (DualFn)f[3], (ContractFn)f[4]};
    Py_INCREF(a[0]); Py_INCREF(a[1]); Py_INCREF(a[2]);
    g_matrix_type = a[0]; g_raw_stream = a[1]; g_device = a[2];
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"setup", (PyCFunction)(void (*)(void))setup, METH_FASTCALL, nullptr},
                           {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
                           {"dual", (PyCFunction)(void (*)(void))dual, METH_FASTCALL, nullptr},
                           {"contract", (PyCFunction)(void (*)(void))contract, METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", "Native marshalling of binding.py's calls.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
    s_re = PyUnicode_InternFromString("re");
    s_im = PyUnicode_InternFromString("im");
    s_layout = PyUnicode_InternFromString("layout");
    s_ld = PyUnicode_InternFromString("ld");
    s_dtype = PyUnicode_InternFromString("dtype");
    pthread_atfork(nullptr, nullptr, [] { g_forked = true; });
    return PyModule_Create(&g_module);
}
