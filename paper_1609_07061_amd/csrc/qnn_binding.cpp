// The Python binding's native part: argument marshalling of the calls that are made per layer or per time step, whose kernels take a
// few microseconds.  ctypes and the reading of shapes and strides through Python objects cost 2.7 of the 5.4 us that such a call took on
// the host (the launch itself 2.7); here they cost 0.2.
//
// Every function returns the C entry point's status, or -1 for "not here": the caller then takes the general path in __init__.py, which
// handles whatever this one does not (no output given, other tensor classes, tensors without memory, numbers that are no integers) and
// raises the errors.  Nothing is kept between calls but the entry points' addresses.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

namespace {

typedef int (*PackSign)(const float *, int64_t, int64_t, int64_t, uint32_t *, int64_t, void *);
typedef int (*LinearQuant)(const float *, int64_t, int64_t, int64_t, float, int32_t, int32_t, int, uint32_t *, int64_t, int64_t, void *);
typedef int (*BinaryGemm)(const uint32_t *, int64_t, const uint32_t *, int64_t, int32_t *, int64_t, int64_t, int64_t, int64_t, void *);
typedef int (*BinaryGemmSign)(const uint32_t *, int64_t, const uint32_t *, int64_t, const int32_t *, const uint8_t *, uint32_t *, int64_t, int64_t,
                              int64_t, int64_t, int, void *);
typedef int (*BitplaneGemm)(const uint32_t *, int, const int32_t *, int, int64_t, int64_t, const uint32_t *, int, const int32_t *, int, int64_t, int64_t,
                            int32_t *, int64_t, int64_t, int64_t, int64_t, void *);
typedef int (*Conv2d)(const uint32_t *, int, const int32_t *, int, int64_t, int64_t, int64_t, int64_t, int64_t, const uint32_t *, int, const int32_t *,
                      int, int64_t, int64_t, int, int, int, int, int32_t *, void *);
void *g_entry[6];
enum { kPackSign, kLinearQuant, kBinaryGemm, kBinaryGemmSign, kBitplaneGemm, kConv2d };

constexpr int kMaxPlanes = 8;  // QNN_MAX_PLANES

PyObject *not_here() {
    PyErr_Clear();
    return PyLong_FromLong(-1);
}

// A plain tensor of this type with memory on a GPU (others have no address, or are not asked for it like this)
const at::Tensor *tensor(PyObject *o, at::ScalarType type, int64_t dims) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.scalar_type() != type || (dims >= 0 && t.dim() != dims)) return nullptr;
    return &t;
}
struct Rows {
    void *p;
    int64_t planes, rows, cols, ld, stride;
};
// [rows][cols], or [planes][rows][cols], with contiguous rows
bool rows_of(PyObject *o, at::ScalarType type, int64_t dims, Rows &r) {
    const at::Tensor *t = tensor(o, type, dims);
    if (!t) return false;
    const auto size = t->sizes(), step = t->strides();
    const int64_t at = dims - 2;
    r.planes = dims == 3 ? size[0] : 1, r.rows = size[at], r.cols = size[at + 1];
    if (r.cols > 1 && step[at + 1] != 1) return false;
    r.ld = r.rows > 1 ? step[at] : (r.cols > 1 ? r.cols : 1);
    r.stride = r.planes > 1 ? step[0] : 0;
    r.p = t->data_ptr();
    return true;
}
bool integer(PyObject *o, int64_t &v) {
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsLongLong(o);
    return !(v == -1 && PyErr_Occurred());
}
// The current stream's handle, from the function that __init__.py has for it (after everything else is known to be in order)
bool stream(PyObject *function, int64_t &v) {
    PyObject *const r = PyObject_CallNoArgs(function);
    if (!r) return false;
    const bool ok = integer(r, v);
    Py_DECREF(r);
    return ok;
}
bool integer32(PyObject *o, int32_t &v) {
    int64_t w;
    if (!integer(o, w) || w < INT32_MIN || w > INT32_MAX) return false;
    v = (int32_t)w;
    return true;
}
bool coefficients(PyObject *o, int64_t count, int32_t (&c)[kMaxPlanes]) {
    if (!(PyList_CheckExact(o) || PyTuple_CheckExact(o)) || count > kMaxPlanes || PySequence_Fast_GET_SIZE(o) != count) return false;
    for (int64_t i = 0; i < count; ++i)
        if (!integer32(PySequence_Fast_GET_ITEM(o, i), c[i])) return false;
    return true;
}
// Calls f, which returns a status, without the interpreter's lock
template <typename F>
PyObject *call(F f) {
    int status;
    Py_BEGIN_ALLOW_THREADS status = f();
    Py_END_ALLOW_THREADS return PyLong_FromLong(status);
}
void *stream_of(int64_t v) { return reinterpret_cast<void *>(v); }
template <typename T>
T *as(const Rows &r) {
    return static_cast<T *>(r.p);
}

// x, out, stream
PyObject *pack_sign(PyObject *const *a) {
    Rows x, o;
    int64_t s;
    if (!rows_of(a[0], at::kFloat, 2, x) || !rows_of(a[1], at::kInt, 2, o) || !stream(a[2], s)) return not_here();
    return call([&] { return reinterpret_cast<PackSign>(g_entry[kPackSign])(as<float>(x), x.rows, x.cols, x.ld, as<uint32_t>(o), o.ld, stream_of(s)); });
}
// x, step, qmin, qmax, nbits, out, stream
PyObject *linear_quant_planes(PyObject *const *a) {
    Rows x, o;
    int32_t lo, hi, bits;
    int64_t s;
    if (!PyFloat_CheckExact(a[1]) || !rows_of(a[0], at::kFloat, 2, x) || !integer32(a[2], lo) || !integer32(a[3], hi) || !integer32(a[4], bits) ||
        !rows_of(a[5], at::kInt, 3, o) || o.planes != bits || !stream(a[6], s))
        return not_here();
    const float step = (float)PyFloat_AS_DOUBLE(a[1]);
    return call([&] { return reinterpret_cast<LinearQuant>(g_entry[kLinearQuant])(as<float>(x), x.rows, x.cols, x.ld, step, lo, hi, bits, as<uint32_t>(o), o.ld, o.stride, stream_of(s)); });
}
// A, W, K, out, stream
PyObject *binary_gemm(PyObject *const *a) {
    Rows A, W, c;
    int64_t K, s;
    if (!rows_of(a[0], at::kInt, 2, A) || !rows_of(a[1], at::kInt, 2, W) || !integer(a[2], K) || !rows_of(a[3], at::kInt, 2, c) || !stream(a[4], s))
        return not_here();
    return call([&] { return reinterpret_cast<BinaryGemm>(g_entry[kBinaryGemm])(as<uint32_t>(A), A.ld, as<uint32_t>(W), W.ld, as<int32_t>(c), c.ld, A.rows, W.rows, K, stream_of(s)); });
}
// A, W, K, T, flip, out, engine, stream
PyObject *binary_gemm_sign(PyObject *const *a) {
    Rows A, W, o;
    int64_t K, s;
    int32_t engine;
    const at::Tensor *T = tensor(a[3], at::kInt, -1), *flip = a[4] == Py_None ? nullptr : tensor(a[4], at::kByte, -1);
    if (!T || (a[4] != Py_None && !flip) || !rows_of(a[0], at::kInt, 2, A) || !rows_of(a[1], at::kInt, 2, W) || !integer(a[2], K) ||
        !rows_of(a[5], at::kInt, 2, o) || !integer32(a[6], engine) || !stream(a[7], s))
        return not_here();
    const int32_t *const t = static_cast<const int32_t *>(T->data_ptr());
    const uint8_t *const f = flip ? static_cast<const uint8_t *>(flip->data_ptr()) : nullptr;
    return call([&] {
        return reinterpret_cast<BinaryGemmSign>(g_entry[kBinaryGemmSign])(as<uint32_t>(A), A.ld, as<uint32_t>(W), W.ld, t, f, as<uint32_t>(o), o.ld, A.rows, W.rows, K, engine, stream_of(s));
    });
}
// A, coefA, modeA, W, coefW, modeW, K, out, stream
PyObject *bitplane_gemm(PyObject *const *a) {
    Rows A, W, c;
    int32_t ca[kMaxPlanes], cw[kMaxPlanes], ma, mw;
    int64_t K, s;
    if (!rows_of(a[0], at::kInt, 3, A) || !coefficients(a[1], A.planes, ca) || !integer32(a[2], ma) || !rows_of(a[3], at::kInt, 3, W) ||
        !coefficients(a[4], W.planes, cw) || !integer32(a[5], mw) || !integer(a[6], K) || !rows_of(a[7], at::kInt, 2, c) || !stream(a[8], s))
        return not_here();
    return call([&] {
        return reinterpret_cast<BitplaneGemm>(g_entry[kBitplaneGemm])(as<uint32_t>(A), (int)A.planes, ca, ma, A.ld, A.stride, as<uint32_t>(W), (int)W.planes, cw, mw, W.ld, W.stride,
                                                                      as<int32_t>(c), c.ld, A.rows, W.rows, K, stream_of(s));
    });
}
// A, coefA, modeA, Cin, W, coefW, modeW, pad, stride, out, stream
PyObject *bitplane_conv2d(PyObject *const *a) {
    const at::Tensor *A = tensor(a[0], at::kInt, 5), *W = tensor(a[4], at::kInt, 5), *out = tensor(a[9], at::kInt, 4);
    int32_t ca[kMaxPlanes], cw[kMaxPlanes], ma, mw, pad, step;
    int64_t cin, s;
    if (!A || !W || !out || !A->is_contiguous() || !W->is_contiguous() || !out->is_contiguous() || !coefficients(a[1], A->size(0), ca) || !integer32(a[2], ma) ||
        !integer(a[3], cin) || !coefficients(a[5], W->size(0), cw) || !integer32(a[6], mw) || !integer32(a[7], pad) || !integer32(a[8], step))
        return not_here();
    const int64_t B = A->size(1), H = A->size(2), Wd = A->size(3), Cw = A->size(4), N = W->size(1), KH = W->size(2), KW = W->size(3);
    if (cin < 1 || Cw != (cin + 31) / 32 || W->size(4) != Cw || step < 1 || H + 2 * (int64_t)pad < KH || Wd + 2 * (int64_t)pad < KW || KH > INT32_MAX || KW > INT32_MAX)
        return not_here();
    if (out->size(0) != B || out->size(1) != (H + 2 * (int64_t)pad - KH) / step + 1 || out->size(2) != (Wd + 2 * (int64_t)pad - KW) / step + 1 || out->size(3) != N || !stream(a[10], s)) return not_here();
    const int Pa = (int)A->size(0), Pb = (int)W->size(0);
    const int64_t sa = Pa > 1 ? A->stride(0) : 0, sw = Pb > 1 ? W->stride(0) : 0;
    const uint32_t *const pa = static_cast<const uint32_t *>(A->data_ptr()), *const pw = static_cast<const uint32_t *>(W->data_ptr());
    int32_t *const po = static_cast<int32_t *>(out->data_ptr());
    return call([&] {
        return reinterpret_cast<Conv2d>(g_entry[kConv2d])(pa, Pa, ca, ma, sa, B, H, Wd, cin, pw, Pb, cw, mw, sw, N, (int)KH, (int)KW, pad, step, po, stream_of(s));
    });
}

// (C++ errors, of a tensor that has no memory for instance, are the general path's)
template <PyObject *(*kCall)(PyObject *const *), Py_ssize_t kArgs, int kEntry>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != kArgs || !g_entry[kEntry]) return not_here();
    try {
        return kCall(args);
    } catch (...) {
        return not_here();
    }
}
// The addresses of the entry points, in the order of the enumeration above
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    for (Py_ssize_t i = 0; i < n && i < 6; ++i) {
        g_entry[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_RETURN_NONE;
}

template <typename F>
PyCFunction function(F f) {
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}
PyMethodDef kMethods[] = {
    {"bind", function(bind), METH_FASTCALL, nullptr},
    {"pack_sign", function(entry<pack_sign, 3, kPackSign>), METH_FASTCALL, nullptr},
    {"linear_quant_planes", function(entry<linear_quant_planes, 7, kLinearQuant>), METH_FASTCALL, nullptr},
    {"binary_gemm", function(entry<binary_gemm, 5, kBinaryGemm>), METH_FASTCALL, nullptr},
    {"binary_gemm_sign", function(entry<binary_gemm_sign, 8, kBinaryGemmSign>), METH_FASTCALL, nullptr},
    {"bitplane_gemm", function(entry<bitplane_gemm, 9, kBitplaneGemm>), METH_FASTCALL, nullptr},
    {"bitplane_conv2d", function(entry<bitplane_conv2d, 11, kConv2d>), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// (BUILT_FOR: the torch and Python whose headers this was compiled with; with others, whose classes may be laid out differently, it is not used)
PyMODINIT_FUNC PyInit__native() {
    PyObject *const m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", QNN_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
