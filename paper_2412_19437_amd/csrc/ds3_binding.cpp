// The marshalling of the small calls' hot entry points, in native code: argument
// checks, output tensors from torch's allocator, the current stream, one call of
// the C entry point.  The Python functions of the package keep their signatures
// and defaults and end here.
//
// In Python (ctypes, torch.empty, views, a Stream object) a call took 12-17 us
// of host time, now 4.8 us, most of it the launch: a small layer's pass of three
// calls (256x512x1024, FP32 input) goes from 45-46 to 16-18 us, its kernels being 12 us.
#include <Python.h>
#include <algorithm>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_strided.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/ds3.h"

namespace {

PyObject* g_check = nullptr;                 // _check(status, where): raises
PyObject* g_workspaces = nullptr;            // {(device index, stream): uint8 tensor}
PyObject* g_gemm_workspace = nullptr;        // gemm_workspace(nbytes, device): makes one and keeps it there

[[noreturn]] void fail(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw python_error();
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch.Tensor");
    return THPVariable_Unpack(o);
}

int64_t integer(PyObject* o) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}

bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw python_error();
    return v != 0;
}

// A 2-D tensor with contiguous rows.
struct Mat { int64_t rows, cols, ld; };
Mat rows2d(const at::Tensor& t, const char* name) {
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) {
        PyErr_Format(PyExc_ValueError, "%s must be 2-D with contiguous rows", name);
        throw python_error();
    }
    const int64_t s0 = t.stride(0);
    return {t.size(0), t.size(1), t.size(0) > 1 ? s0 : std::max(t.size(1), s0)};
}

ds3_dtype dtype_of(const at::Tensor& t) {
    if (t.scalar_type() == at::kFloat) return DS3_F32;
    if (t.scalar_type() == at::kBFloat16) return DS3_BF16;
    PyErr_Format(PyExc_TypeError, "unsupported dtype torch.%s", c10::getDtypeNames(t.scalar_type()).first.c_str());
    throw python_error();
}

at::Tensor empty2d(int64_t rows, int64_t cols, int64_t ld, at::ScalarType type, const at::Tensor& like) {
    at::Tensor t = at::empty({rows, ld}, at::TensorOptions().dtype(type).device(like.device()));
    return ld == cols ? t : t.narrow(1, 0, cols);
}
int64_t up(int64_t v, int64_t to) { return (v + to - 1) / to * to; }
int64_t blocks(int64_t v) { return (v + 127) / 128; }

// uint8 [rows][cols], leading dimension padded to a multiple of 16
at::Tensor codes(int64_t rows, int64_t cols, const at::Tensor& like) { return empty2d(rows, cols, up(cols, 16), at::kByte, like); }
// logical [rows][nb] FP32; k_major stores it as [nb][rows]
at::Tensor scales(int64_t rows, int64_t nb, bool k_major, const at::Tensor& like) {
    const auto opt = at::TensorOptions().dtype(at::kFloat).device(like.device());
    return k_major ? at::empty_strided({rows, nb}, {1, std::max<int64_t>(rows, 1)}, opt) : at::empty({rows, nb}, opt);
}
at::Tensor gemm_out(int64_t rows, int64_t cols, at::ScalarType type, const at::Tensor& like) {
    return empty2d(rows, cols, up(cols, 8), type, like);
}

template <typename T = uint8_t> T* ptr(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }
void* stream() { return c10::hip::getCurrentHIPStream(-1).stream(); }

// The interpreter lock is released while one of these exists, and taken again however its scope is left.
struct Unlocked {
    PyThreadState* const save = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(save); }
};

// The C call without the interpreter lock; a status other than DS3_OK is raised by the package.  What the call
// is given (a tensor's pointer and strides may throw) is worked out by the caller, under the lock.
template <typename F, typename... A> void call(const char* where, F* fn, A... args) {
    ds3_status st;
    {
        const Unlocked unlocked;
        st = fn(args...);
    }
    if (st == DS3_OK) return;
    PyObject* r = PyObject_CallFunction(g_check, "is", (int)st, where);
    Py_XDECREF(r);
    throw python_error();
}

PyObject* pair(const at::Tensor& q, const at::Tensor& s) {
    PyObject* a = THPVariable_Wrap(q);
    PyObject* b = a ? THPVariable_Wrap(s) : nullptr;
    PyObject* t = b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return t;
}

void need(Py_ssize_t n, Py_ssize_t want) {
    if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
}

// `workspace` of the GEMM calls: "auto" (the kept one of this device and stream), None or a tensor.
struct Workspace { void* p = nullptr; size_t n = 0; at::Tensor hold; };
Workspace workspace_of(PyObject* o, size_t nbytes, PyObject* a_obj, const at::Tensor& a, void* st) {
    Workspace w;
    if (o == Py_None) return w;
    if (PyUnicode_Check(o)) {
        if (nbytes == 0) return w;
        const int64_t index = a.device().has_index() ? a.device().index() : 0;
        PyObject* key = Py_BuildValue("(LK)", (long long)index, (unsigned long long)reinterpret_cast<uintptr_t>(st));
        if (!key) throw python_error();
        PyObject* kept = PyDict_GetItemWithError(g_workspaces, key);      // borrowed
        Py_DECREF(key);
        if (!kept && PyErr_Occurred()) throw python_error();
        if (kept) w.hold = tensor(kept);
        if (!kept || (size_t)w.hold.numel() < nbytes) {
            PyObject* dev = PyObject_GetAttrString(a_obj, "device");
            PyObject* made = dev ? PyObject_CallFunction(g_gemm_workspace, "KO", (unsigned long long)nbytes, dev) : nullptr;
            Py_XDECREF(dev);
            if (!made) throw python_error();
            w.hold = THPVariable_Check(made) ? THPVariable_Unpack(made) : at::Tensor();
            Py_DECREF(made);
        }
    } else {
        w.hold = tensor(o);
    }
    if (w.hold.defined()) { w.p = w.hold.data_ptr(); w.n = (size_t)w.hold.numel(); }
    return w;
}

// (x, k_major_scales, pow2) -> (codes, scales)
PyObject* quant_act_1x128(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 3);
    const at::Tensor& x = tensor(o[0]);
    const bool km = truth(o[1]), p2 = truth(o[2]);
    const Mat m = rows2d(x, "x");
    const at::Tensor q = codes(m.rows, m.cols, x), s = scales(m.rows, blocks(m.cols), km, x);
    const ds3_dtype t = dtype_of(x);
    void* st = stream();
    call(p2 ? "ds3_quant_act_1x128_pow2" : "ds3_quant_act_1x128", p2 ? ds3_quant_act_1x128_pow2 : ds3_quant_act_1x128,
         ptr(x), t, m.rows, m.cols, m.ld, ptr(q), up(m.cols, 16), ptr<float>(s), s.stride(0), s.stride(1), st);
    return pair(q, s);
    END_HANDLE_TH_ERRORS
}

// (x, k_major_scales, pow2) -> (codes of the transpose, scales)
PyObject* quant_act_128x1(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 3);
    const at::Tensor& x = tensor(o[0]);
    const bool km = truth(o[1]), p2 = truth(o[2]);
    const Mat m = rows2d(x, "x");
    const at::Tensor q = codes(m.cols, m.rows, x), s = scales(m.cols, blocks(m.rows), km, x);
    const ds3_dtype t = dtype_of(x);
    void* st = stream();
    call(p2 ? "ds3_quant_act_128x1_pow2" : "ds3_quant_act_128x1", p2 ? ds3_quant_act_128x1_pow2 : ds3_quant_act_128x1,
         ptr(x), t, m.rows, m.cols, m.ld, ptr(q), up(m.rows, 16), ptr<float>(s), s.stride(0), s.stride(1), st);
    return pair(q, s);
    END_HANDLE_TH_ERRORS
}

// (w, pow2) -> (codes, scales)
PyObject* quant_w_128x128(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 2);
    const at::Tensor& w = tensor(o[0]);
    const bool p2 = truth(o[1]);
    const Mat m = rows2d(w, "w");
    const at::Tensor q = codes(m.rows, m.cols, w), s = scales(blocks(m.rows), blocks(m.cols), false, w);
    const ds3_dtype t = dtype_of(w);
    void* st = stream();
    call(p2 ? "ds3_quant_w_128x128_pow2" : "ds3_quant_w_128x128", p2 ? ds3_quant_w_128x128_pow2 : ds3_quant_w_128x128,
         ptr(w), t, m.rows, m.cols, m.ld, ptr(q), up(m.cols, 16), ptr<float>(s), st);
    return pair(q, s);
    END_HANDLE_TH_ERRORS
}

// (w, pow2) -> (codes, scales, codes of the transpose, its scales)
PyObject* quant_w_128x128_dual(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 2);
    const at::Tensor& w = tensor(o[0]);
    const bool p2 = truth(o[1]);
    const Mat m = rows2d(w, "w");
    const at::Tensor q = codes(m.rows, m.cols, w), qt = codes(m.cols, m.rows, w);
    const at::Tensor s = scales(blocks(m.rows), blocks(m.cols), false, w), s_t = scales(blocks(m.cols), blocks(m.rows), false, w);
    const ds3_dtype t = dtype_of(w);
    void* st = stream();
    call(p2 ? "ds3_quant_w_128x128_dual_pow2" : "ds3_quant_w_128x128_dual",
         p2 ? ds3_quant_w_128x128_dual_pow2 : ds3_quant_w_128x128_dual,
         ptr(w), t, m.rows, m.cols, m.ld, ptr(q), up(m.cols, 16), ptr<float>(s), ptr(qt), up(m.rows, 16), ptr<float>(s_t), st);
    PyObject* a = pair(q, s);
    PyObject* b = a ? pair(qt, s_t) : nullptr;
    PyObject* r = b ? PySequence_Concat(a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return r;
    END_HANDLE_TH_ERRORS
}

// (h, k_major_scales, pow2) -> (codes, scales)
PyObject* swiglu_quant_1x128(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 3);
    const at::Tensor& h = tensor(o[0]);
    const bool km = truth(o[1]), p2 = truth(o[2]);
    const Mat m = rows2d(h, "h");
    if (h.scalar_type() != at::kBFloat16 || m.cols % 2) fail(PyExc_TypeError, "h must be BF16 with an even number of columns");
    const int64_t inter = m.cols / 2;
    const at::Tensor q = codes(m.rows, inter, h), s = scales(m.rows, blocks(inter), km, h);
    void* st = stream();
    call(p2 ? "ds3_swiglu_quant_1x128_pow2" : "ds3_swiglu_quant_1x128", p2 ? ds3_swiglu_quant_1x128_pow2 : ds3_swiglu_quant_1x128,
         ptr(h), m.rows, inter, m.ld, ptr(q), up(inter, 16), ptr<float>(s), s.stride(0), s.stride(1), st);
    return pair(q, s);
    END_HANDLE_TH_ERRORS
}

// (x, gamma, eps, want_y, k_major_scales, pow2) -> (codes, scales[, y])
PyObject* rmsnorm_quant_1x128(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 6);
    const at::Tensor &x = tensor(o[0]), &gamma = tensor(o[1]);
    const double eps = PyFloat_AsDouble(o[2]);
    if (eps == -1.0 && PyErr_Occurred()) throw python_error();
    const bool want_y = truth(o[3]), km = truth(o[4]), p2 = truth(o[5]);
    const Mat m = rows2d(x, "x");
    if (x.scalar_type() != at::kBFloat16 || gamma.scalar_type() != at::kFloat || gamma.numel() != m.cols || !gamma.is_contiguous())
        fail(PyExc_TypeError, "x must be BF16 and gamma a contiguous FP32 vector of x's width");
    const at::Tensor q = codes(m.rows, m.cols, x), s = scales(m.rows, blocks(m.cols), km, x);
    const at::Tensor y = want_y ? empty2d(m.rows, m.cols, m.cols, at::kBFloat16, x) : at::Tensor();
    void* st = stream();
    call(p2 ? "ds3_rmsnorm_quant_1x128_pow2" : "ds3_rmsnorm_quant_1x128",
         p2 ? ds3_rmsnorm_quant_1x128_pow2 : ds3_rmsnorm_quant_1x128,
         ptr(x), m.rows, m.cols, m.ld, ptr<float>(gamma), (float)eps, want_y ? y.data_ptr() : nullptr, m.cols, ptr(q),
         up(m.cols, 16), ptr<float>(s), s.stride(0), s.stride(1), st);
    PyObject* r = pair(q, s);
    if (!r || !want_y) return r;
    PyObject* yo = THPVariable_Wrap(y);
    PyObject* one = yo ? PyTuple_Pack(1, yo) : nullptr;
    PyObject* all = one ? PySequence_Concat(r, one) : nullptr;
    Py_XDECREF(yo);
    Py_XDECREF(one);
    Py_DECREF(r);
    return all;
    END_HANDLE_TH_ERRORS
}

// (q, s, k_major_scales, pow2) -> (codes of the transpose, scales)
PyObject* retile(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 4);
    const at::Tensor &q = tensor(o[0]), &s = tensor(o[1]);
    const bool km = truth(o[2]), p2 = truth(o[3]);
    const Mat m = rows2d(q, "q");
    if (q.scalar_type() != at::kByte || s.scalar_type() != at::kFloat || s.dim() != 2 || s.size(0) != m.rows || s.size(1) != blocks(m.cols))
        fail(PyExc_ValueError, "q: uint8 [T][C]; s: float32 logical [T][ceil(C/128)]");
    const at::Tensor qt = codes(m.cols, m.rows, q), s_t = scales(m.cols, blocks(m.rows), km, q);
    void* st = stream();
    call(p2 ? "ds3_retile_1x128_to_128x1_pow2" : "ds3_retile_1x128_to_128x1",
         p2 ? ds3_retile_1x128_to_128x1_pow2 : ds3_retile_1x128_to_128x1,
         ptr(q), m.rows, m.cols, m.ld, ptr<float>(s), s.stride(0), s.stride(1), ptr(qt), up(m.rows, 16), ptr<float>(s_t),
         s_t.stride(0), s_t.stride(1), st);
    return pair(qt, s_t);
    END_HANDLE_TH_ERRORS
}

// (x, k_major_scales) -> (packed codes, scales)
PyObject* quant_act_1x128_e5m6(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 2);
    const at::Tensor& x = tensor(o[0]);
    const bool km = truth(o[1]);
    const Mat m = rows2d(x, "x");
    if (x.scalar_type() != at::kBFloat16) fail(PyExc_TypeError, "x must be BF16");
    const int64_t width = m.cols * 3 / 2;
    const at::Tensor q = empty2d(m.rows, width, width, at::kByte, x), s = scales(m.rows, blocks(m.cols), km, x);
    void* st = stream();
    call("ds3_quant_act_1x128_e5m6", ds3_quant_act_1x128_e5m6,
         ptr(x), m.rows, m.cols, m.ld, ptr(q), width, ptr<float>(s), s.stride(0), s.stride(1), st);
    return pair(q, s);
    END_HANDLE_TH_ERRORS
}

// (a, sa, b, sb, sb_mode, f32_out, c or None, accumulate, variant, workspace, pow2) -> c
PyObject* gemm(PyObject*, PyObject* const* o, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    need(n, 11);
    const at::Tensor &a = tensor(o[0]), &sa = tensor(o[1]), &b = tensor(o[2]), &sb = tensor(o[3]);
    const int64_t sb_mode = integer(o[4]), accumulate = integer(o[7]), variant = integer(o[8]);
    const bool f32 = truth(o[5]), p2 = truth(o[10]);
    const Mat ma = rows2d(a, "a"), mb = rows2d(b, "b");
    if (ma.cols != mb.cols) fail(PyExc_ValueError, "a and b disagree on K");
    at::Tensor c = o[6] == Py_None ? gemm_out(ma.rows, mb.rows, f32 ? at::kFloat : at::kBFloat16, a) : tensor(o[6]);
    const Mat mc = rows2d(c, "c");
    const int64_t sar = sa.stride(0), sak = sa.stride(1), sbr = sb.stride(0), sbk = sb.stride(1);     // (fewer than two: an IndexError)
    void* st = stream();
    const size_t bytes = PyUnicode_Check(o[9])
                             ? ds3_gemm_workspace_bytes_v((int)variant, ma.rows, mb.rows, ma.cols, (ds3_bscale)sb_mode) : 0;
    const Workspace w = workspace_of(o[9], bytes, o[0], a, st);
    const ds3_dtype ct = dtype_of(c);
    call(p2 ? "ds3_gemm_fp8_bs_pow2" : "ds3_gemm_fp8_bs_v", p2 ? ds3_gemm_fp8_bs_pow2 : ds3_gemm_fp8_bs_v,
         (int)variant, ma.rows, mb.rows, ma.cols, ptr(a), ma.ld, ptr<float>(sa), sar, sak, ptr(b), mb.ld,
         ptr<float>(sb), sbr, sbk, (ds3_bscale)sb_mode, c.data_ptr(), ct, mc.ld, (int)accumulate, w.p, w.n, st);
    if (o[6] == Py_None) return THPVariable_Wrap(c);
    Py_INCREF(o[6]);
    return o[6];
    END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {
#define M(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
    M(quant_act_1x128), M(quant_act_128x1), M(quant_w_128x128), M(quant_w_128x128_dual), M(swiglu_quant_1x128), M(rmsnorm_quant_1x128), M(retile),
    M(quant_act_1x128_e5m6), M(gemm),
#undef M
    {"init", [](PyObject*, PyObject* args) -> PyObject* {
         PyObject *check, *kept, *make;
         if (!PyArg_ParseTuple(args, "OO!O", &check, &PyDict_Type, &kept, &make)) return nullptr;
         Py_INCREF(check); Py_INCREF(kept); Py_INCREF(make);
         g_check = check; g_workspaces = kept; g_gemm_workspace = make;
         Py_RETURN_NONE;
     }, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "ds3_native", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_ds3_native() { return PyModule_Create(&kModule); }
