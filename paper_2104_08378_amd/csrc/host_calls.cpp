// The calls of the Python binding, marshalled natively: a small product is over in 5 us of which the launch itself
// takes 3.5, and forming the arguments in Python -- a dozen attribute reads and integer conversions through ctypes --
// took another 3 (measured on 256 x 256 x 256: 8.5 us a call in Python, 5.4 from here).
//
// Every function takes the arguments of the sp24.py function of the same name, in its order, positionally.  It handles
// the call when everything about it is as documented and returns the result; when anything is not -- a wrong type,
// shape, stride or device, or a status of the library's own checks, all of which come before any launch -- it returns
// None, and the Python code behind it goes through the same call step by step and raises what is to be raised.
// SP24_ERR_LAUNCH may come after a launch (an error that the runtime held from before the call; the second kernel of a
// split product): it is raised from here, so that no call is made twice and no error is lost.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sp24.h"

namespace {

// One call's view of its arguments; ok turns false with the first that is not as documented.
struct Call {
    PyObject* const* args;
    bool ok;

    const at::Tensor* tensor(int i)
    {
        PyObject* o = args[i];
        if (!ok || !THPVariable_Check(o)) return fail();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda()) return fail();
        return &t;
    }
    const at::Tensor* fail()
    {
        ok = false;
        return nullptr;
    }
    bool none(int i) const { return args[i] == Py_None; }
    void require(bool cond) { ok = ok && cond; }

    // two-dimensional, unit stride along a row (the stride of a dimension of size 1 means nothing)
    const at::Tensor* rowmajor(int i)
    {
        const at::Tensor* t = tensor(i);
        if (!ok || t->dim() != 2 || (t->stride(1) != 1 && t->size(1) > 1)) return fail();
        return t;
    }
    // contiguous, any shape
    const at::Tensor* contiguous(int i)
    {
        const at::Tensor* t = tensor(i);
        if (!ok || !t->is_contiguous()) return fail();
        return t;
    }
    bool text_is(int i, const char* s)
    {
        PyObject* o = args[i];
        return PyUnicode_Check(o) && PyUnicode_CompareWithASCIIString(o, s) == 0;
    }
    sp24_layout layout(int i)
    {
        if (text_is(i, "tiled")) return SP24_LAYOUT_TILED;
        require(text_is(i, "canonical"));
        return SP24_LAYOUT_CANONICAL;
    }
    sp24_border border(int i)
    {
        if (text_is(i, "k")) return SP24_B_KMAJOR;
        require(text_is(i, "n"));
        return SP24_B_NMAJOR;
    }
    at::ScalarType dtype(int i)
    {
        if (!THPDtype_Check(args[i])) {
            ok = false;
            return at::kFloat;
        }
        return reinterpret_cast<THPDtype*>(args[i])->scalar_type;
    }
    int64_t integer(int i)
    {
        if (!PyLong_Check(args[i])) {
            ok = false;
            return 0;
        }
        const long long v = PyLong_AsLongLong(args[i]);
        if (v == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return v;
    }
    float real(int i)
    {
        const double v = PyFloat_AsDouble(args[i]);
        if (v == -1.0 && PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return (float)v;
    }
    int truth(int i)
    {
        const int v = PyObject_IsTrue(args[i]);
        if (v < 0) {
            PyErr_Clear();
            ok = false;
        }
        return v > 0;
    }
    // a pair of integers
    void pair(int i, int& a, int& b)
    {
        PyObject* o = args[i];
        if (!PyTuple_Check(o) || PyTuple_GET_SIZE(o) != 2 || !PyLong_Check(PyTuple_GET_ITEM(o, 0)) || !PyLong_Check(PyTuple_GET_ITEM(o, 1))) {
            ok = false;
            return;
        }
        const long x = PyLong_AsLong(PyTuple_GET_ITEM(o, 0)), y = PyLong_AsLong(PyTuple_GET_ITEM(o, 1));
        if (PyErr_Occurred()) {                        // past a long
            PyErr_Clear();
            ok = false;
        }
        require(x >= 0 && x <= 4096 && y >= 0 && y <= 4096);
        a = (int)x;
        b = (int)y;
    }
    // float32 vector with one entry per row
    const float* row_vector(int i, int64_t M)
    {
        const at::Tensor* t = contiguous(i);
        if (!ok) return nullptr;
        require(t->scalar_type() == at::kFloat && t->numel() == M);
        return static_cast<const float*>(t->data_ptr());
    }
};

sp24_dtype type_of(at::ScalarType t, bool& ok)
{
    switch (t) {
    case at::kHalf: return SP24_F16;
    case at::kBFloat16: return SP24_BF16;
    case at::kChar: return SP24_I8;
    case at::kFloat: return SP24_F32;
    case at::kInt: return SP24_I32;
    case at::kFloat8_e4m3fn: return SP24_F8;
    default: ok = false; return SP24_F32;
    }
}

bool is_input(at::ScalarType t) { return t == at::kHalf || t == at::kBFloat16 || t == at::kChar || t == at::kFloat8_e4m3fn; }

// leading dimension of a row-major matrix; a single row may carry any stride
int64_t ld(const at::Tensor& t) { return t.size(0) > 1 ? t.stride(0) : std::max(t.stride(0), t.size(1)); }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The result: a new tensor, or the caller's (argument i), which must have exactly the result's shape and type.
struct Result {
    at::Tensor fresh;
    const at::Tensor* t = nullptr;
    PyObject* given = nullptr;
    Result(Call& c, int i, at::IntArrayRef shape, at::ScalarType type, const at::Tensor* like)
    {
        if (!c.ok) return;
        if (c.none(i)) {
            fresh = at::empty(shape, at::TensorOptions().dtype(type).device(like->device()));
            t = &fresh;
            return;
        }
        t = c.rowmajor(i);
        if (!c.ok) return;
        c.require(t->sizes() == shape && t->scalar_type() == type);
        given = c.args[i];
    }
    PyObject* object()
    {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(std::move(fresh));
    }
};

template <typename F>
sp24_status without_gil(F&& f)
{
    PyThreadState* state = PyEval_SaveThread();
    const sp24_status s = f();
    PyEval_RestoreThread(state);
    return s;
}

PyObject* not_handled() { Py_RETURN_NONE; }

// What a status other than SP24_OK comes to.  (module: this one, which holds sp24.py's exception as Sp24Error.)
PyObject* refused(PyObject* module, sp24_status s, const char* where)
{
    if (s != SP24_ERR_LAUNCH) return not_handled();
    PyObject* type = PyObject_GetAttrString(module, "Sp24Error");
    if (!type) return nullptr;
    if (PyObject* error = PyObject_CallFunction(type, "is", (int)s, where)) {
        PyErr_SetObject(type, error);
        Py_DECREF(error);
    }
    Py_DECREF(type);
    return nullptr;
}

// First operand of a product: the compressed pair (arguments 0 and 1) or a dense matrix (argument 0).
struct FirstOperand {
    const at::Tensor* A = nullptr;
    const at::Tensor* meta = nullptr;
    int64_t M = 0, K = 0, lda = 0;
    FirstOperand(Call& c, bool sparse)
    {
        if (sparse) {
            A = c.contiguous(0);
            meta = c.contiguous(1);
            if (!c.ok) return;
            c.require(A->dim() == 2 && is_input(A->scalar_type()));
            if (!c.ok) return;
            M = A->size(0);
            K = A->size(1) * 2;
            c.require(meta->numel() * (int64_t)meta->element_size() == M * (K / 8));
        } else {
            A = c.rowmajor(0);
            if (!c.ok) return;
            M = A->size(0);
            K = A->size(1);
            lda = A->stride(0);
        }
    }
};

// Second operand of a plain product
struct SecondOperand {
    const at::Tensor* B = nullptr;
    int64_t N = 0, ldb = 0;
    sp24_border order = SP24_B_KMAJOR;
    SecondOperand(Call& c, int i, int i_order, const FirstOperand& a)
    {
        B = c.rowmajor(i);
        order = c.border(i_order);
        if (!c.ok) return;
        N = B->size(order == SP24_B_KMAJOR ? 0 : 1);
        c.require(B->size(order == SP24_B_KMAJOR ? 1 : 0) == a.K && B->scalar_type() == a.A->scalar_type());
        ldb = ld(*B);
    }
};

// (V, meta, B, out_dtype, b_order, layout, out) / dense: (A, B, out_dtype, b_order, out)
template <bool SPARSE>
PyObject* product(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    constexpr int b = SPARSE ? 2 : 1;
    Call c{args, true};
    FirstOperand a(c, SPARSE);
    SecondOperand x(c, b, b + 2, a);
    const at::ScalarType out = c.dtype(b + 1);
    const sp24_layout l = SPARSE ? c.layout(b + 3) : SP24_LAYOUT_CANONICAL;
    if (!c.ok) return not_handled();
    const int64_t shape[2] = {a.M, x.N};
    Result r(c, SPARSE ? b + 4 : b + 3, shape, out, a.A);
    if (!c.ok) return not_handled();
    const sp24_dtype ti = type_of(a.A->scalar_type(), c.ok), to = type_of(out, c.ok);
    if (!c.ok) return not_handled();
    const void *pa = a.A->data_ptr(), *pm = SPARSE ? a.meta->data_ptr() : nullptr, *pb = x.B->data_ptr();
    void *pd = r.t->data_ptr(), *st = stream();
    const int64_t ldd = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return SPARSE ? sp24_spmm(pa, pm, pb, pd, a.M, x.N, a.K, x.ldb, ldd, ti, to, x.order, l, st)
                      : sp24_gemm_dense(pa, pb, pd, a.M, x.N, a.K, a.lda, x.ldb, ldd, ti, to, x.order, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, SPARSE ? "sp24_spmm" : "sp24_gemm_dense");
}

// (V, meta, B, out_dtype, b_order, layout, workspace, out) / dense: (A, B, out_dtype, b_order, workspace, out)
template <bool SPARSE>
PyObject* product_splitk(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    constexpr int b = SPARSE ? 2 : 1, w = SPARSE ? b + 4 : b + 3;
    Call c{args, true};
    FirstOperand a(c, SPARSE);
    SecondOperand x(c, b, b + 2, a);
    const at::ScalarType out = c.dtype(b + 1);
    const sp24_layout l = SPARSE ? c.layout(b + 3) : SP24_LAYOUT_CANONICAL;
    if (!c.ok) return not_handled();
    const sp24_dtype ti = type_of(a.A->scalar_type(), c.ok), to = type_of(out, c.ok);
    at::Tensor own;
    const at::Tensor* ws = nullptr;
    if (c.ok && c.none(w)) {
        const int64_t need = (int64_t)sp24_splitk_workspace_bytes(a.M, x.N, a.K, ti);
        own = at::empty({std::max<int64_t>(need, 16)}, at::TensorOptions().dtype(at::kByte).device(a.A->device()));
        ws = &own;
    } else ws = c.contiguous(w);
    if (!c.ok) return not_handled();
    const int64_t shape[2] = {a.M, x.N};
    Result r(c, w + 1, shape, out, a.A);
    if (!c.ok) return not_handled();
    const void *pa = a.A->data_ptr(), *pm = SPARSE ? a.meta->data_ptr() : nullptr, *pb = x.B->data_ptr();
    void *pd = r.t->data_ptr(), *pw = ws->data_ptr(), *st = stream();
    const size_t bytes = (size_t)ws->numel() * ws->element_size();
    const int64_t ldd = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return SPARSE ? sp24_spmm_splitk(pa, pm, pb, pd, a.M, x.N, a.K, x.ldb, ldd, ti, to, x.order, l, pw, bytes, st)
                      : sp24_gemm_dense_splitk(pa, pb, pd, a.M, x.N, a.K, a.lda, x.ldb, ldd, ti, to, x.order, pw, bytes, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, SPARSE ? "sp24_spmm_splitk" : "sp24_gemm_dense_splitk");
}

// (V, meta, B, out_dtype, w_scale, x_scale, bias, relu, inv_y_scale, b_order, layout, out) / dense: (A, B, ... b_order, out)
template <bool SPARSE>
PyObject* product_scaled(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    constexpr int b = SPARSE ? 2 : 1, e = b + 2, o = e + 5;
    Call c{args, true};
    FirstOperand a(c, SPARSE);
    SecondOperand x(c, b, o, a);
    const at::ScalarType out = c.dtype(b + 1);
    const sp24_layout l = SPARSE ? c.layout(o + 1) : SP24_LAYOUT_CANONICAL;
    const float* ws = c.row_vector(e, a.M);
    const float xs = c.real(e + 1), iy = c.real(e + 4);
    const float* bias = c.none(e + 2) ? nullptr : c.row_vector(e + 2, a.M);
    const int relu = c.truth(e + 3);
    if (!c.ok) return not_handled();
    const sp24_dtype to = type_of(out, c.ok);
    c.require(a.A->scalar_type() == at::kChar);
    const int64_t shape[2] = {a.M, x.N};
    Result r(c, SPARSE ? o + 2 : o + 1, shape, out, a.A);
    if (!c.ok) return not_handled();
    const void *pa = a.A->data_ptr(), *pm = SPARSE ? a.meta->data_ptr() : nullptr, *pb = x.B->data_ptr();
    void *pd = r.t->data_ptr(), *st = stream();
    const int64_t ldd = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return SPARSE ? sp24_spmm_i8_scaled(pa, pm, pb, pd, a.M, x.N, a.K, x.ldb, ldd, ws, xs, bias, relu, iy, to, x.order, l, st)
                      : sp24_gemm_dense_i8_scaled(pa, pb, pd, a.M, x.N, a.K, a.lda, x.ldb, ldd, ws, xs, bias, relu, iy, to, x.order, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, SPARSE ? "sp24_spmm_i8_scaled" : "sp24_gemm_dense_i8_scaled");
}

// Input and geometry of a convolution: X at argument i, R and S at i + 2 and i + 3, pad and stride at p and p + 1
struct ConvInput {
    const at::Tensor* X = nullptr;
    int64_t n = 0, H = 0, W = 0, C = 0, N = 0;
    int R = 0, S = 0, ph = 0, pw = 0, sh = 0, sw = 0;
    ConvInput(Call& c, int i, int p, const FirstOperand& a)
    {
        X = c.contiguous(i);
        const int64_t r = c.integer(i + 2), s = c.integer(i + 3);
        c.pair(p, ph, pw);
        c.pair(p + 1, sh, sw);
        if (!c.ok) return;
        c.require(X->dim() == 4 && X->scalar_type() == a.A->scalar_type() && r > 0 && r <= 4096 && s > 0 && s <= 4096 && sh > 0 && sw > 0);
        if (!c.ok) return;
        n = X->size(0);
        H = X->size(1);
        W = X->size(2);
        C = X->size(3);
        R = (int)r;
        S = (int)s;
        c.require(a.K == r * s * C && H + 2 * ph >= R && W + 2 * pw >= S);
        if (!c.ok) return;
        N = n * ((H + 2 * ph - R) / sh + 1) * ((W + 2 * pw - S) / sw + 1);
    }
};

// (V, meta, X, out_dtype, R, S, pad, stride, layout, out) / dense: (A, X, ..., stride, out)
template <bool SPARSE>
PyObject* conv(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    constexpr int i = SPARSE ? 2 : 1, p = i + 4;
    Call c{args, true};
    FirstOperand a(c, SPARSE);
    if (!c.ok) return not_handled();
    ConvInput x(c, i, p, a);
    const at::ScalarType out = c.dtype(i + 1);
    const sp24_layout l = SPARSE ? c.layout(p + 2) : SP24_LAYOUT_CANONICAL;
    if (!c.ok) return not_handled();
    const sp24_dtype ti = type_of(a.A->scalar_type(), c.ok), to = type_of(out, c.ok);
    const int64_t shape[2] = {a.M, x.N};
    Result r(c, SPARSE ? p + 3 : p + 2, shape, out, a.A);
    if (!c.ok) return not_handled();
    const void *pa = a.A->data_ptr(), *pm = SPARSE ? a.meta->data_ptr() : nullptr, *px = x.X->data_ptr();
    void *pd = r.t->data_ptr(), *st = stream();
    const int64_t ldd = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return SPARSE ? sp24_spmm_conv2d(pa, pm, px, pd, a.M, x.n, x.H, x.W, x.C, x.R, x.S, x.ph, x.pw, x.sh, x.sw, ldd, ti, to, l, st)
                      : sp24_conv2d_dense(pa, px, pd, a.M, x.n, x.H, x.W, x.C, x.R, x.S, x.ph, x.pw, x.sh, x.sw, a.lda, ldd, ti, to, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, SPARSE ? "sp24_spmm_conv2d" : "sp24_conv2d_dense");
}

// (V, meta, X, out_dtype, R, S, w_scale, x_scale, bias, relu, inv_y_scale, pad, stride, layout, out) / dense: (A, X, ..., stride, out)
template <bool SPARSE>
PyObject* conv_scaled(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    constexpr int i = SPARSE ? 2 : 1, e = i + 4, p = e + 5;
    Call c{args, true};
    FirstOperand a(c, SPARSE);
    if (!c.ok) return not_handled();
    ConvInput x(c, i, p, a);
    const at::ScalarType out = c.dtype(i + 1);
    const sp24_layout l = SPARSE ? c.layout(p + 2) : SP24_LAYOUT_CANONICAL;
    const float* ws = c.row_vector(e, a.M);
    const float xs = c.real(e + 1), iy = c.real(e + 4);
    const float* bias = c.none(e + 2) ? nullptr : c.row_vector(e + 2, a.M);
    const int relu = c.truth(e + 3);
    if (!c.ok) return not_handled();
    const sp24_dtype to = type_of(out, c.ok);
    c.require(a.A->scalar_type() == at::kChar);
    const int64_t shape[2] = {a.M, x.N};
    Result r(c, SPARSE ? p + 3 : p + 2, shape, out, a.A);
    if (!c.ok) return not_handled();
    const void *pa = a.A->data_ptr(), *pm = SPARSE ? a.meta->data_ptr() : nullptr, *px = x.X->data_ptr();
    void *pd = r.t->data_ptr(), *st = stream();
    const int64_t ldd = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return SPARSE ? sp24_spmm_conv2d_i8_scaled(pa, pm, px, pd, a.M, x.n, x.H, x.W, x.C, x.R, x.S, x.ph, x.pw, x.sh, x.sw, ldd, ws, xs, bias, relu, iy, to, l, st)
                      : sp24_conv2d_dense_i8_scaled(pa, px, pd, a.M, x.n, x.H, x.W, x.C, x.R, x.S, x.ph, x.pw, x.sh, x.sw, a.lda, ldd, ws, xs, bias, relu, iy, to, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, SPARSE ? "sp24_spmm_conv2d_i8_scaled" : "sp24_conv2d_dense_i8_scaled");
}

// (A, out) -> a matrix of A's shape and type
template <sp24_status (*OP)(const void*, void*, int64_t, int64_t, int64_t, int64_t, sp24_dtype, void*)>
PyObject* same_shape(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    Call c{args, true};
    const at::Tensor* A = c.rowmajor(0);
    if (!c.ok) return not_handled();
    const sp24_dtype t = type_of(A->scalar_type(), c.ok);
    const int64_t M = A->size(0), K = A->size(1), lda = A->stride(0);
    Result r(c, 1, A->sizes(), A->scalar_type(), A);
    if (!c.ok) return not_handled();
    const void* pa = A->data_ptr();
    void *pp = r.t->data_ptr(), *st = stream();
    const int64_t ldp = r.t->stride(0);
    const sp24_status s = without_gil([&] { return OP(pa, pp, M, K, lda, ldp, t, st); });
    return s == SP24_OK ? r.object() : refused(self, s, OP == sp24_prune ? "sp24_prune" : "sp24_prune_transposable");
}

// (A, layout, out): out None only -- a pair of new tensors
PyObject* compress(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    Call c{args, true};
    const at::Tensor* A = c.rowmajor(0);
    const sp24_layout l = c.layout(1);
    c.require(c.none(2));
    if (!c.ok) return not_handled();
    const sp24_dtype t = type_of(A->scalar_type(), c.ok);
    if (!c.ok) return not_handled();
    const int64_t M = A->size(0), K = A->size(1), lda = A->stride(0);
    at::Tensor V = at::empty({M, K / 2}, at::TensorOptions().dtype(A->scalar_type()).device(A->device()));
    at::Tensor meta = at::empty({M, K / 8}, at::TensorOptions().dtype(at::kByte).device(A->device()));
    const void* pa = A->data_ptr();
    void *pv = V.data_ptr(), *pm = meta.data_ptr(), *st = stream();
    const sp24_status s = without_gil([&] { return sp24_compress(pa, pv, pm, M, K, lda, t, l, st); });
    if (s != SP24_OK) return refused(self, s, "sp24_compress");
    PyObject* pair = PyTuple_New(2);
    if (!pair) return nullptr;
    PyTuple_SET_ITEM(pair, 0, THPVariable_Wrap(std::move(V)));
    PyTuple_SET_ITEM(pair, 1, THPVariable_Wrap(std::move(meta)));
    return pair;
}

// (V, meta, layout, out)
PyObject* decompress(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    Call c{args, true};
    FirstOperand a(c, true);
    const sp24_layout l = c.layout(2);
    if (!c.ok) return not_handled();
    const sp24_dtype t = type_of(a.A->scalar_type(), c.ok);
    const int64_t shape[2] = {a.M, a.K};
    Result r(c, 3, shape, a.A->scalar_type(), a.A);
    if (!c.ok) return not_handled();
    const void *pv = a.A->data_ptr(), *pm = a.meta->data_ptr();
    void *pp = r.t->data_ptr(), *st = stream();
    const int64_t ldp = r.t->stride(0);
    const sp24_status s = without_gil([&] { return sp24_decompress(pv, pm, pp, a.M, a.K, ldp, t, l, st); });
    return s == SP24_OK ? r.object() : refused(self, s, "sp24_decompress");
}

// (W, meta, layout, out): the masked matrix, or (VALUES) its compressed values -- for those out None only
template <bool VALUES>
PyObject* masked(PyObject* self, PyObject* const* args, Py_ssize_t)
{
    Call c{args, true};
    const at::Tensor* W = c.rowmajor(0);
    const at::Tensor* meta = c.contiguous(1);
    const sp24_layout l = c.layout(2);
    c.require(!VALUES || c.none(3));
    if (!c.ok) return not_handled();
    const sp24_dtype t = type_of(W->scalar_type(), c.ok);
    const int64_t M = W->size(0), K = W->size(1), ldw = W->stride(0);
    c.require(meta->numel() * (int64_t)meta->element_size() == M * (K / 8));
    const int64_t shape[2] = {M, VALUES ? K / 2 : K};
    Result r(c, 3, shape, W->scalar_type(), W);
    if (!c.ok) return not_handled();
    const void *pw = W->data_ptr(), *pm = meta->data_ptr();
    void *pp = r.t->data_ptr(), *st = stream();
    const int64_t ldp = r.t->stride(0);
    const sp24_status s = without_gil([&] {
        return VALUES ? sp24_compress_masked(pw, pm, pp, M, K, ldw, t, l, st) : sp24_mask_apply(pw, pm, pp, M, K, ldw, ldp, t, l, st);
    });
    return s == SP24_OK ? r.object() : refused(self, s, VALUES ? "sp24_compress_masked" : "sp24_mask_apply");
}

// No exception of torch's (an allocation that fails) crosses into the interpreter: the Python code meets it again.
using Fn = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
template <Fn F>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n)
{
    try {
        return F(self, args, n);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

#define SP24_METHOD(name, ...) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(static_cast<Fn>(guarded<__VA_ARGS__>))), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SP24_METHOD("sp24_spmm", product<true>),
    SP24_METHOD("sp24_gemm_dense", product<false>),
    SP24_METHOD("sp24_spmm_splitk", product_splitk<true>),
    SP24_METHOD("sp24_gemm_dense_splitk", product_splitk<false>),
    SP24_METHOD("sp24_spmm_i8_scaled", product_scaled<true>),
    SP24_METHOD("sp24_gemm_dense_i8_scaled", product_scaled<false>),
    SP24_METHOD("sp24_spmm_conv2d", conv<true>),
    SP24_METHOD("sp24_conv2d_dense", conv<false>),
    SP24_METHOD("sp24_spmm_conv2d_i8_scaled", conv_scaled<true>),
    SP24_METHOD("sp24_conv2d_dense_i8_scaled", conv_scaled<false>),
    SP24_METHOD("sp24_prune", same_shape<sp24_prune>),
    SP24_METHOD("sp24_prune_transposable", same_shape<sp24_prune_transposable>),
    SP24_METHOD("sp24_compress", compress),
    SP24_METHOD("sp24_decompress", decompress),
    SP24_METHOD("sp24_mask_apply", masked<false>),
    SP24_METHOD("sp24_compress_masked", masked<true>),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sp24_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__sp24_host() { return PyModule_Create(&module); }
