// The compute calls of the Python binding as one CPython extension (module _native): argument checks, output
// allocation from torch's allocator and the C-ABI call, without a Python frame in between.
//
// What bounds the small calls is the host: a kernel of 3 .. 6 us was issued every 8.7 .. 10.9 us when the same steps
// ran in Python over ctypes (tensor attributes one by one, argument conversion, the current stream through
// torch.cuda); a launch by itself takes about 3.7 us of host time.  Here the rest takes about 1 us: tensors are read
// through their C++ object, matrices through the fields of Matrix (the base of binding.SparseMatrix), outputs are
// allocated below the operator dispatcher, and the calls take their arguments as a vector.
//
// Checks, defaults and error classes are those of the functions' Python descriptions: AssertionError for tensors that
// do not fit, KeyError for an unknown precision or output type, binding.MagicubeError for a status of the library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/magicube.h"

namespace {

PyObject *g_error_class = nullptr; // binding.MagicubeError

// ---- Matrix: the native part of binding.SparseMatrix -------------------------------------------------
struct Matrix {
    PyObject_HEAD
    mc_mat *mat;          // null once closed
    int64_t M, V, nvec;
    int lhs_bits;
};

PyObject *matrix_attach(PyObject *self, PyObject *args)
{
    unsigned long long handle;
    long long M, V, nvec;
    int lhs_bits;
    if (!PyArg_ParseTuple(args, "KLLLi", &handle, &M, &V, &nvec, &lhs_bits)) return nullptr;
    Matrix *m = reinterpret_cast<Matrix *>(self);
    m->mat = reinterpret_cast<mc_mat *>(static_cast<uintptr_t>(handle));
    m->M = M; m->V = V; m->nvec = nvec; m->lhs_bits = lhs_bits;
    Py_RETURN_NONE;
}

PyObject *matrix_detach(PyObject *self, PyObject *)
{
    reinterpret_cast<Matrix *>(self)->mat = nullptr;
    Py_RETURN_NONE;
}

PyObject *matrix_set_values(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames);

PyMethodDef matrix_methods[] = {
    {"_attach", matrix_attach, METH_VARARGS, "_attach(handle, M, V, nvec, lhs_bits): the native side of a created matrix"},
    {"_detach", matrix_detach, METH_NOARGS, "_detach(): forgets the handle (the matrix is destroyed)"},
    {"set_values", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(matrix_set_values)), METH_FASTCALL | METH_KEYWORDS,
     "set_values($self, values_dev)\n--\n\nvalues_dev: device tensor, nvec*V elements in interchange (vector-major) order."},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject MatrixType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- arguments ---------------------------------------------------------------------------------------
// Distributes positional and keyword arguments over the N named parameters; missing ones stay null.
template <int N> struct Params {
    const char *func;
    int required;
    const char *name[N];
    PyObject *interned[N];
    void intern()
    {
        for (int i = 0; i < N; ++i) interned[i] = PyUnicode_InternFromString(name[i]);
    }
    bool parse(PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, PyObject **out) const
    {
        if (nargs > N) {
            PyErr_Format(PyExc_TypeError, "%s() takes at most %d positional arguments (%zd given)", func, N, nargs);
            return false;
        }
        for (int i = 0; i < N; ++i) out[i] = i < nargs ? args[i] : nullptr;
        const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
        for (Py_ssize_t k = 0; k < nkw; ++k) {
            PyObject *key = PyTuple_GET_ITEM(kwnames, k);
            int at = -1;
            for (int i = 0; i < N && at < 0; ++i)
                if (key == interned[i]) at = i;
            for (int i = 0; i < N && at < 0; ++i)
                if (PyUnicode_Compare(key, interned[i]) == 0) at = i;
            if (at < 0) {
                PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", func, key);
                return false;
            }
            if (out[at]) {
                PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", func, key);
                return false;
            }
            out[at] = args[nargs + k];
        }
        for (int i = 0; i < required; ++i)
            if (!out[i]) {
                PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", func, name[i]);
                return false;
            }
        return true;
    }
};

inline bool given(PyObject *o) { return o && o != Py_None; }

PyObject *assertion()
{
    if (!PyErr_Occurred()) PyErr_SetNone(PyExc_AssertionError);
    return nullptr;
}

PyObject *status_error(int status, const char *where)
{
    PyObject *e = PyObject_CallFunction(g_error_class, "is", status, where);
    if (e) {
        PyErr_SetObject(g_error_class, e);
        Py_DECREF(e);
    }
    return nullptr;
}

struct Precision { const char *name; mc_prec prec; int lhs, rhs; PyObject *interned; };
Precision g_prec[] = {{"L8R8", MC_L8R8, 8, 8, nullptr}, {"L8R4", MC_L8R4, 8, 4, nullptr}, {"L4R4", MC_L4R4, 4, 4, nullptr},
                      {"L16R8", MC_L16R8, 16, 8, nullptr}, {"L16R16", MC_L16R16, 16, 16, nullptr}, {"L16R4", MC_L16R4, 16, 4, nullptr},
                      {"L12R4", MC_L12R4, 12, 4, nullptr}};

const Precision *precision(PyObject *o)
{
    for (const Precision &p : g_prec)
        if (o == p.interned) return &p;
    if (PyUnicode_Check(o))
        for (const Precision &p : g_prec)
            if (PyUnicode_Compare(o, p.interned) == 0) return &p;
    PyErr_SetObject(PyExc_KeyError, o);
    return nullptr;
}

Matrix *matrix(PyObject *o)
{
    if (!PyObject_TypeCheck(o, &MatrixType)) {
        PyErr_Format(PyExc_TypeError, "expected a SparseMatrix, got %.100s", Py_TYPE(o)->tp_name);
        return nullptr;
    }
    return reinterpret_cast<Matrix *>(o);
}

const at::Tensor *tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a tensor, got %.100s", Py_TYPE(o)->tp_name);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

bool number(PyObject *o, float *out)
{
    const double d = PyFloat_AsDouble(o);
    if (d == -1.0 && PyErr_Occurred()) return false;
    *out = (float)d;
    return true;
}

bool integer(PyObject *o, int fallback, int *out)
{
    *out = fallback;
    if (!o) return true;
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) return false;
    *out = (int)v;
    return true;
}

bool truth(PyObject *o, unsigned flag, unsigned *flags)
{
    if (!o || o == Py_False) return true;
    const int t = PyObject_IsTrue(o);
    if (t < 0) return false;
    if (t) *flags |= flag;
    return true;
}

// torch.float32 / torch.float16 -> the library's output type; anything else is a KeyError
bool out_type(PyObject *o, at::ScalarType *dtype, mc_out_type *type)
{
    *dtype = at::kFloat;
    if (o) {
        if (!THPDtype_Check(o)) {
            PyErr_SetObject(PyExc_KeyError, o);
            return false;
        }
        *dtype = reinterpret_cast<THPDtype *>(o)->scalar_type;
    }
    if (*dtype == at::kFloat) *type = MC_OUT_F32;
    else if (*dtype == at::kHalf) *type = MC_OUT_F16;
    else {
        PyErr_SetObject(PyExc_KeyError, o);
        return false;
    }
    return true;
}

// The mc_options behind a ctypes structure (binding.Options), through its buffer; held while the call runs.
struct OptionsArg {
    Py_buffer view = {};
    const mc_options *ptr = nullptr;
    bool read(PyObject *o)
    {
        if (!given(o)) return true;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
        if (view.len != (Py_ssize_t)sizeof(mc_options)) {
            PyErr_SetString(PyExc_TypeError, "options must be an Options structure");
            return false;
        }
        ptr = static_cast<const mc_options *>(view.buf);
        return true;
    }
    ~OptionsArg() { if (view.obj) PyBuffer_Release(&view); }
};

inline void *stream() { return c10::hip::getCurrentHIPStream().stream(); }
// an allocation as torch.empty makes it, below the dispatcher
inline at::TensorBase empty(at::IntArrayRef sizes, at::ScalarType t, const at::Tensor &like)
{
    return at::detail::empty_cuda(sizes, t, like.device(), std::nullopt);
}
inline int elements(int64_t containers, const at::Tensor &t, int bits) { return (int)(containers * (int64_t)t.element_size() * 8 / bits); }
inline bool dense_rows(const at::Tensor &t) { return t.is_cuda() && t.dim() == 2 && t.stride(1) == 1; }
inline PyObject *wrap(at::TensorBase &&t) { return THPVariable_Wrap(std::move(t)); }
inline PyObject *same(PyObject *o) { Py_INCREF(o); return o; }

// ---- SpMM --------------------------------------------------------------------------------------------
Params<7> p_spmm = {"spmm", 3, {"A", "B", "prec", "out", "lhs_unsigned", "rhs_unsigned", "options"}, {}};

PyObject *spmm(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[7];
    if (!p_spmm.parse(args, nargs, kwnames, v)) return nullptr;
    const at::Tensor *B = tensor(v[1]);
    if (!B) return nullptr;
    if (!dense_rows(*B)) return assertion();
    const Precision *p = precision(v[2]);
    Matrix *A = p ? matrix(v[0]) : nullptr;
    if (!A) return nullptr;
    const int N = elements(B->size(1), *B, p->rhs), ldb = elements(B->stride(0), *B, p->rhs);
    const at::Tensor *out = nullptr;
    if (given(v[3])) {
        if (!(out = tensor(v[3]))) return nullptr;
        if (!(dense_rows(*out) && out->scalar_type() == at::kInt && out->size(0) == A->M && out->size(1) == N)) return assertion();
    }
    unsigned flags = 0;
    OptionsArg opts;
    if (!truth(v[4], MC_LHS_UNSIGNED, &flags) || !truth(v[5], MC_RHS_UNSIGNED, &flags) || !opts.read(v[6])) return nullptr;
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty({A->M, N}, at::kInt, *B);
        int32_t *c = static_cast<int32_t *>(out ? out->data_ptr() : made.data_ptr());
        const int ldc = (int)(out ? out->stride(0) : N);
        rc = opts.ptr ? mc_spmm_ex(A->mat, B->data_ptr(), N, ldb, p->prec, flags, opts.ptr, c, ldc, stream())
                      : mc_spmm_flags(A->mat, B->data_ptr(), N, ldb, p->prec, flags, c, ldc, stream());
    }
    if (rc != MC_OK) return status_error(rc, opts.ptr ? "mc_spmm_ex" : "mc_spmm_flags");
    return out ? same(v[3]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<8> p_spmm_dequant = {"spmm_dequant", 4, {"A", "B", "prec", "scale", "out_dtype", "out", "lhs_unsigned", "rhs_unsigned"}, {}};

PyObject *spmm_dequant(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[8];
    if (!p_spmm_dequant.parse(args, nargs, kwnames, v)) return nullptr;
    const at::Tensor *B = tensor(v[1]);
    if (!B) return nullptr;
    if (!dense_rows(*B)) return assertion();
    const Precision *p = precision(v[2]);
    Matrix *A = p ? matrix(v[0]) : nullptr;
    if (!A) return nullptr;
    const int N = elements(B->size(1), *B, p->rhs), ldb = elements(B->stride(0), *B, p->rhs);
    at::ScalarType dtype;
    mc_out_type type;
    float scale;
    unsigned flags = 0;
    if (!number(v[3], &scale) || !out_type(v[4], &dtype, &type)) return nullptr;
    const at::Tensor *out = nullptr;
    if (given(v[5])) {
        if (!(out = tensor(v[5]))) return nullptr;
        if (!(dense_rows(*out) && out->scalar_type() == dtype && out->size(0) == A->M && out->size(1) == N)) return assertion();
    }
    if (!truth(v[6], MC_LHS_UNSIGNED, &flags) || !truth(v[7], MC_RHS_UNSIGNED, &flags)) return nullptr;
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty({A->M, N}, dtype, *B);
        rc = mc_spmm_dequant(A->mat, B->data_ptr(), N, ldb, p->prec, flags, scale, type, out ? out->data_ptr() : made.data_ptr(),
                             (int)(out ? out->stride(0) : N), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_spmm_dequant");
    return out ? same(v[5]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

// ---- SDDMM -------------------------------------------------------------------------------------------
// The two dense operands of an SDDMM call: row lengths and leading dimensions in elements.
struct SddmmOperands {
    const at::Tensor *Q, *K;
    int Kd, ldq, ldk;
    bool read(PyObject *q, PyObject *k, const Precision *p)
    {
        if (!(Q = tensor(q)) || !(K = tensor(k))) return false;
        if (!(dense_rows(*Q) && dense_rows(*K) && Q->size(1) == K->size(1) && Q->element_size() == K->element_size())) {
            assertion();
            return false;
        }
        Kd = elements(Q->size(1), *Q, p->lhs);
        ldq = elements(Q->stride(0), *Q, p->lhs);
        ldk = elements(K->stride(0), *K, p->lhs);
        return true;
    }
};

Params<8> p_sddmm = {"sddmm", 4, {"Q", "Kmat", "mask", "prec", "out", "lhs_unsigned", "rhs_unsigned", "options"}, {}};

PyObject *sddmm(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[8];
    if (!p_sddmm.parse(args, nargs, kwnames, v)) return nullptr;
    const Precision *p = precision(v[3]);
    Matrix *mask = p ? matrix(v[2]) : nullptr;
    SddmmOperands d;
    if (!mask || !d.read(v[0], v[1], p)) return nullptr;
    const int64_t n = mask->nvec * mask->V;
    const at::Tensor *out = nullptr;
    if (given(v[4])) {
        if (!(out = tensor(v[4]))) return nullptr;
        if (!(out->is_cuda() && out->scalar_type() == at::kInt && out->numel() == n && out->is_contiguous())) return assertion();
    }
    unsigned flags = 0;
    OptionsArg opts;
    if (!truth(v[5], MC_LHS_UNSIGNED, &flags) || !truth(v[6], MC_RHS_UNSIGNED, &flags) || !opts.read(v[7])) return nullptr;
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty({n}, at::kInt, *d.Q);
        int32_t *s = static_cast<int32_t *>(out ? out->data_ptr() : made.data_ptr());
        rc = opts.ptr ? mc_sddmm_ex(d.Q->data_ptr(), d.ldq, d.K->data_ptr(), d.ldk, d.Kd, mask->mat, p->prec, flags, opts.ptr, s, stream())
                      : mc_sddmm_flags(d.Q->data_ptr(), d.ldq, d.K->data_ptr(), d.ldk, d.Kd, mask->mat, p->prec, flags, s, stream());
    }
    if (rc != MC_OK) return status_error(rc, opts.ptr ? "mc_sddmm_ex" : "mc_sddmm_flags");
    return out ? same(v[4]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<9> p_sddmm_dequant = {"sddmm_dequant", 5, {"Q", "Kmat", "mask", "prec", "scale", "out_dtype", "out", "lhs_unsigned", "rhs_unsigned"}, {}};

PyObject *sddmm_dequant(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[9];
    if (!p_sddmm_dequant.parse(args, nargs, kwnames, v)) return nullptr;
    const Precision *p = precision(v[3]);
    Matrix *mask = p ? matrix(v[2]) : nullptr;
    SddmmOperands d;
    if (!mask || !d.read(v[0], v[1], p)) return nullptr;
    const int64_t n = mask->nvec * mask->V;
    float scale;
    at::ScalarType dtype;
    mc_out_type type;
    if (!number(v[4], &scale) || !out_type(v[5], &dtype, &type)) return nullptr;
    const at::Tensor *out = nullptr;
    if (given(v[6])) {
        if (!(out = tensor(v[6]))) return nullptr;
        if (!(out->is_cuda() && out->scalar_type() == dtype && out->numel() == n && out->is_contiguous())) return assertion();
    }
    unsigned flags = 0;
    if (!truth(v[7], MC_LHS_UNSIGNED, &flags) || !truth(v[8], MC_RHS_UNSIGNED, &flags)) return nullptr;
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty({n}, dtype, *d.Q);
        rc = mc_sddmm_dequant(d.Q->data_ptr(), d.ldq, d.K->data_ptr(), d.ldk, d.Kd, mask->mat, p->prec, flags, scale, type,
                              out ? out->data_ptr() : made.data_ptr(), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_sddmm_dequant");
    return out ? same(v[6]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<5> p_sddmm_to_mat = {"sddmm_to_mat", 5, {"Q", "Kmat", "P", "prec", "scale"}, {}};

PyObject *sddmm_to_mat(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[5];
    if (!p_sddmm_to_mat.parse(args, nargs, kwnames, v)) return nullptr;
    const Precision *p = precision(v[3]);
    Matrix *P = p ? matrix(v[2]) : nullptr;
    SddmmOperands d;
    float scale;
    if (!P || !d.read(v[0], v[1], p) || !number(v[4], &scale)) return nullptr;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        rc = mc_sddmm_to_mat(d.Q->data_ptr(), d.ldq, d.K->data_ptr(), d.ldk, d.Kd, p->prec, scale, P->mat, stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_sddmm_to_mat");
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

// ---- values, quantisation, softmax --------------------------------------------------------------------
Params<1> p_set_values = {"set_values", 1, {"values_dev"}, {}};

PyObject *matrix_set_values(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[1];
    if (!p_set_values.parse(args, nargs, kwnames, v)) return nullptr;
    Matrix *A = reinterpret_cast<Matrix *>(self);
    const at::Tensor *x = tensor(v[0]);
    if (!x) return nullptr;
    const int bits = A->lhs_bits == 12 ? 16 : A->lhs_bits;  // a 12-bit value travels as int16
    if (!(x->is_cuda() && x->is_contiguous() && x->numel() * (int64_t)x->element_size() == A->nvec * A->V * bits / 8)) return assertion();
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        rc = mc_mat_set_values_device(A->mat, x->data_ptr(), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_mat_set_values_device");
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

Params<2> p_absmax = {"absmax", 1, {"x", "out"}, {}};

PyObject *absmax(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[2];
    if (!p_absmax.parse(args, nargs, kwnames, v)) return nullptr;
    const at::Tensor *x = tensor(v[0]), *out = nullptr;
    if (!x) return nullptr;
    if (!(x->is_cuda() && x->scalar_type() == at::kFloat && x->is_contiguous())) return assertion();
    if (given(v[1]) && !(out = tensor(v[1]))) return nullptr;
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty({1}, at::kFloat, *x);
        rc = mc_absmax(static_cast<const float *>(x->data_ptr()), x->numel(), static_cast<float *>(out ? out->data_ptr() : made.data_ptr()), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_absmax");
    return out ? same(v[1]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<4> p_quantize = {"quantize", 2, {"x", "scale", "bits", "out"}, {}};

PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[4];
    if (!p_quantize.parse(args, nargs, kwnames, v)) return nullptr;
    const at::Tensor *x = tensor(v[0]), *out = nullptr;
    float scale;
    int bits;
    if (!x || !number(v[1], &scale) || !integer(v[2], 8, &bits)) return nullptr;
    if (!(x->is_cuda() && x->scalar_type() == at::kFloat && x->is_contiguous())) return assertion();
    if (given(v[3])) {
        if (!(out = tensor(v[3]))) return nullptr;
        if (!(out->is_cuda() && out->is_contiguous())) return assertion();
        if ((bits == 4 || bits == 8) && out->numel() * (bits == 4 ? 2 : 1) != x->numel()) return status_error(MC_EINVAL, "quantize(out size)");
    }
    c10::SmallVector<int64_t, 5> sizes(x->sizes().begin(), x->sizes().end());
    if (!out && bits == 4) {
        if (sizes.empty()) return assertion();
        sizes.back() /= 2;
        if (c10::multiply_integers(sizes) * 2 != x->numel()) return status_error(MC_EINVAL, "quantize(out size)");
    }
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty(sizes, bits == 4 ? at::kByte : at::kChar, *x);
        rc = mc_quantize(static_cast<const float *>(x->data_ptr()), x->numel(), scale, bits, out ? out->data_ptr() : made.data_ptr(), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_quantize");
    return out ? same(v[3]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<6> p_softmax = {"sparse_softmax", 4, {"mask", "S", "score_scale", "inv_s_p", "out", "code_bits"}, {}};

PyObject *sparse_softmax(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[6];
    if (!p_softmax.parse(args, nargs, kwnames, v)) return nullptr;
    Matrix *mask = matrix(v[0]);
    const at::Tensor *S = mask ? tensor(v[1]) : nullptr, *out = nullptr;
    float score_scale, inv_s_p;
    int code_bits;
    if (!S || !number(v[2], &score_scale) || !number(v[3], &inv_s_p) || !integer(v[5], 8, &code_bits)) return nullptr;
    const int64_t n = mask->nvec * mask->V;
    if (!(S->is_cuda() && S->scalar_type() == at::kInt && S->is_contiguous() && (n == 0 || S->numel() % n == 0))) return assertion();
    const int64_t batch = n ? S->numel() / n : (S->dim() > 1 ? S->size(0) : 1);
    const at::ScalarType dt = code_bits == 16 ? at::kShort : at::kChar;
    if (given(v[4])) {
        if (!(out = tensor(v[4]))) return nullptr;
        if (!(out->is_cuda() && out->scalar_type() == dt && out->is_contiguous() && out->numel() == batch * n)) return assertion();
    }
    at::TensorBase made;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = empty(S->sizes(), dt, *S);
        rc = mc_sparse_softmax_bits(mask->mat, (int)batch, static_cast<const int32_t *>(S->data_ptr()), score_scale, inv_s_p, code_bits,
                                    out ? out->data_ptr() : made.data_ptr(), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_sparse_softmax_bits");
    return wrap(out ? at::TensorBase(out->reshape(S->sizes())) : std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<4> p_softmax_to_mat = {"sparse_softmax_to_mat", 4, {"P", "S", "score_scale", "inv_s_p"}, {}};

PyObject *sparse_softmax_to_mat(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[4];
    if (!p_softmax_to_mat.parse(args, nargs, kwnames, v)) return nullptr;
    Matrix *P = matrix(v[0]);
    const at::Tensor *S = P ? tensor(v[1]) : nullptr;
    float score_scale, inv_s_p;
    if (!S || !number(v[2], &score_scale) || !number(v[3], &inv_s_p)) return nullptr;
    if (!(S->is_cuda() && S->scalar_type() == at::kInt && S->is_contiguous() && S->numel() == P->nvec * P->V)) return assertion();
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        rc = mc_sparse_softmax_to_mat(P->mat, static_cast<const int32_t *>(S->data_ptr()), score_scale, inv_s_p, stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_sparse_softmax_to_mat");
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

// ---- attention ---------------------------------------------------------------------------------------
// Q / K / V of one layer call: (heads, L, dk) or (batch, heads, L, dk), any strides with unit stride along dk;
// strides in elements (4-bit tensors hold two per byte).
struct AttentionInputs {
    const at::Tensor *q, *k, *v;
    int batch, heads, L, dk, p_bits, qkv_bits;
    int64_t bs, hs, ts;
    float s_q, s_k, s_v, s_p;
    c10::SmallVector<int64_t, 5> out_sizes, out_strides;
    bool read(PyObject *const *a, PyObject *pb, PyObject *qb)
    {
        if (!(q = tensor(a[0])) || !(k = tensor(a[1])) || !(v = tensor(a[2])) || !number(a[4], &s_q) || !number(a[5], &s_k) ||
            !number(a[6], &s_v) || !number(a[7], &s_p) || !integer(pb, 8, &p_bits) || !integer(qb, 8, &qkv_bits))
            return false;
        if (qkv_bits <= 0) {
            assertion();
            return false;
        }
        const int64_t epb = 8 / qkv_bits;   // elements per byte
        const int d = (int)q->dim();
        bool fits = d == 3 || d == 4;
        for (const at::Tensor *t : {q, k, v})
            fits = fits && t->is_cuda() && t->element_size() == 1 && t->sizes() == q->sizes() && t->strides() == q->strides() && t->stride(-1) == 1;
        if (!fits) {
            assertion();
            return false;
        }
        batch = d == 4 ? (int)q->size(0) : 1;
        heads = (int)q->size(d - 3);
        L = (int)q->size(d - 2);
        dk = (int)(q->size(d - 1) * epb);
        bs = d == 4 ? q->stride(0) * epb : 0;
        hs = q->stride(d - 3) * epb;
        ts = q->stride(d - 2) * epb;
        for (int i = 0; i < d; ++i) {
            out_sizes.push_back(i == d - 1 ? dk : q->size(i));
            out_strides.push_back(i == d - 1 ? 1 : q->stride(i) * epb);
        }
        return true;
    }
    bool fits_out(const at::Tensor &o) const
    {
        return o.is_cuda() && o.sizes() == at::IntArrayRef(out_sizes) && o.strides() == at::IntArrayRef(out_strides);
    }
};

Params<14> p_attention = {"sparse_attention", 8,
                          {"Q8", "K8", "V8", "mask", "s_q", "s_k", "s_v", "s_p", "out", "workspace", "p_bits", "qkv_bits", "out_dtype", "options"}, {}};

PyObject *sparse_attention(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[14];
    if (!p_attention.parse(args, nargs, kwnames, v)) return nullptr;
    AttentionInputs in;
    at::ScalarType dtype;
    mc_out_type type;
    Matrix *mask = matrix(v[3]);
    if (!mask || !in.read(v, v[10], v[11]) || !out_type(v[12], &dtype, &type)) return nullptr;
    const at::Tensor *out = nullptr, *ws = nullptr;
    if (given(v[8])) {
        if (!(out = tensor(v[8]))) return nullptr;
        if (!(in.fits_out(*out) && out->scalar_type() == dtype)) return assertion();
    }
    if (given(v[9])) {
        if (!(ws = tensor(v[9]))) return nullptr;
        if (!(ws->is_cuda() && ws->is_contiguous())) return assertion();
    }
    OptionsArg opts;
    if (!opts.read(v[13])) return nullptr;
    at::TensorBase made, scratch;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        if (!out) made = at::detail::empty_strided_cuda(in.out_sizes, in.out_strides, dtype, in.q->device()); // the inputs' layout
        void *o = out ? out->data_ptr() : made.data_ptr(), *w = nullptr;
        size_t wbytes = 0;
        if (ws) {
            w = ws->data_ptr();
            wbytes = (size_t)ws->numel() * ws->element_size();
        } else if (mc_attention_form(mask->mat, in.dk, in.qkv_bits, opts.ptr) != 0 &&
                   (wbytes = mc_attention_workspace_needed(in.heads, in.dk, mask->mat, in.p_bits, opts.ptr)) > 0) {
            scratch = empty({(int64_t)wbytes}, at::kByte, *in.q);
            w = scratch.data_ptr();
        }
        rc = opts.ptr ? mc_sparse_attention_ex(in.q->data_ptr(), in.k->data_ptr(), in.v->data_ptr(), in.batch, in.heads, in.L, in.dk, in.bs,
                                               in.hs, in.ts, mask->mat, in.p_bits, in.qkv_bits, in.s_q, in.s_k, in.s_v, in.s_p, type,
                                               opts.ptr, o, w, wbytes, stream())
                      : mc_sparse_attention_out(in.q->data_ptr(), in.k->data_ptr(), in.v->data_ptr(), in.batch, in.heads, in.L, in.dk, in.bs,
                                                in.hs, in.ts, mask->mat, in.p_bits, in.qkv_bits, in.s_q, in.s_k, in.s_v, in.s_p, type, o, w,
                                                wbytes, stream());
    }
    if (rc != MC_OK) return status_error(rc, opts.ptr ? "mc_sparse_attention_ex" : "mc_sparse_attention_out");
    return out ? same(v[8]) : wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

Params<12> p_attention_static = {"sparse_attention_static", 9,
                                 {"Q8", "K8", "V8", "mask", "s_q", "s_k", "s_v", "s_p", "out", "p_bits", "qkv_bits", "options"}, {}};

PyObject *sparse_attention_static(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    HANDLE_TH_ERRORS
    PyObject *v[12];
    if (!p_attention_static.parse(args, nargs, kwnames, v)) return nullptr;
    AttentionInputs in;
    Matrix *mask = matrix(v[3]);
    const at::Tensor *out = mask ? tensor(v[8]) : nullptr;
    if (!out || !in.read(v, v[9], v[10])) return nullptr;
    if (!(in.fits_out(*out) && (out->scalar_type() == at::kFloat || out->scalar_type() == at::kHalf))) return assertion();
    OptionsArg opts;
    if (!opts.read(v[11])) return nullptr;
    int rc;
    {
        pybind11::gil_scoped_release nogil;
        rc = mc_sparse_attention_static(in.q->data_ptr(), in.k->data_ptr(), in.v->data_ptr(), in.batch, in.heads, in.L, in.dk, in.bs, in.hs,
                                        in.ts, mask->mat, in.p_bits, in.qkv_bits, in.s_q, in.s_k, in.s_v, in.s_p,
                                        out->scalar_type() == at::kHalf ? MC_OUT_F16 : MC_OUT_F32, opts.ptr, out->data_ptr(), stream());
    }
    if (rc != MC_OK) return status_error(rc, "mc_sparse_attention_static");
    return same(v[8]);
    END_HANDLE_TH_ERRORS
}

PyObject *set_error_class(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XSETREF(g_error_class, cls);
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL | METH_KEYWORDS
PyMethodDef functions[] = {
    {"_set_error_class", set_error_class, METH_O, "the exception raised for a status of the library"},
    {"spmm", FAST(spmm),
     "spmm(A, B, prec, out=None, lhs_unsigned=False, rhs_unsigned=False, options=None)\n--\n\n"
     "C = A * B (int32, M x N).  B: device tensor (K, N) int8, (K, N/2) uint8 for R4, (K, N) int16 for R16.\n"
     "lhs_unsigned / rhs_unsigned: read the 8- or 4-bit operand as non-negative values.\n"
     "options: kernel-variant choices of this call (None: the calling thread's defaults)."},
    {"spmm_dequant", FAST(spmm_dequant),
     "spmm_dequant(A, B, prec, scale, out_dtype=torch.float32, out=None, lhs_unsigned=False, rhs_unsigned=False)\n\n"
     "C = scale * (A * B) as fp32 or fp16 (M x N): SpMM with the dequantisation fused into the kernel.\n"
     "(Kernel variants: the thread's options.)"},
    {"sddmm", FAST(sddmm),
     "sddmm(Q, Kmat, mask, prec, out=None, lhs_unsigned=False, rhs_unsigned=False, options=None)\n--\n\n"
     "S (nvec*V int32, interchange order) = (Q * Kmat^T) at the mask's stored vectors."},
    {"sddmm_dequant", FAST(sddmm_dequant),
     "sddmm_dequant(Q, Kmat, mask, prec, scale, out_dtype=torch.float32, out=None, lhs_unsigned=False, rhs_unsigned=False)\n\n"
     "scale * (Q * Kmat^T) at the mask's stored vectors as nvec*V fp32 or fp16 values (interchange order)."},
    {"sddmm_to_mat", FAST(sddmm_to_mat),
     "sddmm_to_mat(Q, Kmat, P, prec, scale)\n--\n\n"
     "(Q * Kmat^T) at P's pattern, re-quantised to P's 8- or 16-bit integers and written into P's device values."},
    {"absmax", FAST(absmax), "absmax(x, out=None)\n--\n\nmax |x| of a contiguous fp32 device tensor, as a one-element device tensor."},
    {"quantize", FAST(quantize),
     "quantize(x, scale, bits=8, out=None)\n--\n\n"
     "Symmetric quantisation of a contiguous fp32 device tensor: int8 codes of the same shape, or\n"
     "(bits=4) uint8 with half the last dimension, two codes per byte."},
    {"sparse_softmax", FAST(sparse_softmax),
     "sparse_softmax(mask, S, score_scale, inv_s_p, out=None, code_bits=8)\n--\n\n"
     "Integer codes (int8, or int16 for code_bits=16) of the row softmax over the stored\n"
     "entries; S: (batch, nvec*V) int32."},
    {"sparse_softmax_to_mat", FAST(sparse_softmax_to_mat),
     "sparse_softmax_to_mat(P, S, score_scale, inv_s_p)\n--\n\n"
     "Softmax of one score set (nvec*V int32) written as integer codes straight into P's device values."},
    {"sparse_attention", FAST(sparse_attention),
     "sparse_attention(Q8, K8, V8, mask, s_q, s_k, s_v, s_p, out=None, workspace=None, p_bits=8, qkv_bits=8,\n"
     "                 out_dtype=torch.float32, options=None)\n\n"
     "Quantized sparse self-attention; Q8/K8/V8: (heads, L, dk) or (batch, heads, L, dk) int8\n"
     "device tensors, or for qkv_bits=4 uint8 tensors of half the last dimension with two 4-bit\n"
     "values per byte.  p_bits is the width of the re-quantised softmax output (8 or 16);\n"
     "out_dtype is torch.float32 or torch.float16.\n\n"
     "Any layout with unit stride along dk is accepted as long as the three tensors (and\n"
     "``out``) share it; a (heads, L, dk) view of a token-major (L, heads, dk) buffer, i.e.\n"
     "``x.permute(1, 0, 2)``, selects the fast two-heads-per-request path."},
    {"sparse_attention_static", FAST(sparse_attention_static),
     "sparse_attention_static(Q8, K8, V8, mask, s_q, s_k, s_v, s_p, out, p_bits=8, qkv_bits=8, options=None)\n--\n\n"
     "sparse_attention for callers that cannot allocate: no workspace argument (the library's own per-GPU array\n"
     "holds the intermediates) and a caller-provided ``out``.  This wrapper allocates nothing on the device either."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "The binding's compute calls over the C ABI of libmagicube.so.", -1, functions};

} // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    MatrixType.tp_name = "paper_2209_06979_amd._native.Matrix";
    MatrixType.tp_basicsize = sizeof(Matrix);
    MatrixType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
    MatrixType.tp_doc = "Native part of binding.SparseMatrix: the handle and sizes that the compute calls read.";
    MatrixType.tp_methods = matrix_methods;
    MatrixType.tp_new = PyType_GenericNew;
    if (PyType_Ready(&MatrixType) < 0) return nullptr;
    for (Precision &p : g_prec) p.interned = PyUnicode_InternFromString(p.name);
    p_spmm.intern(); p_spmm_dequant.intern(); p_sddmm.intern(); p_sddmm_dequant.intern(); p_sddmm_to_mat.intern();
    p_set_values.intern(); p_absmax.intern(); p_quantize.intern(); p_softmax.intern(); p_softmax_to_mat.intern();
    p_attention.intern(); p_attention_static.intern();
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    Py_INCREF(&MatrixType);
    if (PyModule_AddObject(m, "Matrix", reinterpret_cast<PyObject *>(&MatrixType)) < 0) return nullptr;
    return m;
}
