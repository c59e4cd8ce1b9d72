// The usual calls of binding.py in native code.  A small call is bound by the host: of the 6.6 us that one
// spinner_apply_signs took through ctypes (27 us for a layer's forward and backward), 3.2 us are the launch; tensor
// checks, the allocation through torch's Python face and the marshalling of a dozen arguments were the rest.
//
// Each function takes the arguments of its namesake in binding.py, all of them, by position, and returns its result, or
// None when anything about the call is out of the ordinary: a tensor that is no plain contiguous CUDA tensor of the
// type and size expected, a number that is no Python number, an explicit stream, a status that the library finds before it
// launches anything.  binding.py then takes the call its long way, which knows every check and error.  SPINNER_ERR_HIP
// alone may come with kernels already on their way: that call is not made again, its SpinnerError is raised from here.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <pybind11/pybind11.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "spinner.h"

namespace {

using at::Tensor;

// a plain tensor on a GPU with memory of its own (subclasses and wrapped tensors go the long way)
const Tensor* gpu_tensor(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    return t.has_storage() && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}
const Tensor* typed_tensor(PyObject* o, at::ScalarType type)
{
    const Tensor* t = gpu_tensor(o);
    return t && t->scalar_type() == type ? t : nullptr;
}
const Tensor* floats(PyObject* o) { return typed_tensor(o, at::kFloat); }
const Tensor* floats(PyObject* o, int64_t count)
{
    const Tensor* t = floats(o);
    return t && t->numel() == count ? t : nullptr;
}
// rows [batch][n]; n has to fit the int of the C ABI
const Tensor* rows(PyObject* o, long* batch, int* n)
{
    const Tensor* t = floats(o);
    if (!t || t->dim() != 2 || t->size(1) > INT_MAX) return nullptr;
    *batch = (long)t->size(0);
    *n = (int)t->size(1);
    return t;
}
bool whole(PyObject* o, int* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long l = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || l < INT_MIN || l > INT_MAX) return false;
    *v = (int)l;
    return true;
}
// the number of kept rows: None stands for n
bool kept(PyObject* o, int n, int* m)
{
    if (o == Py_None) *m = n;
    else if (!whole(o, m)) return false;
    return *m >= 1 && *m <= n;
}
bool number(PyObject* o, float* v)
{
    if (PyFloat_CheckExact(o)) { *v = (float)PyFloat_AS_DOUBLE(o); return true; }
    int i;
    if (!whole(o, &i)) return false;
    *v = (float)i;
    return true;
}
bool choice(PyObject* o, const char* const* names, int count, int* v)
{
    if (PyUnicode_CheckExact(o)) {
        for (int i = 0; i < count; ++i)
            if (PyUnicode_CompareWithASCIIString(o, names[i]) == 0) { *v = i; return true; }
        return false;
    }
    return whole(o, v) && *v >= 0 && *v < count;
}
bool epilogue(PyObject* o, int* v)
{
    static const char* const names[] = {"none", "cossin"};
    static_assert(SPINNER_EPI_NONE == 0 && SPINNER_EPI_COSSIN == 1, "the order of the names");
    return choice(o, names, 2, v);
}
bool struct_kind(PyObject* o, int* v)
{
    static const char* const names[] = {"circulant", "skew_circulant", "toeplitz", "hankel"};
    static_assert(SPINNER_STRUCT_CIRCULANT == 0 && SPINNER_STRUCT_SKEW_CIRCULANT == 1 && SPINNER_STRUCT_TOEPLITZ == 2 &&
                      SPINNER_STRUCT_HANKEL == 3, "the order of the names");
    return choice(o, names, 4, v);
}

// Memory that the caller may bring: `given` is null where the argument was None, and is checked by usable() before anything
// is allocated.
struct Buffer {
    const Tensor* given = nullptr;
    bool usable(PyObject* o, at::ScalarType type, int64_t count)
    {
        if (o == Py_None) return true;
        given = typed_tensor(o, type);
        return given && given->numel() == count;
    }
    bool usable_bytes(PyObject* o, size_t need)
    {
        if (o == Py_None) return true;
        given = gpu_tensor(o);
        return given && (size_t)given->nbytes() >= need;
    }
    Tensor get(at::IntArrayRef sizes, at::ScalarType type, const Tensor& like) const
    {
        return given ? *given : at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
    }
    // scratch: no tensor at all where none is needed
    Tensor scratch(size_t need, const Tensor& like) const
    {
        return given || need ? get({(int64_t)need}, at::kByte, like) : Tensor();
    }
};
template <typename T = float>
T* ptr(const Tensor& t) { return t.defined() ? static_cast<T*>(t.data_ptr()) : nullptr; }
template <typename T = float>
T* ptr(const Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// packed sign words of `count` triples from triple `first` on
const void* sign_words(PyObject* o, int n, int first, int count)
{
    const Tensor* t = typed_tensor(o, at::kByte);
    const size_t one = spinner_signs_bytes(n, 1);
    if (!t || one == 0 || first < 0 || count < 1 || (size_t)t->numel() < ((size_t)first + count) * one) return nullptr;
    return static_cast<const char*>(t->data_ptr()) + first * one;
}

// a status other than SPINNER_OK: the long way, or the error itself
PyObject* refused(int rc)
{
    if (rc != SPINNER_ERR_HIP) Py_RETURN_NONE;
    const auto error = pybind11::module_::import("paper_1610_06209_amd.binding").attr("SpinnerError");
    PyErr_SetObject(error.ptr(), error(rc).ptr());
    return nullptr;
}

using Args = PyObject* const*;
#define LONG_WAY Py_RETURN_NONE
#define ENTRY(NAME, COUNT)                                                          \
    PyObject* NAME(PyObject*, Args a, Py_ssize_t given)                             \
    {                                                                               \
        HANDLE_TH_ERRORS                                                            \
        if (given != COUNT) { PyErr_SetString(PyExc_TypeError, #NAME ": " #COUNT " arguments"); return nullptr; }
#define ENTRY_END                                                                   \
        END_HANDLE_TH_ERRORS                                                        \
    }

// x, signs, m, epilogue, scale, out, workspace, stream, triple
ENTRY(apply_signs, 9)
    long batch;
    int n, m, epi, triple;
    float scale;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[7] != Py_None || !kept(a[2], n, &m) || !epilogue(a[3], &epi) || !number(a[4], &scale) || !whole(a[8], &triple)) LONG_WAY;
    const void* words = sign_words(a[1], n, triple, 1);
    const int64_t width = epi == SPINNER_EPI_COSSIN ? 2LL * m : m;
    const size_t need = spinner_workspace_bytes(n, batch, m, epi);
    Buffer o, w;
    if (!words || !o.usable(a[5], at::kFloat, batch * width) || !w.usable_bytes(a[6], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, width}, at::kFloat, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_apply_signs(ptr(x), n, batch, words, m, epi, scale, ptr(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, d1, d2, d3, m, epilogue, scale, out, workspace, stream
ENTRY(apply, 10)
    long batch;
    int n, m, epi;
    float scale;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[9] != Py_None || !kept(a[4], n, &m) || !epilogue(a[5], &epi) || !number(a[6], &scale)) LONG_WAY;
    const Tensor *d1 = floats(a[1], n), *d2 = floats(a[2], n), *d3 = floats(a[3], n);
    const int64_t width = epi == SPINNER_EPI_COSSIN ? 2LL * m : m;
    const size_t need = spinner_workspace_bytes(n, batch, m, epi);
    Buffer o, w;
    if (!d1 || !d2 || !d3 || !o.usable(a[7], at::kFloat, batch * width) || !w.usable_bytes(a[8], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, width}, at::kFloat, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_apply(ptr(x), n, batch, ptr(d1), ptr(d2), ptr(d3), m, epi, scale, ptr(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, diag_sets, m, epilogue, scale, out, workspace, stream
ENTRY(apply_blocks, 8)
    long batch;
    int n, m, epi;
    float scale;
    const Tensor *x = rows(a[0], &batch, &n), *d = floats(a[1]);
    if (!x || !d || a[7] != Py_None || !kept(a[2], n, &m) || !epilogue(a[3], &epi) || !number(a[4], &scale)) LONG_WAY;
    if (d->dim() != 3 || d->size(0) > INT_MAX || d->size(1) != 3 || d->size(2) != n) LONG_WAY;
    const int L = (int)d->size(0);
    const int64_t width = (epi == SPINNER_EPI_COSSIN ? 2LL * m : m) * L;
    const size_t need = spinner_blocks_workspace_bytes(n, batch, m, epi);
    Buffer o, w;
    if (!o.usable(a[5], at::kFloat, batch * width) || !w.usable_bytes(a[6], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, width}, at::kFloat, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_apply_blocks(ptr(x), n, batch, L, ptr(d), m, epi, scale, ptr(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, diag_sets, out_idx, stream
ENTRY(hash, 4)
    long batch;
    int n;
    const Tensor *x = rows(a[0], &batch, &n), *d = floats(a[1]);
    if (!x || !d || a[3] != Py_None || d->dim() != 3 || d->size(0) > INT_MAX || d->size(1) != 3 || d->size(2) != n) LONG_WAY;
    const int L = (int)d->size(0);
    Buffer o;
    if (!o.usable(a[2], at::kInt, (int64_t)batch * L)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, L}, at::kInt, *x);
        rc = spinner_hash(ptr(x), n, batch, L, ptr(d), ptr<int>(out), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, signs, L, out_idx, stream
ENTRY(hash_signs, 5)
    long batch;
    int n, L;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[4] != Py_None || !whole(a[2], &L)) LONG_WAY;
    const void* words = sign_words(a[1], n, 0, L);
    Buffer o;
    if (!words || !o.usable(a[3], at::kInt, (int64_t)batch * L)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, L}, at::kInt, *x);
        rc = spinner_hash_signs(ptr(x), n, batch, L, words, ptr<int>(out), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, d1, d2, d3, m, codes, workspace, stream
ENTRY(sign_codes, 8)
    long batch;
    int n, m;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[7] != Py_None || !kept(a[4], n, &m) || spinner_code_bytes(m) == 0) LONG_WAY;
    const Tensor *d1 = floats(a[1], n), *d2 = floats(a[2], n), *d3 = floats(a[3], n);
    const int64_t words = (int64_t)spinner_code_bytes(m) / 8;
    const size_t need = spinner_codes_workspace_bytes(n, batch);
    Buffer o, w;
    if (!d1 || !d2 || !d3 || !o.usable(a[5], at::kLong, batch * words) || !w.usable_bytes(a[6], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, words}, at::kLong, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_sign_codes(ptr(x), n, batch, ptr(d1), ptr(d2), ptr(d3), m, ptr<void>(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, signs, m, codes, workspace, stream, triple
ENTRY(sign_codes_signs, 7)
    long batch;
    int n, m, triple;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[5] != Py_None || !kept(a[2], n, &m) || spinner_code_bytes(m) == 0 || !whole(a[6], &triple)) LONG_WAY;
    const void* signs = sign_words(a[1], n, triple, 1);
    const int64_t words = (int64_t)spinner_code_bytes(m) / 8;
    const size_t need = spinner_codes_workspace_bytes(n, batch);
    Buffer o, w;
    if (!signs || !o.usable(a[3], at::kLong, batch * words) || !w.usable_bytes(a[4], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, words}, at::kLong, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_sign_codes_signs(ptr(x), n, batch, signs, m, ptr<void>(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// codes_a, codes_b, m, out, stream
ENTRY(angular_gram, 5)
    int m;
    const Tensor *p = typed_tensor(a[0], at::kLong), *q = typed_tensor(a[1], at::kLong);
    if (!p || !q || a[4] != Py_None || !whole(a[2], &m) || spinner_code_bytes(m) == 0) LONG_WAY;
    const int64_t words = (int64_t)spinner_code_bytes(m) / 8;
    if (p->dim() != 2 || q->dim() != 2 || p->size(1) != words || q->size(1) != words) LONG_WAY;
    const long na = (long)p->size(0), nb = (long)q->size(0);
    Buffer o;
    if (!o.usable(a[3], at::kFloat, (int64_t)na * nb)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({na, nb}, at::kFloat, *p);
        rc = spinner_angular_gram(ptr<void>(p), na, ptr<void>(q), nb, m, ptr(out), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, d1, d2, d3, scale, y, saved, stream
ENTRY(layer_forward, 8)
    long batch;
    int n;
    float scale;
    const Tensor* x = rows(a[0], &batch, &n);
    if (!x || a[7] != Py_None || !number(a[4], &scale)) LONG_WAY;
    const Tensor *d1 = floats(a[1], n), *d2 = floats(a[2], n), *d3 = floats(a[3], n);
    Buffer o, s;
    if (!d1 || !d2 || !d3 || !o.usable(a[5], at::kFloat, (int64_t)batch * n) || !s.usable(a[6], at::kFloat, 2LL * batch * n)) LONG_WAY;
    Tensor y, saved;
    int rc;
    {
        pybind11::gil_scoped_release free;
        y = o.get({batch, n}, at::kFloat, *x);
        saved = s.get({2, batch, n}, at::kFloat, *x);
        rc = spinner_layer_forward(ptr(x), n, batch, ptr(d1), ptr(d2), ptr(d3), scale, ptr(y), ptr<void>(saved), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(y)), THPVariable_Wrap(std::move(saved)));
ENTRY_END

// dy, x, saved, d1, d2, d3, scale, dx, dd, workspace, stream
ENTRY(layer_backward, 11)
    long batch, dy_batch;
    int n, dy_n;
    float scale;
    const Tensor *dy = rows(a[0], &dy_batch, &dy_n), *x = rows(a[1], &batch, &n);
    if (!dy || !x || dy_batch != batch || dy_n != n || a[10] != Py_None || !number(a[6], &scale)) LONG_WAY;
    const Tensor *saved = floats(a[2], 2LL * batch * n), *d1 = floats(a[3], n), *d2 = floats(a[4], n), *d3 = floats(a[5], n);
    size_t need = spinner_layer_workspace_bytes(n, batch);
    Buffer o, g, w;
    if (!saved || !d1 || !d2 || !d3 || !o.usable(a[7], at::kFloat, (int64_t)batch * n) || !g.usable(a[8], at::kFloat, 3LL * n) ||
        !w.usable_bytes(a[9], need))
        LONG_WAY;
    Tensor dx, dd;
    int rc;
    {
        pybind11::gil_scoped_release free;
        dx = o.get({batch, n}, at::kFloat, *x);
        dd = g.get({3, n}, at::kFloat, *x);
        const Tensor ws = w.scratch(need < 16 ? 16 : need, *x);
        rc = spinner_layer_backward(ptr(dy), ptr(x), ptr<void>(saved), n, batch, ptr(d1), ptr(d2), ptr(d3), scale, ptr(dx), ptr(dd),
                                    ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(dx)), THPVariable_Wrap(std::move(dd)));
ENTRY_END

// A, w, d1, d2, d3, m, scale, out, workspace, stream
ENTRY(sketch, 10)
    long n_rows;
    int d, m;
    float scale;
    const Tensor* A = rows(a[0], &n_rows, &d);
    if (!A || n_rows > INT_MAX || a[9] != Py_None || !kept(a[5], (int)n_rows, &m) || !number(a[6], &scale)) LONG_WAY;
    const int n = (int)n_rows;
    const Tensor *weights = a[1] == Py_None ? nullptr : floats(a[1], n), *d1 = floats(a[2], n), *d2 = floats(a[3], n), *d3 = floats(a[4], n);
    const size_t need = spinner_sketch_workspace_bytes(n, d, m);
    Buffer o, w;
    if ((!weights && a[1] != Py_None) || !d1 || !d2 || !d3 || !o.usable(a[7], at::kFloat, (int64_t)m * d) || !w.usable_bytes(a[8], need))
        LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({m, d}, at::kFloat, *A);
        const Tensor ws = w.scratch(need < 16 ? 16 : need, *A);
        rc = spinner_sketch(ptr(A), n, d, ptr(weights), ptr(d1), ptr(d2), ptr(d3), m, scale, ptr(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// B, out, workspace, stream
ENTRY(sketch_gram, 4)
    long m_rows;
    int d;
    const Tensor* B = rows(a[0], &m_rows, &d);
    if (!B || m_rows > INT_MAX || a[3] != Py_None) LONG_WAY;
    const int m = (int)m_rows;
    const size_t need = spinner_sketch_gram_workspace_bytes(m, d);
    Buffer o, w;
    if (!o.usable(a[1], at::kFloat, (int64_t)d * d) || !w.usable_bytes(a[2], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({d, d}, at::kFloat, *B);
        const Tensor ws = w.scratch(need, *B);
        rc = spinner_sketch_gram(ptr(B), m, d, ptr(out), ptr<void>(ws), current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

// x, kind, spectrum, d1, d2, m, scale, out, workspace, stream
ENTRY(struct_apply_ws, 10)
    long batch;
    int n, m, kind;
    float scale;
    const Tensor *x = rows(a[0], &batch, &n), *spectrum = gpu_tensor(a[2]);
    if (!x || !spectrum || a[9] != Py_None || !struct_kind(a[1], &kind) || !kept(a[5], n, &m) || !number(a[6], &scale)) LONG_WAY;
    const Tensor *d1 = floats(a[3], n), *d2 = floats(a[4], n);
    const size_t need = spinner_struct_workspace_bytes(kind, n, batch);
    Buffer o, w;
    if ((size_t)spectrum->nbytes() < spinner_struct_spectrum_bytes(kind, n) || !d1 || !d2 || !o.usable(a[7], at::kFloat, (int64_t)batch * m) || !w.usable_bytes(a[8], need)) LONG_WAY;
    Tensor out;
    int rc;
    {
        pybind11::gil_scoped_release free;
        out = o.get({batch, m}, at::kFloat, *x);
        const Tensor ws = w.scratch(need, *x);
        rc = spinner_struct_apply_ws(ptr(x), n, batch, kind, ptr<void>(spectrum), ptr(d1), ptr(d2), m, scale, ptr(out), ptr<void>(ws),
                                     current_stream());
    }
    if (rc != SPINNER_OK) return refused(rc);
    return THPVariable_Wrap(std::move(out));
ENTRY_END

#define METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(apply_signs), METHOD(apply), METHOD(apply_blocks), METHOD(hash), METHOD(hash_signs), METHOD(sign_codes),
                         METHOD(sign_codes_signs), METHOD(angular_gram), METHOD(layer_forward), METHOD(layer_backward), METHOD(sketch),
                         METHOD(sketch_gram), METHOD(struct_apply_ws), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module_def); }
