// Python calls into libxgemm without ctypes and without per-call Python code.
//
// A call of gemm() spent about 6 us in Python and ctypes before its first
// launch, as long as the GPU needs for 512^3.  The functions here read the
// tensors' fields directly and call the library's entry points (bound once,
// by address, from the library that ctypes loaded).  They take the plain
// case only and answer None otherwise: any other argument (another type,
// layout or device, a subclass, a missing handle) goes the Python way, which
// handles or refuses it.  The GIL is released around each library call, as
// ctypes does.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>

#include <stdint.h>

namespace {

typedef int (*gemm_fn)(void *, int64_t, int64_t, int64_t, const void *, int64_t, const void *, int64_t, float *,
                       int64_t, int, void *);
typedef int (*batched_fn)(void *, int64_t, int64_t, int64_t, int64_t, const void *, int64_t, int64_t, const void *,
                          int64_t, int64_t, float *, int64_t, int64_t, int, void *);
typedef int (*gemv_fn)(void *, int64_t, int64_t, const float *, int64_t, const float *, float *, void *);

gemm_fn f_run, f_noalloc;
batched_fn f_batched;
gemv_fn f_gemv;
PyObject *handles;  // the module's dict: (device index, stream address) -> handle address

PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long run, noalloc, batched, gemv;
    PyObject *d;
    if (!PyArg_ParseTuple(args, "KKKKO!", &run, &noalloc, &batched, &gemv, &PyDict_Type, &d))
        return nullptr;
    f_run = (gemm_fn)run;
    f_noalloc = (gemm_fn)noalloc;
    f_batched = (batched_fn)batched;
    f_gemv = (gemv_fn)gemv;
    Py_INCREF(d);
    Py_XDECREF(handles);
    handles = d;
    Py_RETURN_NONE;
}

// The tensor behind o if it is a plain strided GPU tensor (no subclass, no
// transform or mode that would look at its accesses).
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet allowed({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView,
                                              c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA});
    if (!t.defined() || (t.key_set().raw_repr() & ~allowed.raw_repr()) != 0 || !t.is_cuda() || !t.has_storage())
        return nullptr;
    return &t;
}

int code_of(const at::Tensor &t)
{
    return t.scalar_type() == at::kBFloat16 ? 0 : t.scalar_type() == at::kHalf ? 1 : -1;
}

// Leading dimension of the matrix in dimensions d and d + 1, or -1 if its
// rows are not contiguous.
int64_t leading(const at::Tensor &t, int d)
{
    const int64_t rows = t.size(d), cols = t.size(d + 1);
    if (cols > 1 && t.stride(d + 1) != 1)
        return -1;
    return rows <= 1 ? std::max(cols, t.stride(d)) : t.stride(d);
}

void *data(const at::Tensor &t) { return t.numel() == 0 ? nullptr : t.mutable_data_ptr(); }

// The stream of a call and the handle the module owns for it.
bool stream_handle(const at::Tensor &t, void **stream, void **handle)
{
    const auto dev = t.device().index();
    *stream = (void *)c10::hip::getCurrentHIPStream(dev).stream();
    PyObject *key = Py_BuildValue("(iK)", (int)dev, (unsigned long long)(uintptr_t)*stream);
    if (!key)
        return false;
    PyObject *h = PyDict_GetItem(handles, key);
    Py_DECREF(key);
    if (!h || !PyLong_Check(h))
        return false;
    *handle = PyLong_AsVoidPtr(h);
    return *handle != nullptr;
}

#define DECLINE                \
    do {                       \
        PyErr_Clear();         \
        Py_RETURN_NONE;        \
    } while (0)

PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 3 || !handles)
        Py_RETURN_NONE;
    const at::Tensor *A = plain(a[0]), *B = plain(a[1]), *C = plain(a[2]);
    if (!A || !B || !C || A->dim() != 2 || B->dim() != 2 || C->dim() != 2 || C->scalar_type() != at::kFloat ||
        A->device() != B->device() || A->device() != C->device())
        Py_RETURN_NONE;
    const int code = code_of(*A);
    const int64_t M = A->size(0), K = A->size(1), N = B->size(1);
    const int64_t lda = leading(*A, 0), ldb = leading(*B, 0), ldc = leading(*C, 0);
    void *stream, *h;
    if (code < 0 || code_of(*B) != code || B->size(0) != K || C->size(0) != M || C->size(1) != N || lda < 0 ||
        ldb < 0 || ldc < 0 || !stream_handle(*A, &stream, &h))
        DECLINE;
    const void *pa = data(*A), *pb = data(*B);
    float *pc = (float *)data(*C);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f_run(h, M, N, K, pa, lda, pb, ldb, pc, ldc, code, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject *bmm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 3 || !handles)
        Py_RETURN_NONE;
    const at::Tensor *A = plain(a[0]), *B = plain(a[1]), *C = plain(a[2]);
    if (!A || !B || !C || A->dim() != 3 || B->dim() != 3 || C->dim() != 3 || C->scalar_type() != at::kFloat ||
        A->device() != B->device() || A->device() != C->device())
        Py_RETURN_NONE;
    const int code = code_of(*A);
    const int64_t L = A->size(0), M = A->size(1), K = A->size(2), N = B->size(2);
    void *stream, *h;
    if (code < 0 || code_of(*B) != code || B->size(0) != L || B->size(1) != K || C->size(0) != L || C->size(1) != M ||
        C->size(2) != N || (K > 1 && A->stride(2) != 1) || (N > 1 && (B->stride(2) != 1 || C->stride(2) != 1)) ||
        !stream_handle(*A, &stream, &h))
        DECLINE;
    const int64_t one = 1;
    const int64_t lda = M > 1 ? A->stride(1) : std::max(K, one), ldb = K > 1 ? B->stride(1) : std::max(N, one),
                  ldc = M > 1 ? C->stride(1) : std::max(N, one);
    const int64_t sa = L > 1 ? A->stride(0) : 0, sb = L > 1 ? B->stride(0) : 0, sc = L > 1 ? C->stride(0) : 0;
    const void *pa = data(*A), *pb = data(*B);
    float *pc = (float *)data(*C);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f_batched(h, L, M, N, K, pa, lda, sa, pb, ldb, sb, pc, ldc, sc, code, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject *gemv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 3 || !handles)
        Py_RETURN_NONE;
    const at::Tensor *A = plain(a[0]), *x = plain(a[1]), *y = plain(a[2]);
    if (!A || !x || !y || A->dim() != 2 || x->dim() != 1 || y->dim() != 1 || A->scalar_type() != at::kFloat ||
        x->scalar_type() != at::kFloat || y->scalar_type() != at::kFloat || A->device() != x->device() ||
        A->device() != y->device())
        Py_RETURN_NONE;
    const int64_t M = A->size(0), K = A->size(1);
    void *stream, *h;
    if (x->size(0) != K || y->size(0) != M || !x->is_contiguous() || !y->is_contiguous() ||
        (M > 0 && K > 1 && A->stride(1) != 1) || !stream_handle(*A, &stream, &h))
        DECLINE;
    const int64_t one = 1, lda = M > 1 ? A->stride(0) : std::max(K, one);
    const float *pa = (const float *)data(*A), *px = (const float *)data(*x);
    float *py = (float *)data(*y);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f_gemv(h, M, K, pa, lda, px, py, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// xgemm_run / xgemm_run_noalloc on twelve plain integers (addresses may be
// None); anything else is declined.
PyObject *twelve(gemm_fn f, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12 || !f)
        Py_RETURN_NONE;
    long long v[12];
    for (int i = 0; i < 12; ++i) {
        const bool address = i == 0 || i == 4 || i == 6 || i == 8 || i == 11;
        if (address && a[i] == Py_None) {
            v[i] = 0;
            continue;
        }
        if (!PyLong_CheckExact(a[i]))
            Py_RETURN_NONE;
        int overflow = 0;
        v[i] = PyLong_AsLongLongAndOverflow(a[i], &overflow);
        if (overflow || (address && v[i] < 0) || (i == 10 && (v[i] < INT32_MIN || v[i] > INT32_MAX)))
            DECLINE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f((void *)v[0], v[1], v[2], v[3], (const void *)v[4], v[5], (const void *)v[6], v[7], (float *)v[8], v[9],
           (int)v[10], (void *)v[11]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject *run(PyObject *, PyObject *const *a, Py_ssize_t n) { return twelve(f_run, a, n); }
PyObject *run_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n) { return twelve(f_noalloc, a, n); }

// no C++ exception crosses into Python's C frames
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (...) {
        DECLINE;
    }
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "Entry point addresses and the handle dict."},
    {"gemm", (PyCFunction)(void *)guarded<gemm>, METH_FASTCALL, "xgemm_run on (A, B, out): a status, or None."},
    {"bmm", (PyCFunction)(void *)guarded<bmm>, METH_FASTCALL, "The strided batched call on (A, B, out)."},
    {"gemv", (PyCFunction)(void *)guarded<gemv>, METH_FASTCALL, "xgemv_run on (A, x, out)."},
    {"run", (PyCFunction)(void *)guarded<run>, METH_FASTCALL, "xgemm_run on its twelve arguments."},
    {"run_noalloc", (PyCFunction)(void *)guarded<run_noalloc>, METH_FASTCALL, "xgemm_run_noalloc likewise."},
    {nullptr, nullptr, 0, nullptr},
};

// (the module's docstring says what it was built for: see build.py)
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", XGEMM_FASTCALL_TAG, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
