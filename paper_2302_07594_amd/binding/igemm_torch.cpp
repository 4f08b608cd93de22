// The tensor calls' native path: checks plain CUDA tensors, plans, takes a
// workspace from torch's caching allocator and makes the C call, in one step
// from Python. The same work in Python (attribute reads, two ctypes calls, the
// plan as a dict) took 13 to 14 us a call, more than most small and mid-size
// products take on the device.
//
// Each function returns the igemm status, or None for anything but the plain
// case (other types, layouts, devices or streams, tensor subclasses, transforms
// and modes in effect, empty products): the Python code then handles the call,
// with its own checks and messages.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/HIPContextLight.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <pybind11/gil.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "igemm.h"

namespace {

// A strided CUDA tensor of type dt with dim dimensions, not a subclass and
// under no functorch transform; nullptr otherwise.
const at::Tensor *plain(PyObject *o, at::ScalarType dt, int64_t dim) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != dt ||
        t.dim() != dim)
        return nullptr;
    static const c10::DispatchKeySet other(
        {c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
         c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
         c10::DispatchKey::Batched, c10::DispatchKey::Functionalize, c10::DispatchKey::Negative,
         c10::DispatchKey::Conjugate, c10::DispatchKey::ZeroTensor});
    return t.key_set().has_any(other) ? nullptr : &t;
}

// Leading dimension of a 2-D tensor with unit stride along rows (any stride
// for a single column), as the Python checks take it; false otherwise.
bool leading(const at::Tensor &t, int64_t *ld) {
    if (t.size(1) > 1 && t.stride(1) != 1) return false;
    *ld = t.size(0) > 1 ? t.stride(0) : (t.size(1) > 1 ? t.size(1) : 1);
    return true;
}

bool modes_active() {
    return c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           at::impl::PythonTorchFunctionTLS::stack_len() > 0;
}

// The stream of the current device if the tensors live there.
bool here(const at::Tensor &c, std::initializer_list<const at::Tensor *> others, void **stream) {
    const auto s = c10::hip::getCurrentHIPStreamMasqueradingAsCUDA();
    if (c.device() != s.device()) return false;
    for (const at::Tensor *t : others)
        if (t->device() != c.device()) return false;
    *stream = (void *)s.stream();
    return true;
}

int num_cu(const at::Tensor &c) {
    return at::cuda::getDeviceProperties(c.device().index())->multiProcessorCount;
}

// bytes of device memory from the caching allocator, 256-byte aligned.
at::Tensor workspace(const at::Tensor &c, int64_t bytes, void **p) {
    at::Tensor ws = at::empty({bytes + 256}, c.options().dtype(at::kByte));
    *p = (void *)(((uintptr_t)ws.data_ptr() + 255) & ~(uintptr_t)255);
    return ws;
}

bool as_i64(PyObject *o, int64_t *v) {
    if (!PyLong_Check(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool as_int(PyObject *o, int *v) {
    int64_t x;
    if (!as_i64(o, &x) || x != (int)x) return false;
    *v = (int)x;
    return true;
}
bool as_pair(PyObject *o, int64_t *a, int64_t *b) {
    return PyTuple_Check(o) && PyTuple_GET_SIZE(o) == 2 && as_i64(PyTuple_GET_ITEM(o, 0), a) &&
           as_i64(PyTuple_GET_ITEM(o, 1), b);
}

struct Product {
    const at::Tensor *a, *b, *c;
    int64_t m, n, k, lda, ldb, ldc;
    void *stream;
};

// A (m x k), B (k x n) of type et, C (m x n) of type ct, nothing empty.
bool product(PyObject *A, PyObject *B, PyObject *C, at::ScalarType et, at::ScalarType ct,
             Product *p) {
    p->a = plain(A, et, 2);
    p->b = p->a ? plain(B, et, 2) : nullptr;
    p->c = p->b ? plain(C, ct, 2) : nullptr;
    if (!p->c || modes_active()) return false;
    p->m = p->a->size(0);
    p->k = p->a->size(1);
    p->n = p->b->size(1);
    return p->m > 0 && p->n > 0 && p->k > 0 && p->b->size(0) == p->k && p->c->size(0) == p->m &&
           p->c->size(1) == p->n && leading(*p->a, &p->lda) && leading(*p->b, &p->ldb) &&
           leading(*p->c, &p->ldc) && here(*p->c, {p->a, p->b}, &p->stream);
}

// gemm(elem_bytes, A, B, C, kernel, split)
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    int es, kernel, split, st;
    Product p;
    if (nargs != 6 || !as_int(args[0], &es) || !as_int(args[4], &kernel) ||
        !as_int(args[5], &split) ||
        !product(args[1], args[2], args[3], es == 2 ? at::kShort : at::kChar, at::kInt, &p))
        Py_RETURN_NONE;
    {
        pybind11::gil_scoped_release no_gil;
        const void *A = p.a->data_ptr(), *B = p.b->data_ptr();
        int32_t *C = (int32_t *)p.c->data_ptr();
        igemm_plan plan;
        st = igemm_query_plan(es, p.m, p.n, p.k, A, p.lda, B, p.ldb, C, p.ldc, num_cu(*p.c),
                              kernel, split, &plan);
        at::Tensor ws;
        void *wp = nullptr;
        if (st == IGEMM_OK && plan.workspace_bytes > 0) ws = workspace(*p.c, plan.workspace_bytes, &wp);
        const int64_t wb = wp ? plan.workspace_bytes : 0;
        if (st == IGEMM_OK)
            st = es == 2 ? igemm_i16_ws(p.m, p.n, p.k, (const int16_t *)A, p.lda,
                                        (const int16_t *)B, p.ldb, C, p.ldc, p.stream, kernel,
                                        split, wp, wb)
                         : igemm_i8_ws(p.m, p.n, p.k, (const int8_t *)A, p.lda, (const int8_t *)B,
                                       p.ldb, C, p.ldc, p.stream, kernel, split, wp, wb);
        else
            st = INT_MIN;  // the plan's refusal: raised by the Python code
    }
    if (st == INT_MIN) Py_RETURN_NONE;
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// srs(A, B, C, kc, shift, round_half_up, kernel)
PyObject *srs(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    int64_t kc;
    int shift, kernel, st;
    Product p;
    if (nargs != 7 || !as_i64(args[3], &kc) || !as_int(args[4], &shift) ||
        !as_int(args[6], &kernel) || !THPVariable_CheckExact(args[0]))
        Py_RETURN_NONE;
    const int half_up = PyObject_IsTrue(args[5]);
    if (half_up < 0) return nullptr;
    const at::ScalarType et = THPVariable_Unpack(args[0]).scalar_type();
    if ((et != at::kShort && et != at::kChar) ||
        !product(args[0], args[1], args[2], et, at::kShort, &p))
        Py_RETURN_NONE;
    const int es = et == at::kShort ? 2 : 1;
    {
        pybind11::gil_scoped_release no_gil;
        const void *A = p.a->data_ptr(), *B = p.b->data_ptr();
        int16_t *C = (int16_t *)p.c->data_ptr();
        int64_t wb = 0;
        st = igemm_srs_query(es, p.m, p.n, p.k, A, p.lda, B, p.ldb, C, p.ldc, kc, num_cu(*p.c),
                             kernel, &wb);
        at::Tensor ws;
        void *wp = nullptr;
        if (st == IGEMM_OK && wb > 0) ws = workspace(*p.c, wb, &wp);
        if (st == IGEMM_OK)
            st = igemm_srs_ws(es, p.m, p.n, p.k, A, p.lda, B, p.ldb, C, p.ldc, kc, shift, half_up,
                              p.stream, kernel, wp, wb);
        else
            st = INT_MIN;
    }
    if (st == INT_MIN) Py_RETURN_NONE;
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// packed_b(elem_bytes, A, packed_b, packed_b_bytes, n, k, C, kernel)
PyObject *packed_b(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    int es, kernel, st;
    int64_t pb_bytes, n, k, lda, ldc;
    void *stream;
    if (nargs != 8 || !as_int(args[0], &es) || !as_i64(args[3], &pb_bytes) ||
        !as_i64(args[4], &n) || !as_i64(args[5], &k) || !as_int(args[7], &kernel))
        Py_RETURN_NONE;
    const at::Tensor *a = plain(args[1], es == 2 ? at::kShort : at::kChar, 2);
    const at::Tensor *pb = a ? plain(args[2], at::kByte, 1) : nullptr;
    const at::Tensor *c = pb ? plain(args[6], at::kInt, 2) : nullptr;
    if (!c || modes_active() || n <= 0 || k <= 0 || a->size(0) <= 0 || a->size(1) != k ||
        c->size(0) != a->size(0) || c->size(1) != n || !leading(*a, &lda) || !leading(*c, &ldc) ||
        !here(*c, {a, pb}, &stream))
        Py_RETURN_NONE;
    const int64_t m = a->size(0);
    {
        pybind11::gil_scoped_release no_gil;
        const void *A = a->data_ptr(), *PB = pb->data_ptr();
        int32_t *C = (int32_t *)c->data_ptr();
        const void *fake = (const void *)(uintptr_t)4096;  // B was consumed by the pack call
        igemm_plan plan;
        st = igemm_query_plan(es, m, n, k, A, lda, fake, n, C, ldc, num_cu(*c), kernel, -1, &plan);
        at::Tensor ws;
        void *wp = nullptr;
        if (st == IGEMM_OK && plan.packed_a_bytes > 0) ws = workspace(*c, plan.packed_a_bytes, &wp);
        const int64_t wb = wp ? plan.packed_a_bytes : 0;
        if (st == IGEMM_OK)
            st = es == 2 ? igemm_i16_packed_b(m, n, k, (const int16_t *)A, lda, PB, pb_bytes, C,
                                              ldc, kernel, wp, wb, stream)
                         : igemm_i8_packed_b(m, n, k, (const int8_t *)A, lda, PB, pb_bytes, C, ldc,
                                             kernel, wp, wb, stream);
        else
            st = INT_MIN;
    }
    if (st == INT_MIN) Py_RETURN_NONE;
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// conv2d(X, W, Y, stride, pad, dil, kernel, split)
PyObject *conv2d(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    igemm_conv2d_desc d;
    int kernel, split, st;
    void *stream;
    if (nargs != 8 || !as_pair(args[3], &d.stride_h, &d.stride_w) ||
        !as_pair(args[4], &d.pad_h, &d.pad_w) || !as_pair(args[5], &d.dil_h, &d.dil_w) ||
        !as_int(args[6], &kernel) || !as_int(args[7], &split) || !THPVariable_CheckExact(args[0]))
        Py_RETURN_NONE;
    const at::ScalarType et = THPVariable_Unpack(args[0]).scalar_type();
    if (et != at::kShort && et != at::kChar) Py_RETURN_NONE;
    const at::Tensor *x = plain(args[0], et, 4);
    const at::Tensor *w = x ? plain(args[1], et, 4) : nullptr;
    const at::Tensor *y = w ? plain(args[2], at::kInt, 4) : nullptr;
    if (!y || modes_active() || !x->is_contiguous() || !w->is_contiguous() ||
        !y->is_contiguous() || y->numel() == 0 || x->numel() == 0 || w->numel() == 0 ||
        !here(*y, {x, w}, &stream))
        Py_RETURN_NONE;
    d.n = x->size(0);
    d.h = x->size(1);
    d.w = x->size(2);
    d.c = x->size(3);
    d.r = w->size(0);
    d.s = w->size(1);
    d.k = w->size(3);
    if (w->size(2) != d.c || y->size(0) != d.n || y->size(3) != d.k ||
        y->size(1) != igemm_conv2d_out_dim(d.h, d.r, d.stride_h, d.pad_h, d.dil_h) ||
        y->size(2) != igemm_conv2d_out_dim(d.w, d.s, d.stride_w, d.pad_w, d.dil_w))
        Py_RETURN_NONE;
    {
        pybind11::gil_scoped_release no_gil;
        st = igemm_conv2d_ex(et == at::kShort ? 2 : 1, &d, x->data_ptr(), w->data_ptr(),
                             (int32_t *)y->data_ptr(), stream, kernel, split);
    }
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

#define IGEMM_FAST(f) (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"gemm", IGEMM_FAST(gemm)},
                         {"srs", IGEMM_FAST(srs)},
                         {"packed_b", IGEMM_FAST(packed_b)},
                         {"conv2d", IGEMM_FAST(conv2d)},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_igemm_torch", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__igemm_torch(void) { return PyModule_Create(&module); }
