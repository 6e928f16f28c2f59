// The common calls of matmul() and conv2d_nchw() over torch tensors, without
// the Python interpreter in between: a product of a few microseconds on the
// GPU waited for its caller, which spent 10 us in argument checks (2.3),
// torch.empty (1.7), the stream lookup (1.9) and ctypes around 3.3 us of
// launch; through this module it is 4.2 us.
//
// Both functions return the output tensor, or None for every call that is
// not the plain one (a tensor subclass, a transform or a dispatch mode is
// active, an operand of another device, type, shape or layout, an error
// status): the caller then takes the Python path, which checks and reports.
// Nothing is kept from one call to the next.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/xtc.h"

namespace {

// A plain strided tensor in GPU memory: an instance of torch.Tensor itself
// (or a Parameter) with no other dispatch key than the dense GPU backend's
// and autograd's.
bool plain(PyObject *o, const at::Tensor **out) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return false;
    const c10::DispatchKeySet usual({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA,
                                     c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutocastCUDA});
    if (t.key_set().raw_repr() & ~usual.raw_repr()) return false;
    *out = &t;
    return true;
}

bool modes_active() {
    return c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           at::impl::PythonTorchFunctionTLS::stack_len() > 0 ||
           (c10::impl::tls_local_dispatch_key_set().included_.raw_repr() &
            ~c10::DispatchKeySet({c10::DispatchKey::BackendSelect, c10::DispatchKey::ADInplaceOrView}).raw_repr());
}

bool dtype_code(const at::Tensor &t, xtc_dtype *code) {
    if (t.scalar_type() == at::kFloat) *code = XTC_F32;
    else if (t.scalar_type() == at::kBFloat16) *code = XTC_BF16;
    else return false;
    return true;
}

bool row_major(const at::Tensor &t) { return t.dim() == 2 && (t.size(1) <= 1 || t.stride(1) == 1); }

void *stream_of(const at::Tensor &t) {
    return static_cast<void *>(c10::hip::getCurrentHIPStream(t.device().index()).stream());
}

// matmul(a, b, out or None, relu)
PyObject *matmul(PyObject *, PyObject *const *args, Py_ssize_t n) {
    const at::Tensor *a, *b, *c = nullptr;
    xtc_dtype dt, dtb;
    if (n != 4 || modes_active() || !plain(args[0], &a) || !plain(args[1], &b) ||
        (args[2] != Py_None && !plain(args[2], &c)) || (args[3] != Py_True && args[3] != Py_False))
        Py_RETURN_NONE;
    if (!row_major(*a) || !row_major(*b) || !dtype_code(*a, &dt) || !dtype_code(*b, &dtb) || dt != dtb ||
        a->device() != b->device() || a->size(1) != b->size(0))
        Py_RETURN_NONE;
    const int64_t M = a->size(0), K = a->size(1), N = b->size(1);
    if (c && (!row_major(*c) || c->scalar_type() != at::kFloat || c->device() != a->device() ||
              c->size(0) != M || c->size(1) != N))
        Py_RETURN_NONE;
    try {
        at::Tensor fresh;
        if (!c) {
            fresh = at::empty({M, N}, at::TensorOptions().dtype(at::kFloat).device(a->device()));
            c = &fresh;
        }
        const int64_t lda = M > 1 ? a->stride(0) : (K > 1 ? K : 1), ldb = K > 1 ? b->stride(0) : (N > 1 ? N : 1),
                      ldc = M > 1 ? c->stride(0) : (N > 1 ? N : 1);
        const void *pa = a->data_ptr(), *pb = b->data_ptr();
        float *pc = static_cast<float *>(c->data_ptr());
        void *stream = stream_of(*a);
        xtc_status st;
        Py_BEGIN_ALLOW_THREADS
        st = (args[3] == Py_True ? xtc_matmul_relu : xtc_matmul)(M, N, K, pa, lda, pb, ldb, pc, ldc, dt, nullptr,
                                                                 stream);
        Py_END_ALLOW_THREADS
        if (st != XTC_OK) Py_RETURN_NONE;
        if (args[2] != Py_None) return Py_NewRef(args[2]);
        return THPVariable_Wrap(std::move(fresh));
    } catch (...) {
        Py_RETURN_NONE;   // the Python path meets the same error and reports it
    }
}

// An int, or a tuple of two ints.
bool pair_of(PyObject *o, int64_t *h, int64_t *w) {
    auto value = [](PyObject *v, int64_t *out) {
        if (!PyLong_CheckExact(v)) return false;
        int overflow = 0;
        *out = PyLong_AsLongLongAndOverflow(v, &overflow);
        return overflow == 0;
    };
    if (PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2)
        return value(PyTuple_GET_ITEM(o, 0), h) && value(PyTuple_GET_ITEM(o, 1), w);
    if (!value(o, h)) return false;
    *w = *h;
    return true;
}

// conv2d_nchw(x, w, stride, pad, out or None, relu)
PyObject *conv2d_nchw(PyObject *, PyObject *const *args, Py_ssize_t n) {
    const at::Tensor *x, *w, *y = nullptr;
    xtc_dtype dt, dtw;
    int64_t sh, sw, ph, pw;
    if (n != 6 || modes_active() || !plain(args[0], &x) || !plain(args[1], &w) || !pair_of(args[2], &sh, &sw) ||
        !pair_of(args[3], &ph, &pw) || (args[4] != Py_None && !plain(args[4], &y)) ||
        (args[5] != Py_True && args[5] != Py_False))
        Py_RETURN_NONE;
    if (x->dim() != 4 || w->dim() != 4 || !x->is_contiguous() || !w->is_contiguous() || !dtype_code(*x, &dt) ||
        !dtype_code(*w, &dtw) || dt != dtw || x->device() != w->device() || x->size(1) != w->size(1))
        Py_RETURN_NONE;
    const int64_t N = x->size(0), C = x->size(1), H = x->size(2), W = x->size(3), OC = w->size(0), R = w->size(2),
                  S = w->size(3);
    constexpr int64_t kLimit = int64_t(1) << 30;   // (also keeps the sums below inside 64 bits)
    if (sh < 1 || sw < 1 || ph < 0 || pw < 0 || sh > kLimit || sw > kLimit || ph > kLimit || pw > kLimit)
        Py_RETURN_NONE;
    if (R < 1 || S < 1 || H + 2 * ph < R || W + 2 * pw < S) Py_RETURN_NONE;
    const int64_t OH = (H + 2 * ph - R) / sh + 1, OW = (W + 2 * pw - S) / sw + 1;
    if (y && (y->dim() != 4 || !y->is_contiguous() || y->scalar_type() != at::kFloat || y->device() != x->device() ||
              y->size(0) != N || y->size(1) != OC || y->size(2) != OH || y->size(3) != OW))
        Py_RETURN_NONE;
    try {
        at::Tensor fresh;
        if (!y) {
            fresh = at::empty({N, OC, OH, OW}, at::TensorOptions().dtype(at::kFloat).device(x->device()));
            y = &fresh;
        }
        const void *px = x->data_ptr(), *pt = w->data_ptr();
        float *py = static_cast<float *>(y->data_ptr());
        void *stream = stream_of(*x);
        xtc_status st;
        Py_BEGIN_ALLOW_THREADS
        st = (args[5] == Py_True ? xtc_conv2d_nchw_relu : xtc_conv2d_nchw)(N, C, H, W, OC, R, S, sh, sw, ph, pw, px,
                                                                           pt, py, dt, nullptr, stream);
        Py_END_ALLOW_THREADS
        if (st != XTC_OK) Py_RETURN_NONE;
        if (args[4] != Py_None) return Py_NewRef(args[4]);
        return THPVariable_Wrap(std::move(fresh));
    } catch (...) {
        Py_RETURN_NONE;
    }
}

PyMethodDef kMethods[] = {
    {"matmul", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&matmul)), METH_FASTCALL,
     "matmul(a, b, out, relu): the product, or None where the general path has to run"},
    {"conv2d_nchw", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&conv2d_nchw)), METH_FASTCALL,
     "conv2d_nchw(x, w, stride, pad, out, relu): the convolution, or None likewise"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&kModule); }
