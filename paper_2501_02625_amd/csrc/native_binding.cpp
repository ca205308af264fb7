// Native half of the Python binding: argument marshalling, output allocation and the call into libhalo's C ABI in one step.
//
// What it is for: a small layer's step is bound by the host.  Through ctypes one forward call cost 19.5 us, of which only
// 5 us are the two kernel launches: five torch.empty (1.7 us each), the current stream (2.9 us) and the conversion of the
// arguments make up the rest.  Here a tensor costs 0.4 us (the caching allocator called directly) and the stream 0.15 us.
//
// Every function takes positional arguments, tensors or None, and returns the outputs, or the halo_status of a failed call
// as an int.  binding.py holds the public signatures and documentation.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/EmptyTensor.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/Allocator.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include "halo.h"

namespace {

PyObject* g_get_device = nullptr;       // torch._C._cuda_getDevice
PyObject* g_get_raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream

PyObject* g_out_of_memory = nullptr;    // torch.OutOfMemoryError

struct Failed {};                       // a Python exception is set

const at::Tensor* tensor(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "expected a tensor or None");
        throw Failed();
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda()) {
        PyErr_SetString(PyExc_ValueError, "libhalo takes device tensors only");
        throw Failed();
    }
    return &t;
}

void require(bool ok, const char* what) {
    if (ok) return;
    PyErr_SetString(PyExc_AssertionError, what);
    throw Failed();
}

long integer(PyObject* o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failed();
    return v;
}

void* data(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
size_t bytes(const at::Tensor* t) { return t ? (size_t)t->numel() : 0; }      // workspaces are uint8

// True if at::empty would do nothing but allocate: no dispatch mode, functorch transform or tracer sees tensors being made.
bool plain_creation() {
    const c10::DispatchKeySet on = c10::impl::tls_local_dispatch_key_set().included_;
    return (on - c10::default_included_set - c10::autocast_dispatch_keyset).empty();
}

at::Tensor new_tensor(at::IntArrayRef size, at::ScalarType dtype, const at::Tensor& like, int current_device) {
    if (!plain_creation() || like.device().index() != current_device)
        return at::empty(size, at::TensorOptions().dtype(dtype).device(like.device()));
    // the allocator that torch.empty uses for device memory, taken from a tensor that it made
    static c10::Allocator* const allocator =
        at::empty({1}, at::TensorOptions().dtype(at::kByte).device(like.device())).storage().allocator();
    if (!allocator) return at::empty(size, at::TensorOptions().dtype(dtype).device(like.device()));
    return at::Tensor(at::detail::empty_generic(size, allocator, c10::DispatchKeySet(c10::DispatchKey::CUDA), dtype,
                                                std::nullopt));
}

// [rows, cols] whose row pitch is a multiple of 16 bytes (the ABI's alignment rule).
at::Tensor new_padded(int64_t rows, int64_t cols, at::ScalarType dtype, const at::Tensor& like, int device) {
    const int64_t per16 = 16 / (int64_t)c10::elementSize(dtype);
    int64_t ld = (cols + per16 - 1) / per16 * per16;
    if (ld < per16) ld = per16;
    at::Tensor t = new_tensor({rows, ld}, dtype, like, device);
    return ld == cols ? t : t.narrow(1, 0, cols);
}

struct Context {
    int device;
    void* stream;
    Context() {
        PyObject* d = PyObject_CallNoArgs(g_get_device);
        if (!d) throw Failed();
        PyObject* s = PyObject_CallOneArg(g_get_raw_stream, d);
        device = (int)PyLong_AsLong(d);
        Py_DECREF(d);
        if (!s) throw Failed();
        stream = PyLong_AsVoidPtr(s);
        Py_DECREF(s);
    }
};

// The halo_linear_desc inside a ctypes structure.
struct Desc {
    Py_buffer view;
    const halo_linear_desc* d;
    explicit Desc(PyObject* o) {
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Failed();
        d = reinterpret_cast<const halo_linear_desc*>(view.buf);
        if ((size_t)view.len != sizeof(halo_linear_desc)) {
            PyBuffer_Release(&view);
            PyErr_SetString(PyExc_TypeError, "expected a LinearDesc");
            throw Failed();
        }
    }
    ~Desc() { PyBuffer_Release(&view); }
    Desc(const Desc&) = delete;
    at::ScalarType out_type() const { return d->out_dt == HALO_BF16 ? at::kBFloat16 : at::kFloat; }
};

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
PyObject* wrap_or_none(bool want, const at::Tensor& t) {
    if (want) return THPVariable_Wrap(t);
    Py_RETURN_NONE;
}

// The given output, or a new one.
at::Tensor output(const at::Tensor* given, bool want, at::IntArrayRef size, at::ScalarType dtype, const at::Tensor& like,
                  const Context& c) {
    if (given) return *given;
    return want ? new_tensor(size, dtype, like, c.device) : at::Tensor();
}
void* data(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

bool bf16(const at::Tensor* t) { return t->scalar_type() == at::kBFloat16; }

// f(args...) with the interpreter lock released.  The pointers are arguments, so they are taken before the release: a tensor
// without storage (inside a functorch transform) makes data_ptr() throw, and the handler in entry() needs the lock.
struct ReleaseGil {
    PyThreadState* state = PyEval_SaveThread();
    ~ReleaseGil() { PyEval_RestoreThread(state); }
};
template <class... P, class... A>
halo_status without_gil(halo_status (*f)(P...), A... args) {
    const ReleaseGil released;
    return f(args...);
}

// desc, X, W, Xq, s_x, Wq, s_w, Y, workspace, new_state.  new_state: the caller has no state, the codes and scales are made
// here; otherwise a missing member of its state goes to the C ABI as the null pointer that it is, and is refused there.
PyObject* linear_fwd(PyObject* const* a) {
    const Desc desc(a[0]);
    const halo_linear_desc& d = *desc.d;
    const at::Tensor *X = tensor(a[1]), *W = tensor(a[2]), *xq = tensor(a[3]), *sx = tensor(a[4]), *wq = tensor(a[5]),
                     *sw = tensor(a[6]), *y = tensor(a[7]), *ws = tensor(a[8]);
    const bool make = a[9] == Py_True;
    const at::Tensor* like = X ? X : xq;
    require(like != nullptr, "X or a state is needed");
    require((!X || (bf16(X) && X->is_contiguous())) && (!W || (bf16(W) && W->is_contiguous())), "X and W are contiguous bf16");
    const Context c;
    const at::Tensor Xq = output(xq, make, {d.b, d.m}, at::kChar, *like, c), s_x = output(sx, make, {d.b}, at::kFloat, *like, c),
                     Wq = output(wq, make, {d.n, d.m}, at::kChar, *like, c), s_w = output(sw, make, {d.n}, at::kFloat, *like, c),
                     Y = output(y, true, {d.b, d.n}, desc.out_type(), *like, c);
    at::Tensor scratch;
    if (!ws && d.scale_mode == HALO_SCALE_PER_TENSOR) {
        const size_t need = halo_linear_workspace_bytes(&d);
        scratch = new_tensor({(int64_t)(need > 16 ? need : 16)}, at::kByte, *like, c.device);
        ws = &scratch;
    }
    const halo_status st = without_gil(
        halo_linear_fwd, &d, data(X), data(W), data(Y), (int8_t*)data(Xq), (float*)data(s_x), (int8_t*)data(Wq),
        (float*)data(s_w), data(ws), bytes(ws), c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NNNNN)", wrap(Y), wrap(Xq), wrap(s_x), wrap(Wq), wrap(s_w));
}

// desc, E, Xq, s_x, Wq, s_w, want_ex, want_g, workspace, EX, G
PyObject* linear_bwd(PyObject* const* a) {
    const Desc desc(a[0]);
    const halo_linear_desc& d = *desc.d;
    const at::Tensor *E = tensor(a[1]), *Xq = tensor(a[2]), *s_x = tensor(a[3]), *Wq = tensor(a[4]), *s_w = tensor(a[5]),
                     *ws = tensor(a[8]), *ex = tensor(a[9]), *g = tensor(a[10]);
    const bool want_ex = a[6] == Py_True, want_g = a[7] == Py_True;
    require(E && bf16(E) && E->is_contiguous(), "E is contiguous bf16");
    const Context c;
    const at::Tensor EX = output(ex, want_ex, {d.b, d.m}, desc.out_type(), *E, c),
                     G = output(g, want_g, {d.n, d.m}, desc.out_type(), *E, c);
    at::Tensor scratch;
    if (!ws) {
        const size_t need = halo_linear_workspace_bytes(&d);
        scratch = new_tensor({(int64_t)(need > 1 ? need : 1)}, at::kByte, *E, c.device);
        ws = &scratch;
    }
    const halo_status st = without_gil(
        halo_linear_bwd, &d, data(E), (int8_t*)data(Xq), (float*)data(s_x), (int8_t*)data(Wq), (float*)data(s_w),
        want_ex ? data(EX) : nullptr, want_g ? data(G) : nullptr, data(ws), bytes(ws), c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap_or_none(want_ex, EX), wrap_or_none(want_g, G));
}

// desc, X, Wq, s_w, U, V, workspace, Y, T
PyObject* peft_fwd(PyObject* const* a) {
    const Desc desc(a[0]);
    const halo_linear_desc& d = *desc.d;
    const at::Tensor *X = tensor(a[1]), *Wq = tensor(a[2]), *s_w = tensor(a[3]), *U = tensor(a[4]), *V = tensor(a[5]),
                     *ws = tensor(a[6]), *y = tensor(a[7]), *t = tensor(a[8]);
    require(X && Wq && s_w && U && V && bf16(X) && bf16(U) && bf16(V), "X, U and V are bf16");
    require(X->is_contiguous() && U->is_contiguous() && V->is_contiguous() && Wq->is_contiguous(), "operands are contiguous");
    require(U->dim() == 2 && V->dim() == 2 && V->size(0) == d.n && V->size(1) == U->size(0) && U->size(1) == d.m,
            "U is [rank, m] and V [n, rank]");
    const int64_t rank = U->size(0);
    const Context c;
    const at::Tensor Y = output(y, true, {d.b, d.n}, desc.out_type(), *X, c), T = output(t, true, {d.b, rank}, at::kFloat, *X, c);
    at::Tensor scratch;
    if (!ws) {
        const size_t need = halo_peft_workspace_bytes(&d, (int32_t)rank);
        scratch = new_tensor({(int64_t)(need > 1 ? need : 1)}, at::kByte, *X, c.device);
        ws = &scratch;
    }
    const halo_status st = without_gil(
        halo_peft_fwd, &d, (int32_t)rank, data(X), (int8_t*)data(Wq), (float*)data(s_w), data(U), data(V), data(Y),
        (float*)data(T), data(ws), bytes(ws), c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap(Y), wrap(T));
}

// desc, E, X, T, Wq, s_w, U, V, want_ex, want_gu, want_gv, workspace, EX, GU, GV
PyObject* peft_bwd(PyObject* const* a) {
    const Desc desc(a[0]);
    const halo_linear_desc& d = *desc.d;
    const at::Tensor *E = tensor(a[1]), *X = tensor(a[2]), *T = tensor(a[3]), *Wq = tensor(a[4]), *s_w = tensor(a[5]),
                     *U = tensor(a[6]), *V = tensor(a[7]), *ws = tensor(a[11]), *ex = tensor(a[12]), *gu = tensor(a[13]),
                     *gv = tensor(a[14]);
    const bool want_ex = a[8] == Py_True, want_gu = a[9] == Py_True, want_gv = a[10] == Py_True;
    require(U && U->dim() == 2 && E && bf16(E) && E->is_contiguous(), "E is contiguous bf16");
    const int64_t rank = U->size(0);
    const Context c;
    const at::Tensor EX = output(ex, want_ex, {d.b, d.m}, desc.out_type(), *E, c),
                     GU = output(gu, want_gu, {rank, d.m}, at::kFloat, *E, c),
                     GV = output(gv, want_gv, {d.n, rank}, at::kFloat, *E, c);
    at::Tensor scratch;
    if (!ws) {
        const size_t need = halo_peft_workspace_bytes(&d, (int32_t)rank);
        scratch = new_tensor({(int64_t)(need > 1 ? need : 1)}, at::kByte, *E, c.device);
        ws = &scratch;
    }
    const halo_status st = without_gil(
        halo_peft_bwd, &d, (int32_t)rank, data(E), data(X), (float*)data(T), (int8_t*)data(Wq), (float*)data(s_w), data(U),
        data(V), want_ex ? data(EX) : nullptr, want_gu ? (float*)data(GU) : nullptr, want_gv ? (float*)data(GV) : nullptr,
        data(ws), bytes(ws), c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NNN)", wrap_or_none(want_ex, EX), wrap_or_none(want_gu, GU), wrap_or_none(want_gv, GV));
}

// x, had_block, out_codes, out_scales
PyObject* mx6_quant(PyObject* const* a) {
    const at::Tensor *x = tensor(a[0]), *codes = tensor(a[2]), *scales = tensor(a[3]);
    require(x && x->dim() == 2 && x->stride(1) == 1 && bf16(x), "x is a bf16 matrix with contiguous rows");
    const int64_t rows = x->size(0), cols = x->size(1);
    const int32_t block = (int32_t)integer(a[1]);
    const Context c;
    const at::Tensor q = output(codes, true, {rows, cols / 32 * 24}, at::kByte, *x, c),
                     s = output(scales, true, {rows, cols / 32}, at::kByte, *x, c);
    const halo_status st = without_gil(
        halo_mx6_quant, data(x), rows, cols, rows ? x->stride(0) : cols, block, (uint8_t*)data(q), rows ? q.stride(0) : 24,
        (uint8_t*)data(s), rows ? s.stride(0) : 1, c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap(q), wrap(s));
}

at::ScalarType out_dtype(long code) { return code == HALO_BF16 ? at::kBFloat16 : at::kFloat; }
halo_dtype dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kBFloat16) return HALO_BF16;
    if (t.scalar_type() == at::kFloat) return HALO_F32;
    PyErr_SetString(PyExc_TypeError, "HALO tensors are bf16 or fp32");
    throw Failed();
}

// a, sa, b, sb, dtype of a new output, out
PyObject* gemm_mx6(PyObject* const* a) {
    const at::Tensor *A = tensor(a[0]), *sa = tensor(a[1]), *B = tensor(a[2]), *sb = tensor(a[3]), *out = tensor(a[5]);
    require(A && sa && B && sb && A->dim() == 2 && B->dim() == 2 && sa->dim() == 2 && sb->dim() == 2, "operands are matrices");
    const int64_t M = A->size(0), N = B->size(0), K = sa->size(1) * 32;
    require(A->size(1) == K / 32 * 24 && B->size(1) == K / 32 * 24 && sb->size(1) * 32 == K, "codes and scales fit together");
    const long code = integer(a[4]);
    const Context c;
    const at::Tensor C = out ? *out : new_padded(M, N, out_dtype(code), *A, c.device);
    const halo_dtype dt = dtype_code(C);
    const halo_status st = without_gil(
        halo_gemm_mx6, (uint8_t*)data(A), M ? A->stride(0) : 24, (uint8_t*)data(sa), M ? sa->stride(0) : 4, (uint8_t*)data(B),
        N ? B->stride(0) : 24, (uint8_t*)data(sb), N ? sb->stride(0) : 4, M, N, K, data(C), dt, M ? C.stride(0) : N, c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return wrap(C);
}

// x, axis, had_block, had_block_left, fold, out_q, out_scale, workspace
PyObject* hadamard_quant(PyObject* const* a) {
    const at::Tensor *x = tensor(a[0]), *fold = tensor(a[4]), *oq = tensor(a[5]), *os = tensor(a[6]), *ws = tensor(a[7]);
    require(x && x->dim() == 2 && x->stride(1) == 1, "x is a matrix with contiguous rows");
    const int64_t rows = x->size(0), cols = x->size(1);
    const halo_axis axis = (halo_axis)integer(a[1]);
    const int32_t block = (int32_t)integer(a[2]), left = (int32_t)integer(a[3]);
    const int64_t qr = axis == HALO_QUANT_ROWS ? rows : cols, qc = axis == HALO_QUANT_ROWS ? cols : rows;
    const halo_dtype dt = dtype_code(*x);
    const Context c;
    const at::Tensor q = oq ? *oq : new_padded(qr, qc, at::kChar, *x, c.device), s = output(os, true, {qr}, at::kFloat, *x, c);
    const size_t need = halo_hadamard_quant_workspace_bytes(rows, cols, axis, left);
    at::Tensor scratch;
    if (!ws && need) {
        scratch = new_tensor({(int64_t)need}, at::kByte, *x, c.device);
        ws = &scratch;
    }
    const halo_status st = without_gil(
        halo_hadamard_quant, data(x), dt, rows, cols, rows ? x->stride(0) : cols, axis, block, left, (float*)data(fold),
        (int8_t*)data(q), q.numel() ? q.stride(0) : qc, (float*)data(s), data(ws), bytes(ws), c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap(q), wrap(s));
}

// a, b, trans_b, row_scale, col_scale, dtype of a new output (-1: none), want_acc, out, acc_out
PyObject* gemm_i8(PyObject* const* a) {
    const at::Tensor *A = tensor(a[0]), *B = tensor(a[1]), *rs = tensor(a[3]), *cs = tensor(a[4]), *out = tensor(a[7]),
                     *acc = tensor(a[8]);
    require(A && B && A->scalar_type() == at::kChar && B->scalar_type() == at::kChar && A->dim() == 2 && B->dim() == 2,
            "operands are int8 matrices");
    const bool trans = PyObject_IsTrue(a[2]) != 0, want_acc = PyObject_IsTrue(a[6]) != 0;
    const int64_t M = A->size(0), K = A->size(1), N = B->size(trans ? 0 : 1);
    require(B->size(trans ? 1 : 0) == K, "operands fit together");
    const long code = integer(a[5]);
    const Context c;
    at::Tensor C = out ? *out : (code >= 0 ? new_padded(M, N, out_dtype(code), *A, c.device) : at::Tensor());
    at::Tensor S = acc ? *acc : (want_acc ? new_padded(M, N, at::kInt, *A, c.device) : at::Tensor());
    const halo_dtype dt = C.defined() ? dtype_code(C) : HALO_F32;
    const halo_status st = without_gil(
        halo_gemm_i8, (int8_t*)data(A), M ? A->stride(0) : K, (int8_t*)data(B), B->size(0) ? B->stride(0) : B->size(1),
        trans ? 1 : 0, M, N, K, (float*)data(rs), (float*)data(cs), data(C), dt, C.defined() ? (M ? C.stride(0) : N) : 0,
        (int32_t*)data(S), S.defined() ? (M ? S.stride(0) : N) : 0, c.stream);
    if (st != HALO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap_or_none(C.defined(), C), wrap_or_none(S.defined(), S));
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t count) {
    if (count != N) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", N, count);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Failed&) {
        return nullptr;
    } catch (const c10::OutOfMemoryError& e) {
        PyErr_SetString(g_out_of_memory, e.what_without_backtrace());
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define HALO_ENTRY(F, N) {#F, (PyCFunction)(void (*)(void))entry<F, N>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HALO_ENTRY(linear_fwd, 10), HALO_ENTRY(linear_bwd, 11), HALO_ENTRY(peft_fwd, 9), HALO_ENTRY(peft_bwd, 15),
                         HALO_ENTRY(mx6_quant, 4),  HALO_ENTRY(gemm_mx6, 6),    HALO_ENTRY(hadamard_quant, 8),
                         HALO_ENTRY(gemm_i8, 9),    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_halo_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__halo_native(void) {
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_get_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    g_out_of_memory = PyObject_GetAttrString(c, "OutOfMemoryError");
    Py_DECREF(c);
    if (!g_out_of_memory || !g_get_device || !g_get_raw_stream) return nullptr;
    return PyModule_Create(&module);
}
