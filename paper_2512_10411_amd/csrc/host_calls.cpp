// The way from torch tensors to libswaa's C entry points in native code, for calls in plain form: torch's own dense
// GPU tensors, all on the device that is current, results to be allocated, torch's current stream, no mode
// or transform of torch in between.  Whatever else a call is, these functions return None, and the binding's Python takes
// it, with its checks, messages and streams; so this file refuses nothing and reports nothing by itself.
//
// A prompt of 64 tokens took 8.9 us a call and takes 5.7, decode of 682 tokens 14.2 and 8.4: argument checks, two results
// from torch's allocator and the foreign-function call each cost about as much in Python as the launch.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/version.h>

#include <cmath>
#include <cstring>

#include "swaa.h"

namespace {

// libswaa's entry points: addresses from the library that the binding has loaded.
decltype(&swaa_attn_fwd) fwd_entry;
decltype(&swaa_attn_fwd_fa_decode) fwd_fa_decode_entry;
decltype(&swaa_attn_decode) decode_entry;
decltype(&swaa_attn_decode_workspace_bytes) decode_workspace_entry;
decltype(&swaa_attn_decode_ex) decode_ex_entry;
decltype(&swaa_attn_decode_ex_workspace_bytes) decode_ex_workspace_entry;

// Does nothing of torch stand between a call and its tensors (function or dispatch modes, transforms, tracing)?
bool nothing_between() {
    return at::impl::PythonTorchFunctionTLS::stack_len() == 0 && !c10::impl::dispatch_mode_enabled() &&
           (c10::impl::tls_local_dispatch_key_set().included_.raw_repr() & ~c10::default_included_set.raw_repr()) == 0;
}

// torch's current device and the handle of its current stream (Python's torch._C._cuda_getDevice and _cuda_getCurrentRawStream).
PyObject *current_device, *current_stream;

// Is q one of torch's own tensors, on the GPU that is current?  Then that GPU and its current stream.
bool plain_call(PyObject *q, int &device, void *&stream) {
    if (!THPVariable_CheckExact(q) || !THPVariable_Unpack(q).defined() || !THPVariable_Unpack(q).is_cuda() || !nothing_between())
        return false;
    PyObject *dev = PyObject_CallNoArgs(current_device);
    if (!dev) throw python_error();
    device = (int)PyLong_AsLong(dev);
    PyObject *handle = device == THPVariable_Unpack(q).get_device() ? PyObject_CallOneArg(current_stream, dev) : nullptr;
    Py_DECREF(dev);
    if (PyErr_Occurred()) {
        Py_XDECREF(handle);
        throw python_error();
    }
    if (!handle) return false;
    stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (PyErr_Occurred()) throw python_error();
    return true;
}

// The tensor behind o if it is one of torch's own, dense and plain, on GPU `device`; else null.
const at::Tensor *plain_tensor(PyObject *o, int device) {
    static const uint64_t plain_keys = c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA,
                                                            c10::DispatchKey::AutocastCUDA, c10::DispatchKey::ADInplaceOrView}).raw_repr();
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || (t.key_set().raw_repr() & ~plain_keys) != 0 || !t.has_storage() || t.get_device() != device)
        return nullptr;
    return &t;
}
bool plain_vector(PyObject *o, int device, int64_t n, const at::Tensor *&t) {  // n ints, contiguous
    t = plain_tensor(o, device);
    return t && t->scalar_type() == at::kInt && t->dim() == 1 && t->is_contiguous() && (n < 0 || t->numel() == n);
}
// An int as ctypes passes it (the low 32 bits), if o is one.
bool plain_int(PyObject *o, int &x) {
    if (!PyLong_CheckExact(o)) return false;
    x = (int)PyLong_AsUnsignedLongMask(o);
    return true;
}
bool plain_scale(PyObject *o, int64_t D, float &scale) {
    if (o == Py_None) {
        if (D <= 0) return false;
        scale = (float)(1.0 / std::sqrt((double)D));
        return true;
    }
    if (!PyFloat_CheckExact(o)) return false;
    scale = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool contiguous_bf16_4d(const at::Tensor *t) {
    return t && t->scalar_type() == at::kBFloat16 && t->dim() == 4 && t->is_contiguous();
}

// (out, lse), or the entry point's status for the binding to raise.
PyObject *results(long long rc, const at::Tensor &out, const at::Tensor &lse) {
    if (rc != SWAA_OK) return PyLong_FromLongLong(rc);
    PyObject *pair = PyTuple_New(2);
    if (!pair) return nullptr;
    PyTuple_SET_ITEM(pair, 0, THPVariable_Wrap(out));
    PyTuple_SET_ITEM(pair, 1, THPVariable_Wrap(lse));
    return pair;
}
at::Tensor result_like(const at::Tensor &t) { return at::empty_strided(t.sizes(), t.strides(), t.options()); }
at::Tensor empty_floats(const at::Tensor &on, at::IntArrayRef sizes) { return at::empty(sizes, on.options().dtype(at::kFloat)); }
at::Tensor empty_bytes(const at::Tensor &on, int64_t n) { return at::empty({n}, on.options().dtype(at::kByte)); }

// fwd(q, k, v, window, n_sink, n_prompt or None, scale or None)
PyObject *fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int window, n_sink, n_prompt = 0, device;
    float scale;
    void *stream;
    if (n != 7 || !plain_call(a[0], device, stream)) Py_RETURN_NONE;
    const at::Tensor *q = plain_tensor(a[0], device), *k = plain_tensor(a[1], device), *v = plain_tensor(a[2], device);
    if (!contiguous_bf16_4d(q) || !contiguous_bf16_4d(k) || !contiguous_bf16_4d(v)) Py_RETURN_NONE;
    const int64_t B = q->size(0), Hq = q->size(1), N = q->size(2), D = q->size(3), Hkv = k->size(1);
    if (k->sizes() != v->sizes() || k->size(0) != B || k->size(2) != N || k->size(3) != D) Py_RETURN_NONE;
    if (!plain_int(a[3], window) || !plain_int(a[4], n_sink) || !plain_scale(a[6], D, scale)) Py_RETURN_NONE;
    if (a[5] != Py_None && !plain_int(a[5], n_prompt)) Py_RETURN_NONE;
    const at::Tensor out = result_like(*q), lse = empty_floats(*q, {B, Hq, N});
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
    void *op = out.data_ptr();
    float *lp = static_cast<float *>(lse.data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (a[5] == Py_None)
        rc = fwd_entry(qp, kp, vp, op, lp, (int)B, (int)Hq, (int)Hkv, (int)N, (int)D, window, n_sink, scale, stream);
    else
        rc = fwd_fa_decode_entry(qp, kp, vp, op, lp, (int)B, (int)Hq, (int)Hkv, (int)N, (int)D, window, n_sink, n_prompt, scale, stream);
    Py_END_ALLOW_THREADS
    return results(rc, out, lse);
    END_HANDLE_TH_ERRORS
}

// decode(q, k, v, window, n_sink, scale or None, workspace or None)
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int window, n_sink, device;
    float scale;
    void *stream;
    if (n != 7 || !plain_call(a[0], device, stream)) Py_RETURN_NONE;
    const at::Tensor *q = plain_tensor(a[0], device), *k = plain_tensor(a[1], device), *v = plain_tensor(a[2], device);
    if (!contiguous_bf16_4d(q) || !contiguous_bf16_4d(k) || !contiguous_bf16_4d(v)) Py_RETURN_NONE;
    const int64_t B = q->size(0), Hq = q->size(1), Nq = q->size(2), D = q->size(3), Hkv = k->size(1), Nk = k->size(2);
    if (k->sizes() != v->sizes() || k->size(0) != B || k->size(3) != D || q->numel() == 0 || k->numel() == 0) Py_RETURN_NONE;
    if (!plain_int(a[3], window) || !plain_int(a[4], n_sink) || !plain_scale(a[5], D, scale)) Py_RETURN_NONE;
    at::Tensor workspace;
    if (a[6] == Py_None) {
        const long long need = decode_workspace_entry((int)B, (int)Hq, (int)Hkv, (int)Nq, (int)Nk, (int)D, window, n_sink);
        if (need < 0) return PyLong_FromLongLong(need);
        workspace = empty_bytes(*q, need);
    } else {
        const at::Tensor *given = plain_tensor(a[6], device);
        if (!given || given->scalar_type() != at::kByte || !given->is_contiguous()) Py_RETURN_NONE;
        workspace = *given;
    }
    const at::Tensor out = result_like(*q), lse = empty_floats(*q, {B, Hq, Nq});
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
    void *op = out.data_ptr(), *wp = workspace.data_ptr();
    float *lp = static_cast<float *>(lse.data_ptr());
    const long long bytes = workspace.numel();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = decode_entry(qp, kp, vp, op, lp, (int)B, (int)Hq, (int)Hkv, (int)Nq, (int)Nk, (int)D, window, n_sink, scale, wp, bytes, stream);
    Py_END_ALLOW_THREADS
    return results(rc, out, lse);
    END_HANDLE_TH_ERRORS
}

bool view_4d(const at::Tensor *t, at::ScalarType dtype) { return t && t->scalar_type() == dtype && t->dim() == 4 && t->stride(3) == 1; }

// decode_ex(q, k, v, window, n_sink, scale, seq_lens, block_table, max_seqlen_k, workspace); None for what is not given
PyObject *decode_ex(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int device;
    swaa_decode_args s{};
    if (n != 10 || !plain_call(a[0], device, s.stream)) Py_RETURN_NONE;
    const at::Tensor *q = plain_tensor(a[0], device), *k = plain_tensor(a[1], device), *v = plain_tensor(a[2], device);
    if (!q || (q->scalar_type() != at::kBFloat16 && q->scalar_type() != at::kHalf) || q->dim() != 4 || !q->is_contiguous()) Py_RETURN_NONE;
    if (!view_4d(k, q->scalar_type()) || !view_4d(v, q->scalar_type())) Py_RETURN_NONE;
    const int64_t B = q->size(0), Hq = q->size(1), Nq = q->size(2), D = q->size(3);
    if (!plain_int(a[3], s.window) || !plain_int(a[4], s.n_sink) || !plain_scale(a[5], D, s.scale)) Py_RETURN_NONE;
    s.B = (int)B, s.Hq = (int)Hq, s.Nq = (int)Nq, s.D = (int)D, s.Hkv = (int)k->size(1), s.Nk = (int)k->size(2);
    const at::Tensor *t;
    if (a[6] != Py_None) {
        if (!plain_vector(a[6], device, B, t)) Py_RETURN_NONE;
        s.seq_lens = static_cast<const int *>(t->data_ptr());
    }
    if (a[7] != Py_None) {
        t = plain_tensor(a[7], device);
        if (!t || t->scalar_type() != at::kInt || t->dim() != 2 || t->stride(1) != 1 || t->size(0) != B || a[8] == Py_None) Py_RETURN_NONE;
        s.block_table = static_cast<const int *>(t->data_ptr());
        s.block_table_stride = (int)t->stride(0), s.page_size = (int)k->size(2), s.num_pages = (int)k->size(0);
    }
    if (a[8] != Py_None && !plain_int(a[8], s.Nk)) Py_RETURN_NONE;
    s.dtype = q->scalar_type() == at::kHalf ? SWAA_F16 : SWAA_BF16;
    s.q = q->data_ptr();
    s.k = {k->data_ptr(), k->stride(0), k->stride(1), k->stride(2)};
    s.v = {v->data_ptr(), v->stride(0), v->stride(1), v->stride(2)};
    at::Tensor workspace;
    if (a[9] == Py_None) {
        const long long need = decode_ex_workspace_entry(&s);
        if (need < 0) return PyLong_FromLongLong(need);
        workspace = empty_bytes(*q, need);
    } else {
        const at::Tensor *given = plain_tensor(a[9], device);
        if (!given) Py_RETURN_NONE;
        workspace = *given;
    }
    s.workspace = workspace.data_ptr(), s.workspace_bytes = workspace.numel();
    const at::Tensor out = result_like(*q), lse = empty_floats(*q, {B, Hq, Nq});
    s.out = out.data_ptr(), s.lse = static_cast<float *>(lse.data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = decode_ex_entry(&s);
    Py_END_ALLOW_THREADS
    return results(rc, out, lse);
    END_HANDLE_TH_ERRORS
}

// fill_fwd_ex(args, q, k, v, window, n_sink, n_prompt, scale, cu_seqlens_q, cu_seqlens_k, max_seqlen_q, max_seqlen_k, block_table,
// total_rows_q, n_prompts): fills the argument block `args` (writable bytes) and returns the results it points at.
PyObject *fill_fwd_ex(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int device;
    swaa_fwd_args s{};
    if (n != 15 || !plain_call(a[1], device, s.stream)) Py_RETURN_NONE;
    const bool packed = a[8] != Py_None || a[9] != Py_None, paged = a[12] != Py_None;
    const at::Tensor *q = plain_tensor(a[1], device), *k = plain_tensor(a[2], device), *v = plain_tensor(a[3], device);
    if (!q || (q->scalar_type() != at::kBFloat16 && q->scalar_type() != at::kHalf)) Py_RETURN_NONE;
    const int64_t q_dims = packed ? 3 : 4, kv_dims = paged ? 4 : q_dims;
    if (q->dim() != q_dims || q->stride(-1) != 1) Py_RETURN_NONE;
    for (const at::Tensor *t : {k, v})
        if (!t || t->scalar_type() != q->scalar_type() || t->dim() != kv_dims || t->stride(-1) != 1) Py_RETURN_NONE;
    const int64_t D = q->size(-1);
    s.D = (int)D, s.Hq = (int)q->size(-3), s.Hkv = (int)k->size(-3);
    if (!plain_int(a[4], s.window) || !plain_int(a[5], s.n_sink) || !plain_scale(a[7], D, s.scale)) Py_RETURN_NONE;
    s.n_prompt = 0x7fffffff;
    if (a[6] != Py_None && !plain_int(a[6], s.n_prompt)) Py_RETURN_NONE;
    int64_t B;
    const at::Tensor *t;
    if (packed) {
        const at::Tensor *cu_q, *cu_k;
        if (!plain_vector(a[8], device, -1, cu_q) || !plain_vector(a[9], device, cu_q->numel(), cu_k)) Py_RETURN_NONE;
        B = cu_q->numel() - 1;
        s.cu_seqlens_q = static_cast<const int *>(cu_q->data_ptr()), s.cu_seqlens_k = static_cast<const int *>(cu_k->data_ptr());
        if (!plain_int(a[10], s.Nq) || !plain_int(a[11], s.Nk)) Py_RETURN_NONE;
    } else {
        B = q->size(0), s.Nq = (int)q->size(2), s.Nk = (int)k->size(2);
    }
    s.B = (int)B;
    if (paged) {
        t = plain_tensor(a[12], device);
        if (!t || t->scalar_type() != at::kInt || t->dim() != 2 || t->stride(1) != 1 || t->size(0) != B || !plain_int(a[11], s.Nk))
            Py_RETURN_NONE;
        s.block_table = static_cast<const int *>(t->data_ptr());
        s.block_table_stride = (int)t->stride(0), s.page_size = (int)k->size(2), s.num_pages = (int)k->size(0);
    }
    s.total_rows_q = packed ? q->size(1) : 0;
    if (a[13] != Py_None) {
        if (!PyLong_CheckExact(a[13])) Py_RETURN_NONE;
        s.total_rows_q = (long long)PyLong_AsUnsignedLongLongMask(a[13]);
    }
    if (a[14] != Py_None) {
        if (!plain_vector(a[14], device, B, t)) Py_RETURN_NONE;
        s.n_prompts = static_cast<const int *>(t->data_ptr());
    }
    s.dtype = q->scalar_type() == at::kHalf ? SWAA_F16 : SWAA_BF16;
    auto strided = [](const at::Tensor &t) {
        return t.dim() == 3 ? swaa_tensor{t.data_ptr(), 0, t.stride(0), t.stride(1)}
                            : swaa_tensor{t.data_ptr(), t.stride(0), t.stride(1), t.stride(2)};
    };
    const at::Tensor out = result_like(*q), lse = packed ? empty_floats(*q, {q->size(0), q->size(1)}) : empty_floats(*q, {B, q->size(1), q->size(2)});
    s.q = strided(*q), s.k = strided(*k), s.v = strided(*v), s.out = strided(out);
    s.lse = static_cast<float *>(lse.data_ptr());
    s.lse_stride_b = packed ? 0 : lse.stride(0), s.lse_stride_h = lse.stride(packed ? 0 : 1);
    Py_buffer block;
    if (PyObject_GetBuffer(a[0], &block, PyBUF_WRITABLE) != 0) return nullptr;
    const bool fits = block.len == (Py_ssize_t)sizeof(s);
    if (fits) std::memcpy(block.buf, &s, sizeof(s));
    PyBuffer_Release(&block);
    if (!fits) Py_RETURN_NONE;
    return results(SWAA_OK, out, lse);
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the six entry points above, in their order, then current_device and current_stream, the library's version, the
// sizes of the binding's two argument blocks, torch's version).  ImportError if this file was compiled for others: a call from here
// hands the library pointers and strides where the header it was compiled with has them.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *at[6];
    if (n != 12) {
        PyErr_SetString(PyExc_TypeError, "bind takes six addresses, two functions, three numbers and a text");
        return nullptr;
    }
    for (int i = 0; i < 6; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    const long long version = PyLong_AsLongLong(a[8]), fwd_bytes = PyLong_AsLongLong(a[9]), decode_bytes = PyLong_AsLongLong(a[10]);
    const char *torch_version = PyErr_Occurred() ? nullptr : PyUnicode_AsUTF8(a[11]);
    if (!torch_version) return nullptr;
    if (version != SWAA_VERSION || fwd_bytes != (long long)sizeof(swaa_fwd_args) || decode_bytes != (long long)sizeof(swaa_decode_args)) {
        PyErr_Format(PyExc_ImportError, "compiled for libswaa %d with argument blocks of %zu and %zu bytes, not %lld with %lld and %lld",
                     SWAA_VERSION, sizeof(swaa_fwd_args), sizeof(swaa_decode_args), version, fwd_bytes, decode_bytes);
        return nullptr;
    }
    if (std::strncmp(torch_version, TORCH_VERSION, std::strlen(TORCH_VERSION)) != 0) {
        PyErr_Format(PyExc_ImportError, "compiled for torch %s, not %s", TORCH_VERSION, torch_version);
        return nullptr;
    }
    fwd_entry = reinterpret_cast<decltype(fwd_entry)>(at[0]);
    fwd_fa_decode_entry = reinterpret_cast<decltype(fwd_fa_decode_entry)>(at[1]);
    decode_entry = reinterpret_cast<decltype(decode_entry)>(at[2]);
    decode_workspace_entry = reinterpret_cast<decltype(decode_workspace_entry)>(at[3]);
    decode_ex_entry = reinterpret_cast<decltype(decode_ex_entry)>(at[4]);
    decode_ex_workspace_entry = reinterpret_cast<decltype(decode_ex_workspace_entry)>(at[5]);
    Py_INCREF(a[6]);
    Py_INCREF(a[7]);
    Py_XSETREF(current_device, a[6]);
    Py_XSETREF(current_stream, a[7]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(&name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind), METHOD(fwd), METHOD(decode), METHOD(decode_ex), METHOD(fill_fwd_ex), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_calls() { return PyModule_Create(&module); }
