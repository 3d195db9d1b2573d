// The tensor calls of binding.py without their Python: reads the tensors through torch's C++ interface, fills the C ABI's argument
// struct and calls the library on torch's current stream.  What bounds the smallest calls is the host: one fp32 prefill of 128
// tokens has 5.3 us of GPU work and took 6.1 us to issue from Python, a decode of one context 7.5 and 8.8.  Calls one after the
// other, through Python and through here: that prefill 6.4 -> 5.3 us, that decode 9.1 -> 8.2, short cache writes, norms and decodes
// 5.1-6.0 -> 4.1-4.3.
//
// Only the plain case is taken: exact torch tensors on one GPU, built-in ints and floats, values that fit their fields, every check
// of the Python path passed, no torch function mode.  Anything else returns None with nothing enqueued, and the caller goes
// the general way, which also raises the errors.
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cfloat>
#include <cmath>
#include <cstring>
#include <exception>
#include <initializer_list>

#include "../../include/attn.h"
#include "../../include/rmsnorm.h"

namespace {

typedef int (*call_t)(const void *, void *);
call_t g_attn[3] = {nullptr, nullptr, nullptr};  // attn_prefill_varlen, attn_decode_paged, attn_decode_paged_static
call_t g_kv_write = nullptr, g_rmsnorm = nullptr;

// nullptr unless `o` is a plain tensor
const at::Tensor *plain(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool dtype_code(at::ScalarType t, int32_t *code)
{
    if (t == at::kBFloat16) *code = ATTN_BF16;
    else if (t == at::kHalf) *code = ATTN_F16;
    else if (t == at::kFloat) *code = ATTN_F32;
    else return false;
    return true;
}
bool fits(int64_t x, int32_t *out)
{
    *out = (int32_t)x;
    return x == (int64_t)*out;
}
bool as_int32(PyObject *o, int32_t *out)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0 && fits(x, out);
}
bool as_float(PyObject *o, float *out)
{
    double x;
    if (PyFloat_CheckExact(o)) x = PyFloat_AS_DOUBLE(o);
    else if (PyLong_CheckExact(o)) {
        x = PyLong_AsDouble(o);
        if (x == -1.0 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
    } else return false;
    if (std::isfinite(x) && std::fabs(x) > FLT_MAX) return false;
    *out = (float)x;
    return true;
}
// Whether all tensors (null pointers aside) are where the first one is, and that is on a GPU if a kernel is to be launched with them.
bool together(std::initializer_list<const at::Tensor *> tensors, bool launch)
{
    const at::Tensor *first = *tensors.begin();
    if (launch && !first->is_cuda()) return false;
    for (const at::Tensor *t : tensors)
        if (t && t->device() != first->device()) return false;
    return true;
}
// None or a contiguous int32 tensor; *t stays null for None
bool int32_tensor(PyObject *o, const at::Tensor **t)
{
    *t = nullptr;
    if (o == Py_None) return true;
    *t = plain(o);
    return *t && (*t)->scalar_type() == at::kInt && (*t)->is_contiguous();
}

// The 13 values of binding._attn_fields: q, k, v, out, seq_lens, scale, max_q_len, max_kv_len, query_start_loc, kv_start_loc,
// block_table, causal, workspace.
bool fill_attn(PyObject *const *o, attn_args *a, bool launch)
{
    const at::Tensor *q = plain(o[0]), *k = plain(o[1]), *v = plain(o[2]), *out = plain(o[3]), *lens, *qsl, *kvsl, *table;
    if (!q || !k || !v || !out || !int32_tensor(o[4], &lens) || !lens || !int32_tensor(o[8], &qsl) || !int32_tensor(o[9], &kvsl) ||
        !int32_tensor(o[10], &table) || !PyBool_Check(o[11]))
        return false;
    const at::Tensor *ws = o[12] == Py_None ? nullptr : plain(o[12]);
    if (!ws && o[12] != Py_None) return false;
    if (!together({q, k, v, out, lens, qsl, kvsl, table, ws}, launch)) return false;
    if (q->dim() != 3 || out->dim() != 3 || k->dim() != (table ? 4 : 3) || lens->dim() < 1 || (table && table->dim() < 1)) return false;
    memset(a, 0, sizeof *a);
    a->struct_bytes = sizeof *a;
    if (!dtype_code(q->scalar_type(), &a->dtype) || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() ||
        out->scalar_type() != q->scalar_type() || k->sizes() != v->sizes() || k->strides() != v->strides())
        return false;
    const auto qs = q->strides(), ks = k->strides(), os = out->strides();
    if (qs[2] != 1 || os[2] != 1 || ks.back() != 1) return false;
    if (!fits(lens->size(0), &a->num_seqs) || !fits(q->size(1), &a->num_q_heads) || !fits(q->size(2), &a->head_dim) ||
        !fits(q->size(0), &a->total_q) || !as_float(o[5], &a->scale) || !as_int32(o[6], &a->max_q_len) || !as_int32(o[7], &a->max_kv_len))
        return false;
    a->q = q->data_ptr();
    a->q_stride_tok = qs[0];
    a->q_stride_head = qs[1];
    a->out = out->data_ptr();
    a->o_stride_tok = os[0];
    a->o_stride_head = os[1];
    a->k = k->data_ptr();
    a->v = v->data_ptr();
    const int paged = table ? 1 : 0;
    if (!fits(k->size(1 + paged), &a->num_kv_heads)) return false;
    a->kv_stride_tok = ks[paged];
    a->kv_stride_head = ks[1 + paged];
    if (paged) {
        a->kv_stride_block = ks[0];
        if (!fits(k->size(0), &a->num_blocks) || !fits(k->size(1), &a->block_size) || !fits(table->stride(0), &a->block_table_stride)) return false;
        a->block_table = (const int32_t *)table->data_ptr();
    }
    a->query_start_loc = qsl ? (const int32_t *)qsl->data_ptr() : nullptr;
    a->kv_start_loc = kvsl ? (const int32_t *)kvsl->data_ptr() : nullptr;
    a->seq_lens = (const int32_t *)lens->data_ptr();
    a->causal = o[11] == Py_True ? 1 : 0;
    if (ws) {
        a->workspace = ws->data_ptr();
        a->workspace_bytes = (uint64_t)ws->numel() * ws->element_size();
    }
    return true;
}

// k_new, v_new, k_cache, v_cache, slot_mapping
bool fill_kv_write(PyObject *const *o, attn_kv_write_args *a, bool launch)
{
    const at::Tensor *kn = plain(o[0]), *vn = plain(o[1]), *kc = plain(o[2]), *vc = plain(o[3]), *slots;
    if (!kn || !vn || !kc || !vc || !int32_tensor(o[4], &slots) || !slots) return false;
    if (!together({kn, vn, kc, vc, slots}, launch)) return false;
    if (kn->dim() != 3 || vn->dim() != 3 || kc->dim() != 4 || vc->dim() != 4) return false;
    if (kn->strides() != vn->strides() || kc->strides() != vc->strides() || kn->stride(2) != 1 || kc->stride(3) != 1) return false;
    memset(a, 0, sizeof *a);
    a->struct_bytes = sizeof *a;
    if (!dtype_code(kn->scalar_type(), &a->dtype) || !fits(kn->size(0), &a->num_tokens) || !fits(kn->size(1), &a->num_kv_heads) ||
        !fits(kn->size(2), &a->head_dim) || !fits(kc->size(1), &a->block_size) || !fits(kc->size(0), &a->num_blocks))
        return false;
    a->k_new = kn->data_ptr();
    a->v_new = vn->data_ptr();
    a->new_stride_tok = kn->stride(0);
    a->new_stride_head = kn->stride(1);
    a->k_cache = kc->data_ptr();
    a->v_cache = vc->data_ptr();
    a->kv_stride_block = kc->stride(0);
    a->kv_stride_tok = kc->stride(1);
    a->kv_stride_head = kc->stride(2);
    a->slot_mapping = (const int32_t *)slots->data_ptr();
    return true;
}

// x, weight, out, eps, residual
bool fill_rmsnorm(PyObject *const *o, rmsnorm_args *a, bool launch)
{
    const at::Tensor *x = plain(o[0]), *w = plain(o[1]), *out = plain(o[2]), *res = o[4] == Py_None ? nullptr : plain(o[4]);
    if (!x || !w || !out || (!res && o[4] != Py_None)) return false;
    if (!together({x, w, out, res}, launch)) return false;
    if (x->dim() != 2 || out->dim() != 2 || w->dim() != 1 || (res && res->dim() != 2)) return false;
    if (x->stride(1) != 1 || out->stride(1) != 1 || w->stride(0) != 1 || (res && res->stride(1) != 1)) return false;
    memset(a, 0, sizeof *a);
    a->struct_bytes = sizeof *a;
    if (!dtype_code(x->scalar_type(), &a->dtype) || !fits(x->size(0), &a->num_tokens) || !fits(x->size(1), &a->hidden) || !as_float(o[3], &a->eps))
        return false;
    a->x = x->data_ptr();
    a->x_stride = x->stride(0);
    if (res) {
        a->residual = res->data_ptr();
        a->residual_stride = res->stride(0);
    }
    a->weight = w->data_ptr();
    a->out = out->data_ptr();
    a->out_stride = out->stride(0);
    return true;
}

// Fills the struct and calls `f` on the current stream; None where the general path has to decide.  With f null the struct is returned
// as bytes (for the test that compares the two paths).
template <typename Args, typename Fill>
PyObject *call(call_t f, PyObject *const *o, Fill fill)
{
    Args a;
    void *stream = nullptr;
    try {
        if (at::impl::torch_function_mode_enabled() || !fill(o, &a, f != nullptr)) Py_RETURN_NONE;
        if (!f) return PyBytes_FromStringAndSize((const char *)&a, sizeof a);
        stream = (void *)c10::hip::getCurrentHIPStream().stream();
    } catch (...) {  // (a tensor without storage, symbolic sizes, no device: the general path reports it)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(&a, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

bool arguments(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return false;
}
// kind (0 prefill, 1 decode, 2 decode with the static records, -1: only pack), then the 13 values of fill_attn
PyObject *py_attn(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    if (!arguments(n, 14)) return nullptr;
    const long kind = PyLong_AsLong(o[0]);
    if (kind < -1 || kind > 2) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "kind");
        return nullptr;
    }
    return call<attn_args>(kind < 0 ? nullptr : g_attn[kind], o + 1, fill_attn);
}
PyObject *py_kv_write(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return arguments(n, 5) ? call<attn_kv_write_args>(g_kv_write, o, fill_kv_write) : nullptr;
}
PyObject *py_rmsnorm(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return arguments(n, 5) ? call<rmsnorm_args>(g_rmsnorm, o, fill_rmsnorm) : nullptr;
}
PyObject *py_pack_kv_write(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return arguments(n, 5) ? call<attn_kv_write_args>(nullptr, o, fill_kv_write) : nullptr;
}
PyObject *py_pack_rmsnorm(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return arguments(n, 5) ? call<rmsnorm_args>(nullptr, o, fill_rmsnorm) : nullptr;
}
// Scratch memory for a prefill call: bytes and stream handle -> address, or 0 where the call has to do without.  The block belongs
// to the stream's pool of torch's caching allocator, so once released it only goes to later work of the same stream.  Taken from the
// allocator itself and not as a tensor, which modes (fake tensors, deterministic filling) would see.
PyObject *py_scratch(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    if (!arguments(n, 2)) return nullptr;
    const size_t bytes = PyLong_AsSize_t(o[0]);
    const hipStream_t stream = PyErr_Occurred() ? nullptr : (hipStream_t)PyLong_AsVoidPtr(o[1]);
    if (PyErr_Occurred()) return nullptr;
    // A failed request makes the allocator give its whole cache back and wait for the GPU: after one the thread's next calls do not ask.
    static thread_local int do_without = 0;
    if (do_without > 0) {
        --do_without;
        return PyLong_FromLong(0);
    }
    void *p = nullptr;
    Py_BEGIN_ALLOW_THREADS
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (stream == hipStreamPerThread) {  // (one handle for the streams of all threads)
    } else if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
        (void)hipGetLastError();
    } else if (status == hipStreamCaptureStatusNone) {  // (else: nobody would hold the memory for the replays)
        // another stream may be capturing, which an allocation must not end
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        try {
            p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream);
        } catch (...) {
            p = nullptr;
        }
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (!p) do_without = 1000;
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromVoidPtr(p);
}
// Whether any of the arguments is a tensor in host memory.
PyObject *py_any_on_host(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    for (Py_ssize_t i = 0; i < n; ++i)
        if (THPVariable_Check(o[i]) && THPVariable_Unpack(o[i]).device().is_cpu()) Py_RETURN_TRUE;
    Py_RETURN_FALSE;
}
PyObject *py_release(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    if (!arguments(n, 1)) return nullptr;
    void *p = PyLong_AsVoidPtr(o[0]);
    if (PyErr_Occurred()) return nullptr;
    try {
        c10::hip::HIPCachingAllocator::raw_delete(p);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    Py_RETURN_NONE;
}
// addresses of attn_prefill_varlen, attn_decode_paged, attn_decode_paged_static, attn_kv_cache_write, rmsnorm_fused_add
PyObject *py_bind(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    if (!arguments(n, 5)) return nullptr;
    void *p[5];
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(o[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int i = 0; i < 3; ++i) g_attn[i] = (call_t)p[i];
    g_kv_write = (call_t)p[3];
    g_rmsnorm = (call_t)p[4];
    Py_RETURN_NONE;
}

#define FASTCALL(f) (PyCFunction)(void (*)(void)) f, METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", FASTCALL(py_bind), nullptr},
    {"attn", FASTCALL(py_attn), nullptr},
    {"kv_write", FASTCALL(py_kv_write), nullptr},
    {"rmsnorm", FASTCALL(py_rmsnorm), nullptr},
    {"scratch", FASTCALL(py_scratch), nullptr},
    {"release", FASTCALL(py_release), nullptr},
    {"any_on_host", FASTCALL(py_any_on_host), nullptr},
    {"pack_kv_write", FASTCALL(py_pack_kv_write), nullptr},
    {"pack_rmsnorm", FASTCALL(py_pack_rmsnorm), nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
