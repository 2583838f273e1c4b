// The accepted case of the Python entry points, in native code: unpacks the tensors, makes the binding's checks on them,
// allocates what the caller left out and calls the C ABI.  Small calls were bound by marshalling through ctypes: two fp32
// examples of 8 queries and 64 keys (kernel 4 us) 10.0 -> 4.3 us a pass, 27 -> 17 us alone; a training step through autograd
// whose kernels take less: 124 to 144 -> 82 to 96 us on the host, most of it torch's own.
//
// A function returns None for everything that is not plainly right - another type or dtype, a strided view, a tensor of a
// subclass or a transform, a wrong shape or device, an int that is no int, the error status of an argument - before anything
// is enqueued; the Python function then takes its own way, which raises what there is to raise.  So nothing is accepted here
// that is not accepted there.  A launch that the HIP runtime refuses raises KunlunError here: work may be enqueued by then,
// and the call is not made again.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>

#include "../../include/kunlun.h"

// (of the library, behind its public interface: the bytes that one call of kunlun_sumkron_fwd can use)
extern "C" size_t kunlun_sumkron_batch_bytes(int B, int S, int T, int D, int k, int dtype);

// Device type of the tensors; the module can be built for host tensors, to run its checks in front of another library.
#ifndef KUNLUN_CALL_DEVICE
#define KUNLUN_CALL_DEVICE CUDA
#endif

namespace {

PyObject* g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

constexpr int64_t ANY = -1;

// Arguments of one call.  Every accessor leaves ok = false where the argument is not of the plain kind.
struct Call {
    bool ok = true;
    static constexpr int NONE_YET = -2;  // (-1: the index of a host tensor)
    int device = NONE_YET;
    at::ScalarType type = at::ScalarType::Undefined;  // of the first tensor: bfloat16 or float32

    static bool is_plain(const at::Tensor& t) {
        if (!t.defined() || t.layout() != at::kStrided || t.device().type() != c10::DeviceType::KUNLUN_CALL_DEVICE || !t.has_storage()) return false;
        const c10::DispatchKeySet odd({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                       c10::DispatchKey::BatchedNestedTensor, c10::DispatchKey::Functionalize, c10::DispatchKey::ZeroTensor,
                                       c10::DispatchKey::Conjugate, c10::DispatchKey::Negative});
        return !t.key_set().has_any(odd) && t.is_contiguous();
    }
    bool same_device(const at::Tensor& t) {
        if (device == NONE_YET) device = t.device().index();
        return t.device().index() == device;
    }
    // A tensor of the call's dtype (the first one sets it), shape (a, b, c); ANY: any extent.
    const at::Tensor* rows(PyObject* o, int64_t a, int64_t b, int64_t c) {
        if (!ok || !THPVariable_CheckExact(o)) return fail();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!is_plain(t) || t.dim() != 3 || !same_device(t)) return fail();
        if (type == at::ScalarType::Undefined) {
            if (t.scalar_type() != at::kBFloat16 && t.scalar_type() != at::kFloat) return fail();
            type = t.scalar_type();
        }
        const auto s = t.sizes();
        if (s[1] > INT32_MAX || s[2] > INT32_MAX) return fail();
        if (t.scalar_type() != type || (a != ANY && s[0] != a) || (b != ANY && s[1] != b) || (c != ANY && s[2] != c)) return fail();
        return &t;
    }
    // int32 offsets [n + 1] (n = ANY: any number of examples)
    const at::Tensor* offsets(PyObject* o, int64_t n) {
        if (!ok || !THPVariable_CheckExact(o)) return fail();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!is_plain(t) || t.scalar_type() != at::kInt || t.dim() != 1 || t.numel() < 1 || t.numel() > INT32_MAX || (n != ANY && t.numel() != n + 1) || !same_device(t))
            return fail();
        return &t;
    }
    const at::Tensor* lse(PyObject* o, int64_t H, int64_t n) {
        if (!ok || !THPVariable_CheckExact(o)) return fail();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!is_plain(t) || t.scalar_type() != at::kFloat || t.dim() != 2 || t.size(0) != H || t.size(1) != n || !same_device(t)) return fail();
        return &t;
    }
    const at::Tensor* bytes(PyObject* o) {
        if (!ok || !THPVariable_CheckExact(o)) return fail();
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!is_plain(t) || t.scalar_type() != at::kByte || !same_device(t)) return fail();
        return &t;
    }
    int integer(PyObject* o) {
        if (!ok || !PyLong_CheckExact(o)) return fail_int();
        int overflow = 0;
        const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow || x < INT32_MIN || x > INT32_MAX) return fail_int();
        return (int)x;
    }
    float real(PyObject* o) {
        if (!ok || !(PyFloat_CheckExact(o) || PyLong_CheckExact(o))) return (float)fail_int();
        const double x = PyFloat_AsDouble(o);
        if (x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return (float)fail_int(); }
        return (float)x;
    }
    // raw handle of the stream argument: None = the current stream of the current device
    void* stream(PyObject* o) {
        if (!ok) return nullptr;
        PyObject* h;
        if (o == Py_None) {
            PyObject* dev = PyLong_FromLong(c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice().index());
            h = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
            Py_XDECREF(dev);
        } else {
            h = PyObject_GetAttrString(o, "cuda_stream");
        }
        void* s = h && PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
        if (!h || !PyLong_Check(h) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        Py_XDECREF(h);
        return s;
    }
    int dtype() const { return type == at::kFloat ? KUNLUN_FP32 : KUNLUN_BF16; }
    const at::Tensor* fail() { ok = false; return nullptr; }
    int fail_int() { ok = false; return 0; }
};

// The given tensor, or a new one.
struct Out {
    at::Tensor fresh;
    const at::Tensor* t = nullptr;
    void* ptr() const { return t ? t->data_ptr() : nullptr; }
    void make(const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType type) {
        fresh = at::empty(sizes, like.options().dtype(type));
        t = &fresh;
    }
    PyObject* object(PyObject* given) const {
        if (given != Py_None) { Py_INCREF(given); return given; }
        if (!t) Py_RETURN_NONE;
        return THPVariable_Wrap(*t);
    }
};

// The items of a caller's list are held: another thread may replace them while the kernels are enqueued.
struct Grads {
    Out g[3];
    THPObjectPtr given[3];
    // out: None or a sequence of three tensors shaped like the inputs
    void take(Call& c, PyObject* out, const at::Tensor* const (&like)[3]) {
        if (!c.ok) return;
        if (out != Py_None) {
            if (!(PyTuple_CheckExact(out) || PyList_CheckExact(out)) || PySequence_Fast_GET_SIZE(out) != 3) { c.ok = false; return; }
            for (int i = 0; i < 3; ++i) {
                given[i] = Py_NewRef(PySequence_Fast_GET_ITEM(out, i));
                g[i].t = c.rows(given[i], like[i]->size(0), like[i]->size(1), like[i]->size(2));
            }
        }
    }
    void allocate(const at::Tensor* const (&like)[3]) {
        for (int i = 0; i < 3; ++i)
            if (!g[i].t) g[i].make(*like[i], like[i]->sizes(), like[i]->scalar_type());
    }
    PyObject* result() const {
        PyObject* r = PyTuple_New(3);
        if (!r) return nullptr;
        for (int i = 0; i < 3; ++i) {
            PyObject* o = given[i] ? Py_NewRef(given[i].get()) : g[i].object(Py_None);
            if (!o) { Py_DECREF(r); return nullptr; }
            PyTuple_SET_ITEM(r, i, o);
        }
        return r;
    }
};

PyObject* pair(const Out& a, PyObject* given_a, const Out& b, PyObject* given_b) {
    PyObject* x = a.object(given_a);
    PyObject* y = x ? b.object(given_b) : nullptr;
    PyObject* r = y ? PyTuple_New(2) : nullptr;
    if (!r) { Py_XDECREF(x); Py_XDECREF(y); return nullptr; }
    PyTuple_SET_ITEM(r, 0, x);
    PyTuple_SET_ITEM(r, 1, y);
    return r;
}

void take_workspace(Call& c, PyObject* o, Out& ws) {
    if (o != Py_None) ws.t = c.bytes(o);
}
// (given back when the call returns: the allocator is told of the caller's stream, on which its kernels may still be to run)
void make_workspace(Out& ws, const at::Tensor& like, size_t nbytes, PyObject* stream) {
    if (ws.t) return;
    ws.make(like, {(int64_t)(nbytes > 256 ? nbytes : 256)}, at::kByte);
    if (stream != Py_None && THPStream_Check(stream)) {
        const THPStream* s = (THPStream*)stream;
        ws.fresh.record_stream(c10::Stream::unpack3(s->stream_id, (c10::DeviceIndex)s->device_index, (c10::DeviceType)s->device_type));
    }
}

template <typename T> const T* data(const at::Tensor* t) { return t ? (const T*)t->data_ptr() : nullptr; }

// A call of the C ABI.  The arguments are complete before the interpreter's lock is given up: a tensor whose memory may not be
// had throws where it can be reported, and no other thread changes a tensor between the checks and the reading of its pointer.
template <typename... P, typename... A>
int enqueue(int (*entry)(P...), A... arguments) {
    struct Unlocked {
        PyThreadState* const state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    } unlocked;
    return entry(arguments...);
}

PyObject* raise_status(int rc) {
    THPObjectPtr binding(PyImport_ImportModule("paper_2602_10016_amd.binding"));
    THPObjectPtr type(binding ? PyObject_GetAttrString(binding, "KunlunError") : nullptr);
    THPObjectPtr error(type ? PyObject_CallFunction(type, "i", rc) : nullptr);
    if (error) PyErr_SetObject(type, error);
    return nullptr;
}

#define ENTRY(NAME, N)                                                              \
    PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n) {                   \
        HANDLE_TH_ERRORS                                                            \
        if (n != N) { PyErr_SetString(PyExc_TypeError, #NAME ": " #N " arguments"); return nullptr; } \
        Call c;
#define END_ENTRY       \
        END_HANDLE_TH_ERRORS \
    }
#define PLAIN_OR_NONE \
    if (!c.ok) Py_RETURN_NONE
#define DONE_OR_NONE(RC) \
    if ((RC) == KUNLUN_ERR_LAUNCH) return raise_status(RC); \
    if ((RC) != KUNLUN_OK) Py_RETURN_NONE

// q, k, v, kv_offsets, scale, act, q_offsets, max_q, max_kv, out, lse, want_lse, workspace, stream
ENTRY(gdpa_fwd, 14)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t total_q = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], ANY, H, d);
    PLAIN_OR_NONE;
    const int64_t total_kv = k->size(0);
    const at::Tensor* v = c.rows(a[2], total_kv, H, d);
    const at::Tensor* kvo = c.offsets(a[3], ANY);
    PLAIN_OR_NONE;
    const int64_t B = kvo->numel() - 1;
    const float scale = c.real(a[4]);
    const int act = c.integer(a[5]);
    const at::Tensor* qo = a[6] == Py_None ? nullptr : c.offsets(a[6], B);
    const int max_q = c.integer(a[7]), max_kv = c.integer(a[8]);
    Out o, lse, ws;
    if (a[9] != Py_None) o.t = c.rows(a[9], total_q, H, d);
    if (a[10] != Py_None) lse.t = c.lse(a[10], H, total_q);
    const int want_lse = PyObject_IsTrue(a[11]);
    if (want_lse < 0) return nullptr;
    take_workspace(c, a[12], ws);
    void* s = c.stream(a[13]);
    PLAIN_OR_NONE;
    if (!o.t) o.make(*q, q->sizes(), q->scalar_type());
    if (!lse.t && want_lse) lse.make(*q, {H, total_q}, at::kFloat);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_GDPA_FWD, (int)B, (int)H, (int)d, max_q, max_kv, total_q, total_kv), a[13]);
    const int rc = enqueue(kunlun_gdpa_fwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), o.ptr(), (float*)lse.ptr(),
                           data<int32_t>(qo), data<int32_t>(kvo), (int)B, (int)H, (int)d, max_q, max_kv, total_q, total_kv,
                           scale, act, nullptr, c.dtype(), ws.ptr(), (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return pair(o, a[9], lse, a[10]);
END_ENTRY

// q, k, v, d_o, kv_offsets, scale, act, o, lse, q_offsets, max_q, max_kv, out, workspace, stream
ENTRY(gdpa_bwd, 15)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t total_q = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], ANY, H, d);
    PLAIN_OR_NONE;
    const int64_t total_kv = k->size(0);
    const at::Tensor* v = c.rows(a[2], total_kv, H, d);
    const at::Tensor* d_o = c.rows(a[3], total_q, H, d);
    const at::Tensor* kvo = c.offsets(a[4], ANY);
    PLAIN_OR_NONE;
    const int64_t B = kvo->numel() - 1;
    const float scale = c.real(a[5]);
    const int act = c.integer(a[6]);
    const at::Tensor* o = a[7] == Py_None ? nullptr : c.rows(a[7], total_q, H, d);
    const at::Tensor* lse = a[8] == Py_None ? nullptr : c.lse(a[8], H, total_q);
    const at::Tensor* qo = a[9] == Py_None ? nullptr : c.offsets(a[9], B);
    const int max_q = c.integer(a[10]), max_kv = c.integer(a[11]);
    Grads grads;
    const at::Tensor* const like[3] = {q, k, v};
    grads.take(c, a[12], like);
    Out ws;
    take_workspace(c, a[13], ws);
    void* s = c.stream(a[14]);
    PLAIN_OR_NONE;
    grads.allocate(like);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_GDPA_BWD, (int)B, (int)H, (int)d, max_q, max_kv, total_q, total_kv), a[14]);
    const int rc = enqueue(kunlun_gdpa_bwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), data<void>(o), data<float>(lse),
                           d_o->data_ptr(), grads.g[0].ptr(), grads.g[1].ptr(), grads.g[2].ptr(), data<int32_t>(qo),
                           data<int32_t>(kvo), (int)B, (int)H, (int)d, max_q, max_kv, total_q, total_kv, scale, act, nullptr,
                           c.dtype(), ws.ptr(), (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return grads.result();
END_ENTRY

// e_seed, k, v, kv_offsets, scale, act, max_kv, out, lse, want_lse, workspace, stream
ENTRY(seed_attn_fwd, 12)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t seeds = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], ANY, H, d);
    PLAIN_OR_NONE;
    const int64_t total_kv = k->size(0);
    const at::Tensor* v = c.rows(a[2], total_kv, H, d);
    const at::Tensor* kvo = c.offsets(a[3], ANY);
    PLAIN_OR_NONE;
    const int64_t B = kvo->numel() - 1, total_q = B * seeds;
    const float scale = c.real(a[4]);
    const int act = c.integer(a[5]), max_kv = c.integer(a[6]);
    if (seeds > INT32_MAX) c.ok = false;
    Out o, lse, ws;
    if (a[7] != Py_None) o.t = c.rows(a[7], total_q, H, d);
    if (a[8] != Py_None) lse.t = c.lse(a[8], H, total_q);
    const int want_lse = PyObject_IsTrue(a[9]);
    if (want_lse < 0) return nullptr;
    take_workspace(c, a[10], ws);
    void* s = c.stream(a[11]);
    PLAIN_OR_NONE;
    if (!o.t) o.make(*q, {total_q, H, d}, q->scalar_type());
    if (!lse.t && want_lse) lse.make(*q, {H, total_q}, at::kFloat);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_SEED_FWD, (int)B, (int)H, (int)d, (int)seeds, max_kv, total_q, total_kv), a[11]);
    const int rc = enqueue(kunlun_seed_attn_fwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), o.ptr(), (float*)lse.ptr(),
                           data<int32_t>(kvo), (int)B, (int)H, (int)d, (int)seeds, max_kv, total_kv, scale, act, nullptr,
                           c.dtype(), ws.ptr(), (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return pair(o, a[7], lse, a[8]);
END_ENTRY

// e_seed, k, v, d_o, kv_offsets, scale, act, o, lse, max_kv, out, workspace, stream
ENTRY(seed_attn_bwd, 13)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t seeds = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], ANY, H, d);
    PLAIN_OR_NONE;
    const int64_t total_kv = k->size(0);
    const at::Tensor* v = c.rows(a[2], total_kv, H, d);
    const at::Tensor* kvo = c.offsets(a[4], ANY);
    PLAIN_OR_NONE;
    const int64_t B = kvo->numel() - 1, total_q = B * seeds;
    const at::Tensor* d_o = c.rows(a[3], total_q, H, d);
    const float scale = c.real(a[5]);
    const int act = c.integer(a[6]);
    const at::Tensor* o = a[7] == Py_None ? nullptr : c.rows(a[7], total_q, H, d);
    const at::Tensor* lse = a[8] == Py_None ? nullptr : c.lse(a[8], H, total_q);
    const int max_kv = c.integer(a[9]);
    if (seeds > INT32_MAX) c.ok = false;
    Grads grads;
    const at::Tensor* const like[3] = {q, k, v};
    grads.take(c, a[10], like);
    Out ws;
    take_workspace(c, a[11], ws);
    void* s = c.stream(a[12]);
    PLAIN_OR_NONE;
    grads.allocate(like);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_SEED_BWD, (int)B, (int)H, (int)d, (int)seeds, max_kv, total_q, total_kv), a[12]);
    const int rc = enqueue(kunlun_seed_attn_bwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), data<void>(o), data<float>(lse),
                           d_o->data_ptr(), grads.g[0].ptr(), grads.g[1].ptr(), grads.g[2].ptr(), data<int32_t>(kvo), (int)B,
                           (int)H, (int)d, (int)seeds, max_kv, total_kv, scale, act, nullptr, c.dtype(), ws.ptr(),
                           (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return grads.result();
END_ENTRY

// q, k, v, offsets, window_left, window_right, scale, max_len, out, lse, want_lse, workspace, stream
ENTRY(swa_fwd, 13)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t total = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], total, H, d);
    const at::Tensor* v = c.rows(a[2], total, H, d);
    const at::Tensor* off = c.offsets(a[3], ANY);
    PLAIN_OR_NONE;
    const int64_t B = off->numel() - 1;
    const int left = c.integer(a[4]), right = c.integer(a[5]);
    const float scale = c.real(a[6]);
    const int max_len = c.integer(a[7]);
    Out o, lse, ws;
    if (a[8] != Py_None) o.t = c.rows(a[8], total, H, d);
    if (a[9] != Py_None) lse.t = c.lse(a[9], H, total);
    const int want_lse = PyObject_IsTrue(a[10]);
    if (want_lse < 0) return nullptr;
    take_workspace(c, a[11], ws);
    void* s = c.stream(a[12]);
    PLAIN_OR_NONE;
    if (!o.t) o.make(*q, q->sizes(), q->scalar_type());
    if (!lse.t && want_lse) lse.make(*q, {H, total}, at::kFloat);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_SWA_FWD, (int)B, (int)H, (int)d, max_len, max_len, total, total), a[12]);
    const int rc = enqueue(kunlun_swa_fwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), o.ptr(), (float*)lse.ptr(),
                           data<int32_t>(off), (int)B, (int)H, (int)d, max_len, total, left, right, scale, c.dtype(), ws.ptr(),
                           (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return pair(o, a[8], lse, a[9]);
END_ENTRY

// q, k, v, o, lse, d_o, offsets, window_left, window_right, scale, max_len, out, workspace, stream
ENTRY(swa_bwd, 14)
    const at::Tensor* q = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t total = q->size(0), H = q->size(1), d = q->size(2);
    const at::Tensor* k = c.rows(a[1], total, H, d);
    const at::Tensor* v = c.rows(a[2], total, H, d);
    const at::Tensor* o = c.rows(a[3], total, H, d);
    const at::Tensor* lse = c.lse(a[4], H, total);
    const at::Tensor* d_o = c.rows(a[5], total, H, d);
    const at::Tensor* off = c.offsets(a[6], ANY);
    PLAIN_OR_NONE;
    const int64_t B = off->numel() - 1;
    const int left = c.integer(a[7]), right = c.integer(a[8]);
    const float scale = c.real(a[9]);
    const int max_len = c.integer(a[10]);
    Grads grads;
    const at::Tensor* const like[3] = {q, k, v};
    grads.take(c, a[11], like);
    Out ws;
    take_workspace(c, a[12], ws);
    void* s = c.stream(a[13]);
    PLAIN_OR_NONE;
    grads.allocate(like);
    make_workspace(ws, *q, ws.t ? 0 : kunlun_workspace_bytes(KUNLUN_OP_SWA_BWD, (int)B, (int)H, (int)d, max_len, max_len, total, total), a[13]);
    const int rc = enqueue(kunlun_swa_bwd, q->data_ptr(), k->data_ptr(), v->data_ptr(), o->data_ptr(), data<float>(lse),
                           d_o->data_ptr(), grads.g[0].ptr(), grads.g[1].ptr(), grads.g[2].ptr(), data<int32_t>(off), (int)B,
                           (int)H, (int)d, max_len, total, left, right, scale, c.dtype(), ws.ptr(), (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return grads.result();
END_ENTRY

// x, z, w, out, workspace, stream
ENTRY(sumkron_fwd, 6)
    const at::Tensor* x = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t B = x->size(0), S = x->size(1), D = x->size(2);
    const at::Tensor* z = c.rows(a[1], ANY, S, ANY);
    PLAIN_OR_NONE;
    const int64_t k = z->size(0), T = z->size(2);
    const at::Tensor* w = c.rows(a[2], k, D, D);
    Out y, ws;
    if (a[3] != Py_None) y.t = c.rows(a[3], B, T, D);
    take_workspace(c, a[4], ws);
    void* s = c.stream(a[5]);
    for (int64_t n : {B, S, D, k, T})
        if (n > INT32_MAX) c.ok = false;
    PLAIN_OR_NONE;
    if (!y.t) y.make(*x, {B, T, D}, x->scalar_type());
    make_workspace(ws, *x, ws.t ? 0 : kunlun_sumkron_batch_bytes((int)B, (int)S, (int)T, (int)D, (int)k, c.dtype()), a[5]);
    const int rc = enqueue(kunlun_sumkron_fwd, x->data_ptr(), z->data_ptr(), w->data_ptr(), y.ptr(), (int)B, (int)S, (int)T,
                           (int)D, (int)k, c.dtype(), ws.ptr(), (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return y.object(a[3]);
END_ENTRY

// x, z, w, dy, workspace, stream
ENTRY(sumkron_bwd, 6)
    const at::Tensor* x = c.rows(a[0], ANY, ANY, ANY);
    PLAIN_OR_NONE;
    const int64_t B = x->size(0), S = x->size(1), D = x->size(2);
    const at::Tensor* z = c.rows(a[1], ANY, S, ANY);
    PLAIN_OR_NONE;
    const int64_t k = z->size(0), T = z->size(2);
    const at::Tensor* w = c.rows(a[2], k, D, D);
    const at::Tensor* dy = c.rows(a[3], B, T, D);
    Out ws;
    take_workspace(c, a[4], ws);
    void* s = c.stream(a[5]);
    for (int64_t n : {B, S, D, k, T})
        if (n > INT32_MAX) c.ok = false;
    PLAIN_OR_NONE;
    Grads grads;
    const at::Tensor* const like[3] = {x, z, w};
    grads.allocate(like);
    make_workspace(ws, *x, ws.t ? 0 : kunlun_sumkron_bwd_workspace_bytes((int)B, (int)S, (int)T, (int)D, (int)k, c.dtype()), a[5]);
    const int rc = enqueue(kunlun_sumkron_bwd, x->data_ptr(), z->data_ptr(), w->data_ptr(), dy->data_ptr(), grads.g[0].ptr(),
                           grads.g[1].ptr(), grads.g[2].ptr(), (int)B, (int)S, (int)T, (int)D, (int)k, c.dtype(), ws.ptr(),
                           (size_t)ws.t->numel(), s);
    DONE_OR_NONE(rc);
    return grads.result();
END_ENTRY

#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(gdpa_fwd), METHOD(gdpa_bwd), METHOD(seed_attn_fwd), METHOD(seed_attn_bwd), METHOD(swa_fwd), METHOD(swa_bwd),
                         METHOD(sumkron_fwd), METHOD(sumkron_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_call() {
    PyObject* c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    Py_DECREF(c);
    if (!g_raw_stream) return nullptr;
    return PyModule_Create(&module);
}
