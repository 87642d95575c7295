// Native argument marshalling of the Python binding: torch tensors in, one C-ABI call (include/dd.h), torch tensors out.
//
// No step of the computation is here.  Per call: shapes, types and placement are checked, missing outputs are
// allocated, the scratch tensor of (device, stream) is looked up and the library is called on torch's current stream.
// It is native because the small calls of a cycle are shorter than their marshalling was: through ctypes a drafter call cost
// the host 13.7 us, an unmasking step 14.5 us (attribute reads on eight tensors, three allocations through Python, twenty
// converted arguments), for 9-12 us of GPU work; here 6.1 and 7.7 us, most of it the launches.  A whole cycle on one sequence
// of 512 positions (18 calls), host bound before, went from 268 to 211 us.
//
// Every function takes positional arguments only (the Python wrappers own names and defaults), absent tensors as None,
// absent dtype tags as None, and raises what the wrappers' documentation says: ValueError for a bad shape or placement,
// TypeError for a bad element type, the registered error class for a status of the library, torch's own classes for what
// torch throws (torch.OutOfMemoryError when an output or the scratch memory cannot be allocated).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <map>
#include <utility>

#include "../../include/dd.h"

namespace {

struct Raised {};                                            // a Python exception is set

[[noreturn]] void value_error(const char *what, const char *msg)
{
    PyErr_Format(PyExc_ValueError, "%s%s%s", what, *what ? ": " : "", msg);
    throw Raised{};
}

const at::Tensor *opt_tensor(PyObject *o, const char *what)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s: a tensor is required", what);
        throw Raised{};
    }
    return &THPVariable_Unpack(o);
}
const at::Tensor &tensor(PyObject *o, const char *what)
{
    const at::Tensor *t = opt_tensor(o, what);
    if (t == nullptr) {
        PyErr_Format(PyExc_TypeError, "%s: a tensor is required", what);
        throw Raised{};
    }
    return *t;
}
// int(o), and the value as a C int (its low bits, as through ctypes)
int integer(PyObject *o)
{
    PyObject *n = PyNumber_Long(o);
    if (n == nullptr) throw Raised{};
    const unsigned long v = PyLong_AsUnsignedLongMask(n);
    Py_DECREF(n);
    return (int)(unsigned)v;
}
// float(o)
double real(PyObject *o)
{
    PyObject *n = PyNumber_Float(o);
    if (n == nullptr) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(n);
    Py_DECREF(n);
    return v;
}
// an integer as it stands: a float is refused, with the error ctypes has for it
PyObject *exact_integer(PyObject *o, const char *what)
{
    PyObject *n = PyNumber_Index(o);
    if (n != nullptr) return n;
    PyErr_Clear();
    PyObject *ctypes = PyImport_ImportModule("ctypes"), *cls = ctypes ? PyObject_GetAttrString(ctypes, "ArgumentError") : nullptr;
    if (cls != nullptr) PyErr_Format(cls, "%s: an integer is required, not %s", what, Py_TYPE(o)->tp_name);
    Py_XDECREF(cls);
    Py_XDECREF(ctypes);
    throw Raised{};
}

// device pointer of a tensor in GPU memory (nullptr for an absent one)
void *dev(const at::Tensor *t, const char *what)
{
    if (t == nullptr) return nullptr;
    if (!t->is_cuda()) value_error(what, "must live in GPU memory");
    if (!t->is_contiguous()) value_error(what, "must be contiguous");
    return t->data_ptr();
}
void *dev(const at::Tensor &t, const char *what) { return dev(&t, what); }

int dtype_tag(const at::Tensor &t, const char *what)
{
    switch (t.scalar_type()) {
    case at::kFloat: return DD_F32;
    case at::kBFloat16: case at::kShort: case at::kUInt16: return DD_BF16;
    case at::kByte: case at::kFloat8_e4m3fn: return DD_FP8_E4M3;
    default:
        PyErr_Format(PyExc_TypeError, "%s: unsupported tensor dtype %s", what, c10::toString(t.scalar_type()));
        throw Raised{};
    }
}
int tag_or(PyObject *given, const at::Tensor &t, const char *what)
{
    if (given == Py_None) return dtype_tag(t, what);
    PyObject *n = exact_integer(given, "dtype tag");
    const unsigned long v = PyLong_AsUnsignedLongMask(n);
    Py_DECREF(n);
    return (int)(unsigned)v;                                  // (the library refuses what is no tag)
}
// B and G of a verification or unmasking call, whose logits have P rows
std::pair<int64_t, int64_t> batch_and_rows(PyObject *pb, PyObject *pg, int64_t P, const char *rows_msg)
{
    long long v[2];
    PyObject *const o[2] = {pb, pg};
    bool fits = true;
    for (int i = 0; i < 2; ++i) {
        PyObject *n = exact_integer(o[i], i == 0 ? "B" : "G");
        int over = 0;
        v[i] = PyLong_AsLongLongAndOverflow(n, &over);
        Py_DECREF(n);
        fits = fits && over == 0;
    }
    if (!fits || (__int128)v[0] * v[1] != P) value_error("", rows_msg);
    return {v[0], v[1]};
}
void one_byte(const at::Tensor &t, const char *what, const char *msg)
{
    if (t.element_size() != 1) {
        PyErr_Format(PyExc_TypeError, "%s: %s", what, msg);
        throw Raised{};
    }
}
// Shapes say how many elements the library reads and writes, dtype tags how large they are: a tensor that holds fewer bytes
// than that never gets to a launch.
int64_t tag_bytes(int tag) { return tag == DD_F32 ? 4 : tag == DD_BF16 ? 2 : tag == DD_FP8_E4M3 ? 1 : 0; }
void elements_of(const at::Tensor *t, int tag, const char *what)
{
    if (t == nullptr || tag_bytes(tag) == 0 || (int64_t)t->element_size() == tag_bytes(tag)) return;   // (no tag: the library refuses it)
    PyErr_Format(PyExc_TypeError, "%s: elements of %lld bytes expected, has %s", what, (long long)tag_bytes(tag), c10::toString(t->scalar_type()));
    throw Raised{};
}
void room_for(const at::Tensor *t, int64_t elements, int64_t bytes_each, const char *what)
{
    if (t == nullptr || (__int128)t->numel() * t->element_size() >= (__int128)elements * bytes_each) return;
    PyErr_Format(PyExc_ValueError, "%s: too small for %lld elements of %lld bytes", what, (long long)elements, (long long)bytes_each);
    throw Raised{};
}
int64_t out_bytes(int v_tag) { return v_tag == DD_F32 ? 4 : 2; }
// per-head scales
void scales_of(const at::Tensor *t, int64_t heads, const char *what)
{
    if (t == nullptr) return;
    if (t->scalar_type() != at::kFloat) {
        PyErr_Format(PyExc_TypeError, "%s: float32 expected, has %s", what, c10::toString(t->scalar_type()));
        throw Raised{};
    }
    room_for(t, heads, 4, what);
}
bool has_shape(const at::Tensor &t, std::initializer_list<int64_t> s) { return t.sizes() == at::IntArrayRef(s.begin(), s.size()); }

// a per-position vector: n elements of the given type
void check_vec(const at::Tensor *t, int64_t n, at::ScalarType type, const char *what)
{
    if (t == nullptr || (t->scalar_type() == type && t->numel() == n)) return;
    PyErr_Format(PyExc_ValueError, "%s: must have %lld elements of %s, has %lld of %s", what, (long long)n, c10::toString(type),
                 (long long)t->numel(), c10::toString(t->scalar_type()));
    throw Raised{};
}

PyObject *error_class = nullptr;                             // DDError(status, where)
void check(int rc, const char *where)
{
    if (rc == 0) return;
    PyObject *e = error_class ? PyObject_CallFunction(error_class, "is", rc, where) : nullptr;
    if (e != nullptr) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s: status %d", where, rc);
    }
    throw Raised{};
}

hipStream_t current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// ---- scratch memory: one tensor per (device, stream) - calls on one stream run in order and may share it, calls on
// different streams may overlap and must not - or the one a fixed_workspace() block has set.  Guarded by the interpreter
// lock; never destroyed (the runtime may be gone by then).
struct Scratch {
    std::map<std::pair<int, hipStream_t>, at::Tensor> by_stream;
    at::Tensor fixed;
    size_t peak = 0;
};
Scratch &scratch()
{
    static Scratch *s = new Scratch;
    return *s;
}
// (`or_less`: the library itself says whether a fixed workspace of fewer bytes serves the call)
at::Tensor workspace(size_t nbytes, const at::Device &device, hipStream_t stream, bool or_less)
{
    if (nbytes == 0) return at::Tensor();
    Scratch &s = scratch();
    if (nbytes > s.peak) s.peak = nbytes;
    if (s.fixed.defined()) {
        if (((size_t)s.fixed.numel() < nbytes && !or_less) || s.fixed.device() != device) {
            PyErr_Format(PyExc_RuntimeError, "the fixed workspace holds %lld bytes on %s; this call needs %zu on %s",
                         (long long)s.fixed.numel(), s.fixed.device().str().c_str(), nbytes, device.str().c_str());
            throw Raised{};
        }
        return s.fixed;
    }
    if (c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None) {
        // memory allocated under capture would come from that graph's private pool and a cached tensor of it
        // could be handed to a later, unrelated call: the scratch memory of captured calls is allocated beforehand
        PyErr_SetString(PyExc_RuntimeError,
                        "a call that needs scratch memory is being captured without a fixed workspace: "
                        "capture through paper_2604_05250_amd.step.capture_step, or inside fixed_workspace()");
        throw Raised{};
    }
    at::Tensor &t = s.by_stream[{device.index(), stream}];
    if (!t.defined() || (size_t)t.numel() < nbytes)
        t = at::empty({(int64_t)(nbytes > (1u << 20) ? nbytes : (1u << 20))}, at::TensorOptions().dtype(at::kByte).device(device));
    return t;
}

struct Call {                                                // one library call: stream, scratch
    hipStream_t stream;
    at::Tensor ws;
    Call(size_t need, const at::Tensor &on, bool or_less = false) : stream(current_stream()), ws(workspace(need, on.device(), stream, or_less)) {}
    void *ptr() const { return ws.defined() ? ws.data_ptr() : nullptr; }
    size_t bytes() const { return ws.defined() ? (size_t)ws.numel() : 0; }
};
template <typename F> int unlocked(F &&f)                     // the library call itself runs without the interpreter lock
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

// An output.  The allocator is asked directly, past the dispatcher (a cycle of ten calls in fp32 51.1 -> 47.5 us on the host's side, 59.5 -> 56.1
// where it is slower), unless something may be listening there: a dispatch mode, tracer or transform (each adds keys to this thread's
// set), a profiler or another observer of calls, or the fill of uninitialised memory in deterministic mode.  Device, stream, capture pool
// and inference mode are the same either way.
at::Tensor empty_like_type(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &on)
{
    const bool heard = !(c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() || at::hasCallbacks() ||
                       at::globalContext().deterministicAlgorithms();
    if (heard) return at::empty(shape, at::TensorOptions().dtype(type).device(on.device()));
    return at::detail::empty_cuda(shape, type, on.device(), std::nullopt);
}

void want(Py_ssize_t got, Py_ssize_t n)
{
    if (got == n) return;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", n, got);
    throw Raised{};
}

// (Q, K, V, O, q_scale, k_scale, qk_dtype, v_dtype) -> O
PyObject *bidir(PyObject *const *a, Py_ssize_t n)
{
    want(n, 8);
    const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V");
    const at::Tensor *O = opt_tensor(a[3], "O"), *qs = opt_tensor(a[4], "q_scale"), *ks = opt_tensor(a[5], "k_scale");
    if (Q.dim() != 4 || K.dim() != 4) value_error("", "Q, K, V must have four dimensions");
    const int64_t B = Q.size(0), H = Q.size(1), N = Q.size(2), d = Q.size(3), Hkv = K.size(1);
    if (!has_shape(K, {B, Hkv, N, d}) || !has_shape(V, {B, Hkv, N, d})) value_error("", "K/V shape must be [B,Hkv,N,d] matching Q");
    const int qk = tag_or(a[6], Q, "Q"), vd = tag_or(a[7], V, "V");
    elements_of(&Q, qk, "Q"); elements_of(&K, qk, "K"); elements_of(&V, vd, "V");
    room_for(O, B * H * N * d, out_bytes(vd), "O");
    scales_of(qs, B * H, "q_scale"); scales_of(ks, B * Hkv, "k_scale");
    void *const q = dev(Q, "Q"), *const k = dev(K, "K"), *const v = dev(V, "V");
    const at::Tensor out = O ? *O : empty_like_type({B, H, N, d}, V.scalar_type(), V);
    void *const o = dev(out, "O");
    const float *q_s = (const float *)dev(qs, "q_scale"), *k_s = (const float *)dev(ks, "k_scale");
    const Call c(dd_bidir_attention_workspace_bytes(B, H, Hkv, N, d, (dd_dtype)qk, (dd_dtype)vd), Q);
    check(unlocked([&] { return dd_bidir_attention(q, k, v, o, B, H, Hkv, N, d, (dd_dtype)qk, (dd_dtype)vd, q_s, k_s, c.ptr(),
                                                   c.bytes(), c.stream); }), "dd_bidir_attention");
    return THPVariable_Wrap(out);
}

enum { kCached = 0, kRefresh = 1, kWindow = 2, kBatched = 3 };
// (kind, Qblk, Kc, Vc, block_start | block_starts, win_start, win_len, O, Kblk, Vblk, q_scale, k_scale, qk_dtype, v_dtype) -> O
PyObject *block(PyObject *const *a, Py_ssize_t n)
{
    want(n, 14);
    const int kind = integer(a[0]);
    const at::Tensor &Q = tensor(a[1], "Qblk"), &Kc = tensor(a[2], "Kc"), &Vc = tensor(a[3], "Vc");
    const at::Tensor *O = opt_tensor(a[7], "O"), *Kb = opt_tensor(a[8], "Kblk"), *Vb = opt_tensor(a[9], "Vblk");
    const at::Tensor *qs = opt_tensor(a[10], "q_scale"), *ks = opt_tensor(a[11], "k_scale");
    if (Q.dim() != 4 || Kc.dim() != 4) value_error("", "Qblk, Kc, Vc must have four dimensions");
    const int64_t B = Q.size(0), H = Q.size(1), bl = Q.size(2), d = Q.size(3), Hkv = Kc.size(1), N = Kc.size(2);
    if (!has_shape(Kc, {B, Hkv, N, d}) || !has_shape(Vc, {B, Hkv, N, d})) value_error("", "Kc/Vc shape must be [B,Hkv,N,d]");
    if (kind == kBatched && (!Kb || !Vb)) value_error("", "Kblk and Vblk are required");
    if (Kb && !(has_shape(*Kb, {B, Hkv, bl, d}) && Vb && has_shape(*Vb, {B, Hkv, bl, d}))) value_error("", "Kblk/Vblk shape must be [B,Hkv,block_len,d]");
    const int qk = tag_or(a[12], Q, "Qblk"), vd = tag_or(a[13], Vc, "Vc");
    elements_of(&Q, qk, "Qblk"); elements_of(&Kc, qk, "Kc"); elements_of(&Vc, vd, "Vc");
    elements_of(Kb, qk, "Kblk"); elements_of(Vb, vd, "Vblk");
    room_for(O, B * H * bl * d, out_bytes(vd), "O");
    scales_of(qs, B * H, "q_scale"); scales_of(ks, B * Hkv, "k_scale");
    const at::Tensor *starts = nullptr;
    int bs = 0, ws0 = 0, wsn = 0;
    if (kind == kBatched) {
        starts = &tensor(a[4], "block_starts");
        if (starts->scalar_type() != at::kInt || starts->numel() != B) value_error("", "block_starts must be int32 with B entries");
    } else {
        bs = integer(a[4]);
    }
    if (kind == kWindow) {
        ws0 = integer(a[5]);
        wsn = integer(a[6]);
    }
    void *const q = dev(Q, "Qblk"), *const k = dev(Kc, "Kc"), *const v = dev(Vc, "Vc"), *const kb = dev(Kb, "Kblk"), *const vb = dev(Vb, "Vblk");
    const at::Tensor out = O ? *O : empty_like_type({B, H, bl, d}, Vc.scalar_type(), Vc);
    void *const o = dev(out, "O");
    const float *q_s = (const float *)dev(qs, "q_scale"), *k_s = (const float *)dev(ks, "k_scale");
    const int32_t *st = (const int32_t *)dev(starts, "block_starts");
    const dd_dtype tq = (dd_dtype)qk, tv = (dd_dtype)vd;
    const Call c(kind == kWindow ? dd_block_attention_window_workspace_bytes(bl, wsn, B, H, Hkv, N, d, tq, tv)
                                 : dd_block_attention_cached_workspace_bytes(bl, B, H, Hkv, N, d, tq, tv), Q);
    switch (kind) {
    case kCached:
        check(unlocked([&] { return dd_block_attention_cached(q, k, v, o, bs, bl, kb, vb, B, H, Hkv, N, d, tq, tv, q_s, k_s, c.ptr(),
                                                              c.bytes(), c.stream); }), "dd_block_attention_cached");
        break;
    case kRefresh:
        check(unlocked([&] { return dd_block_attention_refresh(q, k, v, o, bs, bl, kb, vb, B, H, Hkv, N, d, tq, tv, q_s, k_s, c.ptr(),
                                                               c.bytes(), c.stream); }), "dd_block_attention_refresh");
        break;
    case kWindow:
        check(unlocked([&] { return dd_block_attention_window(q, k, v, o, bs, bl, ws0, wsn, kb, vb, B, H, Hkv, N, d, tq, tv, q_s, k_s,
                                                              c.ptr(), c.bytes(), c.stream); }), "dd_block_attention_window");
        break;
    default:
        check(unlocked([&] { return dd_block_attention_batched(q, k, v, o, st, bl, kb, vb, B, H, Hkv, N, d, tq, tv, q_s, k_s, c.ptr(),
                                                               c.bytes(), c.stream); }), "dd_block_attention_batched");
    }
    return THPVariable_Wrap(out);
}

// (Q, K, V, q_scale, k_scale, v_scale, O) -> O
PyObject *bidir_fp8v(PyObject *const *a, Py_ssize_t n)
{
    want(n, 7);
    const at::Tensor &Q = tensor(a[0], "Q"), &K = tensor(a[1], "K"), &V = tensor(a[2], "V");
    const at::Tensor *qs = opt_tensor(a[3], "q_scale"), *ks = opt_tensor(a[4], "k_scale"), *vs = opt_tensor(a[5], "v_scale");
    const at::Tensor *O = opt_tensor(a[6], "O");
    if (Q.dim() != 4 || K.dim() != 4) value_error("", "Q, K, V must have four dimensions");
    const int64_t B = Q.size(0), H = Q.size(1), N = Q.size(2), d = Q.size(3), Hkv = K.size(1);
    if (!has_shape(K, {B, Hkv, N, d}) || !has_shape(V, {B, Hkv, N, d})) value_error("", "K/V shape must be [B,Hkv,N,d] matching Q");
    const char *msg = "one byte per element (e4m3 codes) expected";
    one_byte(Q, "Q", msg); one_byte(K, "K", msg); one_byte(V, "V", msg);
    room_for(O, B * H * N * d, 2, "O");
    scales_of(qs, B * H, "q_scale"); scales_of(ks, B * Hkv, "k_scale"); scales_of(vs, B * Hkv, "v_scale");
    void *const q = dev(Q, "Q"), *const k = dev(K, "K"), *const v = dev(V, "V");
    const at::Tensor out = O ? *O : empty_like_type({B, H, N, d}, at::kShort, V);
    void *const o = dev(out, "O");
    const float *q_s = (const float *)dev(qs, "q_scale"), *k_s = (const float *)dev(ks, "k_scale"), *v_s = (const float *)dev(vs, "v_scale");
    const hipStream_t stream = current_stream();
    check(unlocked([&] { return dd_bidir_attention_fp8v(q, k, v, o, B, H, Hkv, N, d, q_s, k_s, v_s, stream); }), "dd_bidir_attention_fp8v");
    return THPVariable_Wrap(out);
}

// (Q, Qs, K, Ks, V, Vs, O) -> O
PyObject *bidir_mx(PyObject *const *a, Py_ssize_t n)
{
    want(n, 7);
    const at::Tensor &Q = tensor(a[0], "Q"), &Qs = tensor(a[1], "Qs"), &K = tensor(a[2], "K"), &Ks = tensor(a[3], "Ks");
    const at::Tensor &V = tensor(a[4], "V"), &Vs = tensor(a[5], "Vs");
    const at::Tensor *O = opt_tensor(a[6], "O");
    if (Q.dim() != 4 || K.dim() != 4) value_error("", "Q, K, V must have four dimensions");
    const int64_t B = Q.size(0), H = Q.size(1), N = Q.size(2), d = Q.size(3), Hkv = K.size(1);
    if (!has_shape(K, {B, Hkv, N, d}) || !has_shape(V, {B, Hkv, N, d / 2})) value_error("", "K must be [B,Hkv,N,d] and V [B,Hkv,N,d/2] matching Q");
    if (!has_shape(Qs, {B, H, N, d / 32}) || !has_shape(Ks, {B, Hkv, N, d / 32}) || !has_shape(Vs, {B, Hkv, N, d / 32}))
        value_error("", "scales must be [..., d/32] matching their tensors");
    const char *msg = "one byte per entry expected";
    one_byte(Q, "Q", msg); one_byte(K, "K", msg); one_byte(V, "V", msg);
    one_byte(Qs, "Qs", msg); one_byte(Ks, "Ks", msg); one_byte(Vs, "Vs", msg);
    room_for(O, B * H * N * d, 2, "O");
    void *const q = dev(Q, "Q"), *const q_s = dev(Qs, "Qs"), *const k = dev(K, "K"), *const k_s = dev(Ks, "Ks"), *const v = dev(V, "V"), *const v_s = dev(Vs, "Vs");
    const at::Tensor out = O ? *O : empty_like_type({B, H, N, d}, at::kShort, V);
    void *const o = dev(out, "O");
    const hipStream_t stream = current_stream();
    check(unlocked([&] { return dd_bidir_attention_mx(q, q_s, k, k_s, v, v_s, o, B, H, Hkv, N, d, stream); }), "dd_bidir_attention_mx");
    return THPVariable_Wrap(out);
}

// (Qblk, Kc, Vc, block_start, q_scale, k_scale, v_scale, O, Kblk, Vblk) -> O
PyObject *block_fp8v(PyObject *const *a, Py_ssize_t n)
{
    want(n, 10);
    const at::Tensor &Q = tensor(a[0], "Qblk"), &Kc = tensor(a[1], "Kc"), &Vc = tensor(a[2], "Vc");
    const int bs = integer(a[3]);
    const at::Tensor *qs = opt_tensor(a[4], "q_scale"), *ks = opt_tensor(a[5], "k_scale"), *vs = opt_tensor(a[6], "v_scale");
    const at::Tensor *O = opt_tensor(a[7], "O"), *Kb = opt_tensor(a[8], "Kblk"), *Vb = opt_tensor(a[9], "Vblk");
    if (Q.dim() != 4 || Kc.dim() != 4) value_error("", "Qblk, Kc, Vc must have four dimensions");
    const int64_t B = Q.size(0), H = Q.size(1), bl = Q.size(2), d = Q.size(3), Hkv = Kc.size(1), N = Kc.size(2);
    if (!has_shape(Kc, {B, Hkv, N, d}) || !has_shape(Vc, {B, Hkv, N, d})) value_error("", "Kc/Vc shape must be [B,Hkv,N,d]");
    if (Kb && !(has_shape(*Kb, {B, Hkv, bl, d}) && Vb && has_shape(*Vb, {B, Hkv, bl, d}))) value_error("", "Kblk/Vblk shape must be [B,Hkv,block_len,d]");
    const char *msg = "one byte per element (e4m3 codes) expected";
    one_byte(Q, "Qblk", msg); one_byte(Kc, "Kc", msg); one_byte(Vc, "Vc", msg);
    if (Kb) { one_byte(*Kb, "Kblk", msg); one_byte(*Vb, "Vblk", msg); }
    room_for(O, B * H * bl * d, 2, "O");
    scales_of(qs, B * H, "q_scale"); scales_of(ks, B * Hkv, "k_scale"); scales_of(vs, B * Hkv, "v_scale");
    void *const q = dev(Q, "Qblk"), *const k = dev(Kc, "Kc"), *const v = dev(Vc, "Vc"), *const kb = dev(Kb, "Kblk"), *const vb = dev(Vb, "Vblk");
    const at::Tensor out = O ? *O : empty_like_type({B, H, bl, d}, at::kShort, Vc);
    void *const o = dev(out, "O");
    const float *q_s = (const float *)dev(qs, "q_scale"), *k_s = (const float *)dev(ks, "k_scale"), *v_s = (const float *)dev(vs, "v_scale");
    const Call c(dd_block_attention_cached_fp8v_workspace_bytes(bl, B, H, Hkv, N, d), Q);
    check(unlocked([&] { return dd_block_attention_cached_fp8v(q, k, v, o, bs, bl, kb, vb, B, H, Hkv, N, d, q_s, k_s, v_s, c.ptr(), c.bytes(),
                                                               c.stream); }), "dd_block_attention_cached_fp8v");
    return THPVariable_Wrap(out);
}

// (Kc, Vc, Krows, Vrows, positions, qk_dtype, v_dtype) -> None
PyObject *cache_insert(PyObject *const *a, Py_ssize_t n)
{
    want(n, 7);
    const at::Tensor &Kc = tensor(a[0], "Kc"), &Vc = tensor(a[1], "Vc"), &Kr = tensor(a[2], "Krows"), &Vr = tensor(a[3], "Vrows");
    const at::Tensor &pos = tensor(a[4], "positions");
    if (Kc.dim() != 4 || Kr.dim() != 4) value_error("", "Kc, Vc, Krows, Vrows must have four dimensions");
    const int64_t B = Kc.size(0), Hkv = Kc.size(1), N = Kc.size(2), d = Kc.size(3), rows = Kr.size(2);
    if (!has_shape(Vc, {B, Hkv, N, d}) || !has_shape(Kr, {B, Hkv, rows, d}) || !has_shape(Vr, {B, Hkv, rows, d}))
        value_error("", "shapes must be Kc,Vc [B,Hkv,N,d] and Krows,Vrows [B,Hkv,n,d]");
    if (pos.scalar_type() != at::kInt || pos.numel() != B * rows) value_error("", "positions must be int32 with B*n entries");
    const int qk = tag_or(a[5], Kc, "Kc"), vd = tag_or(a[6], Vc, "Vc");
    elements_of(&Kc, qk, "Kc"); elements_of(&Kr, qk, "Krows"); elements_of(&Vc, vd, "Vc"); elements_of(&Vr, vd, "Vrows");
    void *const k = dev(Kc, "Kc"), *const v = dev(Vc, "Vc"), *const kr = dev(Kr, "Krows"), *const vr = dev(Vr, "Vrows"), *const p = dev(pos, "positions");
    const hipStream_t stream = current_stream();
    check(unlocked([&] { return dd_cache_insert_rows(k, v, kr, vr, (const int32_t *)p, rows, B, Hkv, N, d, (dd_dtype)qk, (dd_dtype)vd, stream); }),
          "dd_cache_insert_rows");
    Py_RETURN_NONE;
}

PyObject *triple(const at::Tensor &x, const at::Tensor &y, const at::Tensor &z)
{
    PyObject *t = PyTuple_New(3);
    if (t == nullptr) throw Raised{};
    PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(x));
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(y));
    PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(z));
    return t;
}

// (static, logits_d, logits_v, mask, mode, threshold, seed, B, G, out_mask, out_tokens, out_scores, logit_dtype) -> the three outputs
PyObject *verify_remask(PyObject *const *a, Py_ssize_t n)
{
    want(n, 13);
    const bool fixed_scratch = integer(a[0]) != 0;
    const at::Tensor *D = opt_tensor(a[1], "logits_d");
    const at::Tensor &L = tensor(a[2], "logits_v");
    const at::Tensor *mask = opt_tensor(a[3], "mask"), *om = opt_tensor(a[9], "out_mask"), *ot = opt_tensor(a[10], "out_tokens"), *os = opt_tensor(a[11], "out_scores");
    const int mode = integer(a[4]);
    const float threshold = (float)real(a[5]);
    PyObject *seed_int = PyNumber_Long(a[6]);
    if (seed_int == nullptr) throw Raised{};
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(seed_int);
    Py_DECREF(seed_int);
    if (PyErr_Occurred()) throw Raised{};
    if (L.dim() != 2) value_error("", "logits_v must have two dimensions");
    const int64_t P = L.size(0), V = L.size(1);
    const std::pair<int64_t, int64_t> bg = batch_and_rows(a[7], a[8], P, "logits_v must have B*G rows");
    const int64_t B = bg.first, G = bg.second;
    if (D && !has_shape(*D, {P, V})) value_error("", "logits_d shape must match logits_v");
    const dd_dtype dt = (dd_dtype)tag_or(a[12], L, "logits_v");
    elements_of(&L, dt, "logits_v");
    if (mode == DD_KL_THRESH || mode == DD_KL_PROB || mode == DD_KL_TOPK) elements_of(D, dt, "logits_d");   // (the other rules do not read them)
    check_vec(mask, P, at::kByte, "mask");
    check_vec(om, P, at::kByte, "out_mask");
    check_vec(ot, P, at::kInt, "out_tokens");
    check_vec(os, P, at::kFloat, "out_scores");
    void *const ld = dev(D, "logits_d"), *const lv = dev(L, "logits_v"), *const mk = dev(mask, "mask");
    // (with the static scratch an absent output stays absent: the library says what it makes of that)
    auto output = [&](const at::Tensor *given, at::ScalarType type) { return given ? *given : fixed_scratch ? at::Tensor() : empty_like_type({P}, type, L); };
    const at::Tensor rm = output(om, at::kByte), rt = output(ot, at::kInt), rs = output(os, at::kFloat);
    uint8_t *const pm = (uint8_t *)dev(rm.defined() ? &rm : nullptr, "out_mask");
    int32_t *const pt = (int32_t *)dev(rt.defined() ? &rt : nullptr, "out_tokens");
    float *const ps = (float *)dev(rs.defined() ? &rs : nullptr, "out_scores");
    if (fixed_scratch) {
        const hipStream_t stream = current_stream();
        check(unlocked([&] { return dd_verify_remask_static(ld, lv, (const uint8_t *)mk, (dd_mode)mode, threshold, seed, pm, pt, ps, B, G, V, dt, stream); }),
              "dd_verify_remask_static");
    } else {
        const Call c(dd_verify_remask_workspace_bytes(B, G, V, dt), L, true);
        check(unlocked([&] { return dd_verify_remask(ld, lv, (const uint8_t *)mk, (dd_mode)mode, threshold, seed, pm, pt, ps, B, G, V, dt, c.ptr(),
                                                     c.bytes(), c.stream); }), "dd_verify_remask");
    }
    return triple(rm, rt, rs);
}

// (logits_d, mask, mode, threshold, B, G, x_tokens, out_mask, out_tokens, out_conf, logit_dtype) -> the three outputs
PyObject *unmask(PyObject *const *a, Py_ssize_t n)
{
    want(n, 11);
    const at::Tensor &L = tensor(a[0], "logits_d");
    const at::Tensor *mask = opt_tensor(a[1], "mask"), *x = opt_tensor(a[6], "x_tokens");
    const at::Tensor *om = opt_tensor(a[7], "out_mask"), *ot = opt_tensor(a[8], "out_tokens"), *oc = opt_tensor(a[9], "out_conf");
    const int mode = integer(a[2]);
    const float threshold = (float)real(a[3]);
    if (L.dim() != 2) value_error("", "logits_d must have two dimensions");
    const int64_t P = L.size(0), V = L.size(1);
    const std::pair<int64_t, int64_t> bg = batch_and_rows(a[4], a[5], P, "logits_d must have B*G rows");
    const int64_t B = bg.first, G = bg.second;
    const dd_dtype dt = (dd_dtype)tag_or(a[10], L, "logits_d");
    elements_of(&L, dt, "logits_d");
    check_vec(mask, P, at::kByte, "mask");
    check_vec(x, P, at::kInt, "x_tokens");
    check_vec(om, P, at::kByte, "out_mask");
    check_vec(ot, P, at::kInt, "out_tokens");
    check_vec(oc, P, at::kFloat, "out_conf");
    void *const ld = dev(L, "logits_d"), *const mk = dev(mask, "mask");
    int32_t *const px = (int32_t *)dev(x, "x_tokens");
    const at::Tensor rm = om ? *om : empty_like_type({P}, at::kByte, L);
    const at::Tensor rt = ot ? *ot : empty_like_type({P}, at::kInt, L);
    const at::Tensor rc = oc ? *oc : empty_like_type({P}, at::kFloat, L);
    uint8_t *const pm = (uint8_t *)dev(rm, "out_mask");
    int32_t *const pt = (int32_t *)dev(rt, "out_tokens");
    float *const pc = (float *)dev(rc, "out_conf");
    const Call c(dd_unmask_workspace_bytes(B, G, V, dt), L, true);
    check(unlocked([&] { return dd_unmask(ld, (const uint8_t *)mk, (dd_unmask_mode)mode, threshold, px, pm, pt, pc, B, G, V, dt, c.ptr(), c.bytes(),
                                          c.stream); }), "dd_unmask");
    return triple(rm, rt, rc);
}

// (logits_d, logits_v, drafter, logit_dtype) -> (kl, conf_v, tok_v, conf_d | None, tok_d | None)
PyObject *verify_scores(PyObject *const *a, Py_ssize_t n)
{
    want(n, 4);
    const at::Tensor &D = tensor(a[0], "logits_d"), &L = tensor(a[1], "logits_v");
    const int drafter = PyObject_IsTrue(a[2]);
    if (drafter < 0) throw Raised{};
    if (L.dim() != 2) value_error("", "logits_v must have two dimensions");
    const int64_t P = L.size(0), V = L.size(1);
    if (!has_shape(D, {P, V})) value_error("", "logits_d and logits_v must have the same shape");
    const bool given = a[3] != Py_None;
    const dd_dtype dt = (dd_dtype)tag_or(a[3], L, "logits_v");
    if (!given && dtype_tag(D, "logits_d") != dt) value_error("", "logits_d and logits_v must have the same dtype");
    elements_of(&L, dt, "logits_v"); elements_of(&D, dt, "logits_d");
    void *const ld = dev(D, "logits_d"), *const lv = dev(L, "logits_v");
    const at::Tensor kl = empty_like_type({P}, at::kFloat, L), cv = empty_like_type({P}, at::kFloat, L), tv = empty_like_type({P}, at::kInt, L);
    const at::Tensor cd = drafter ? empty_like_type({P}, at::kFloat, L) : at::Tensor(), td = drafter ? empty_like_type({P}, at::kInt, L) : at::Tensor();
    const Call c(dd_verify_scores_workspace_bytes(P, V, dt), L, true);
    float *const pk = (float *)kl.data_ptr(), *const pcv = (float *)cv.data_ptr(), *const pcd = drafter ? (float *)cd.data_ptr() : nullptr;
    int32_t *const ptv = (int32_t *)tv.data_ptr(), *const ptd = drafter ? (int32_t *)td.data_ptr() : nullptr;
    check(unlocked([&] { return dd_verify_scores(ld, lv, pk, pcv, ptv, pcd, ptd, P, V, dt, c.ptr(), c.bytes(), c.stream); }), "dd_verify_scores");
    PyObject *t = PyTuple_New(5);
    if (t == nullptr) throw Raised{};
    PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(kl));
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(cv));
    PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(tv));
    if (drafter) {
        PyTuple_SET_ITEM(t, 3, THPVariable_Wrap(cd));
        PyTuple_SET_ITEM(t, 4, THPVariable_Wrap(td));
    } else {
        Py_INCREF(Py_None); PyTuple_SET_ITEM(t, 3, Py_None);
        Py_INCREF(Py_None); PyTuple_SET_ITEM(t, 4, Py_None);
    }
    return t;
}

// (DDError) -> None
PyObject *set_error_class(PyObject *const *a, Py_ssize_t n)
{
    want(n, 1);
    Py_INCREF(a[0]);
    Py_XDECREF(error_class);
    error_class = a[0];
    Py_RETURN_NONE;
}
// (tensor | None) -> the one set before, or None
PyObject *set_fixed_workspace(PyObject *const *a, Py_ssize_t n)
{
    want(n, 1);
    const at::Tensor *t = opt_tensor(a[0], "workspace");
    if (t) dev(t, "workspace");
    at::Tensor prev = scratch().fixed;
    scratch().fixed = t ? *t : at::Tensor();
    if (!prev.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(prev);
}
PyObject *reset_workspace_peak(PyObject *const *, Py_ssize_t n)
{
    want(n, 0);
    scratch().peak = 0;
    Py_RETURN_NONE;
}
PyObject *workspace_peak(PyObject *const *, Py_ssize_t n)
{
    want(n, 0);
    return PyLong_FromSize_t(scratch().peak);
}

template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        return F(a, n);
    } catch (const Raised &) {
        return nullptr;
    } catch (...) {                                          // as torch itself raises it: torch.OutOfMemoryError for an allocation
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}
#define DD_METHOD(name) {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DD_METHOD(bidir), DD_METHOD(block), DD_METHOD(bidir_fp8v), DD_METHOD(bidir_mx), DD_METHOD(block_fp8v),
                         DD_METHOD(cache_insert), DD_METHOD(verify_remask), DD_METHOD(unmask), DD_METHOD(verify_scores),
                         DD_METHOD(set_error_class), DD_METHOD(set_fixed_workspace), DD_METHOD(reset_workspace_peak),
                         DD_METHOD(workspace_peak), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "argument marshalling of paper_2604_05250_amd", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
