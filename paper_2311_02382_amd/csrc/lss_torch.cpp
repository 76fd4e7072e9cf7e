// The binding's argument marshalling in native code: a CPython module whose functions take torch tensors, check
// them, allocate outputs that were not passed and call the C ABI (include/lss_attn.h) on the current stream.
// lss.py declares the public signatures and forwards positionally to the functions here.
//
// Why native: a pass over short segments is a dozen calls of a few microseconds of GPU work each, and the same
// marshalling in Python with ctypes took 13 us per call (attribute look-ups on up to nine tensors, one ctypes
// object per pointer), more than the kernels it launched; here it is below 1 us beside the launches.
//
// Errors: a tensor that does not fit raises ValueError; a status code of the library raises the exception type
// handed in through set_error_type() as type(code, message); torch's own errors keep their types (OutOfMemoryError).
#include "lss_attn.h"

#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <map>
#include <stdexcept>
#include <vector>

namespace lss {
size_t least_workspace_bytes(int l_s, int l_x, int B, int H, int d, int elem_bytes);       // lss_kernels.h, which is HIP code's
}

namespace {

PyObject *g_error_type = nullptr;

struct PythonError {};      // a Python exception is set
struct ValueError : std::runtime_error { using std::runtime_error::runtime_error; };

constexpr auto kBf16 = at::kBFloat16;
constexpr auto kF32 = at::kFloat;

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %s", Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    return THPVariable_Unpack(o);
}
bool none(PyObject *o) { return o == Py_None; }
int64_t integer(PyObject *o)
{
    const long long v = PyLong_Check(o) ? PyLong_AsLongLong(o) : [&] {
        PyObject *i = PyNumber_Long(o);
        if (!i) throw PythonError{};
        const long long r = PyLong_AsLongLong(i);
        Py_DECREF(i);
        return r;
    }();
    if (v == -1 && PyErr_Occurred()) throw PythonError{};
    return v;
}
uint64_t seed_bits(PyObject *o)     // any integer, reduced modulo 2^64
{
    PyObject *i = PyNumber_Long(o);
    if (!i) throw PythonError{};
    const unsigned long long r = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (r == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError{};
    return r;
}
double real(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PythonError{};
    return v;
}
bool truth(PyObject *o)
{
    const int t = PyObject_IsTrue(o);
    if (t < 0) throw PythonError{};
    return t != 0;
}

void require(bool ok, const char *msg)
{
    if (!ok) throw ValueError(msg);
}
bool on_gpu(const at::Tensor &t) { return t.is_cuda() && t.is_contiguous(); }
bool plain(const at::Tensor &t, at::ScalarType dt) { return on_gpu(t) && t.scalar_type() == dt; }
bool shaped(const at::Tensor &t, std::initializer_list<int64_t> s) { return t.sizes() == at::IntArrayRef(s.begin(), s.size()); }
void dev(const at::Tensor &t, at::ScalarType dt, const char *what)
{
    if (!plain(t, dt))
        throw ValueError(std::string(what) + " must be a contiguous " + (dt == kBf16 ? "torch.bfloat16" : dt == kF32 ? "torch.float32" : "torch.uint8") + " device tensor");
}

at::Tensor fresh(at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(dt).device(like.device()));
}
std::string written(at::IntArrayRef shape)      // as Python writes a tuple
{
    std::string s = "(";
    for (size_t i = 0; i < shape.size(); ++i) s += (i ? ", " : "") + std::to_string(shape[i]);
    return s + (shape.size() == 1 ? ",)" : ")");
}
// the caller's output if given (checked), else a new tensor
at::Tensor output(PyObject *o, at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like)
{
    if (none(o)) return fresh(shape, dt, like);
    const at::Tensor &t = tensor(o);
    if (t.sizes() != shape) throw ValueError("output has shape " + written(t.sizes()) + ", expected " + written(shape));
    dev(t, dt, "output");
    return t;
}
// outputs whose shape and type the caller vouches for (the attention calls check sizes only through the library)
at::Tensor output_as_is(PyObject *o, at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like)
{
    return none(o) ? fresh(shape, dt, like) : tensor(o);
}
void *ptr(const at::Tensor &t) { return t.data_ptr(); }
float *fptr(const at::Tensor &t) { return static_cast<float *>(t.data_ptr()); }

void *stream_of(PyObject *o)
{
    if (none(o)) return c10::hip::getCurrentHIPStream().stream();
    PyObject *h = PyObject_HasAttrString(o, "cuda_stream") ? PyObject_GetAttrString(o, "cuda_stream") : PyNumber_Long(o);
    if (!h) throw PythonError{};
    const unsigned long long v = PyLong_AsUnsignedLongLong(h);
    Py_DECREF(h);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError{};
    return reinterpret_cast<void *>(v);
}

void check(int rc)
{
    if (rc == LSS_OK) return;
    PyObject *exc = g_error_type ? PyObject_CallFunction(g_error_type, "is", rc, lss_last_error()) : nullptr;
    if (exc) {
        PyErr_SetObject(g_error_type, exc);
        Py_DECREF(exc);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "status %d: %s", rc, lss_last_error());
    }
    throw PythonError{};
}

// One call of the library, without the interpreter lock (a launch may wait for room in the stream's queue).
template <typename F, typename... A>
void invoke(F f, A... args)
{
    PyThreadState *ts = PyEval_SaveThread();
    const int rc = f(args...);
    PyEval_RestoreThread(ts);
    check(rc);
}

PyObject *wrap(const at::Tensor &t) { return THPVariable_Wrap(t); }
// (an output that was passed in is returned as the object it was passed as)
PyObject *give(PyObject *passed, const at::Tensor &t)
{
    if (none(passed)) return wrap(t);
    Py_INCREF(passed);
    return passed;
}
PyObject *pack(std::initializer_list<PyObject *> items)
{
    PyObject *r = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject *o : items) PyTuple_SET_ITEM(r, i++, o);
    return r;
}

// ---- scratch of the attention calls: one buffer per GPU, passed with every call and registered with the
// library by every call (direct calls of the C entry points without a buffer of their own find it there).  Outgrown buffers are kept alive, because kernels in flight may still use them and nothing here
// synchronises; a buffer at least doubles when it grows, so together they stay below the current one.
// (All of this runs under the interpreter lock.)
std::map<int, at::Tensor> g_ws;
std::vector<at::Tensor> g_ws_retired;

void *shared_workspace(size_t need, const at::Tensor &like, size_t &bytes)
{
    at::Tensor &cur = g_ws[like.device().index()];
    if (!cur.defined() || (size_t)cur.numel() < need) {
        int64_t grown = 1 << 20;
        if (cur.defined()) { grown = 2 * cur.numel(); g_ws_retired.push_back(cur); }
        cur = fresh({(int64_t)need > grown ? (int64_t)need : grown}, at::kByte, like);
    }
    check(lss_set_workspace(ptr(cur), (size_t)cur.numel()));
    bytes = (size_t)cur.numel();
    return ptr(cur);
}

struct Dims { int64_t B, l_s, l_x, H, d; int eb; };
Dims dims(const at::Tensor &q, const at::Tensor &k, const at::Tensor &v)
{
    require(q.dim() == 4 && k.dim() == 4 && k.sizes() == v.sizes(), "q_seg, k, v must be [B, L, H, d] with k.shape == v.shape");
    Dims m{q.size(0), q.size(1), k.size(1), q.size(2), q.size(3), 0};
    require(k.size(0) == m.B && k.size(2) == m.H && k.size(3) == m.d, "q_seg and k disagree on B, H or d");
    require(on_gpu(q) && on_gpu(k) && on_gpu(v), "tensors must be contiguous device tensors");
    const auto dt = q.scalar_type();
    require(k.scalar_type() == dt && v.scalar_type() == dt && (dt == kBf16 || dt == kF32), "q_seg, k, v must share dtype bfloat16 or float32");
    m.eb = dt == kF32 ? 4 : 2;
    return m;
}
// scratch for a call of this shape: the caller's own tensor (checked) or the shared one
void *scratch_for(PyObject *workspace, const Dims &m, const at::Tensor &like, size_t &bytes)
{
    const size_t need = lss_workspace_bytes(m.l_s, m.l_x, m.B, m.H, m.d, m.eb);
    if (none(workspace)) return shared_workspace(need, like, bytes);
    const at::Tensor &w = tensor(workspace);
    require(on_gpu(w), "workspace must be a contiguous device tensor");
    bytes = (size_t)w.numel() * w.element_size();
    // (no less than the library itself accepts)
    if (need > 0 && bytes < lss::least_workspace_bytes((int)m.l_s, (int)m.l_x, (int)m.B, (int)m.H, (int)m.d, m.eb))
        throw ValueError("workspace of " + std::to_string(bytes) + " bytes, need " + std::to_string(need));
    return ptr(w);
}
void like_q(const at::Tensor &t, const at::Tensor &q, const char *msg)
{
    require(t.sizes() == q.sizes() && t.scalar_type() == q.scalar_type() && t.is_contiguous(), msg);
}
void check_lse(const at::Tensor &lse, const Dims &m)
{
    require(shaped(lse, {m.B, m.H, m.l_s}) && lse.scalar_type() == kF32 && lse.is_contiguous(), "lse must be contiguous float32 [B, H, l_s]");
}

// ------------------------------------------------------------------------------------ attention
// q_seg k v seg_offset causal out lse stream p_drop seed workspace
PyObject *attn_fwd(PyObject *const *a)
{
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    const Dims m = dims(q, k, v);
    const at::Tensor out = none(a[5]) ? at::empty_like(q) : tensor(a[5]);
    const at::Tensor lse = output_as_is(a[6], {m.B, m.H, m.l_s}, kF32, q);
    size_t wn;
    void *wp = scratch_for(a[10], m, q, wn);
    invoke(lss_segment_attn_fwd_ex, ptr(q), ptr(k), ptr(v), integer(a[3]), m.l_s, m.l_x, m.B, m.H, m.d, truth(a[4]),
                                  none(a[8]) ? 0.0 : real(a[8]), seed_bits(a[9]), m.eb, 0, wp, wn, ptr(out), fptr(lse), stream_of(a[7]));
    return pack({give(a[5], out), give(a[6], lse)});
}
// q_seg k v seg_offset out lse d_out causal dq dk_partial dv_partial stream p_drop seed skip_masked_tail workspace
PyObject *attn_bwd(PyObject *const *a)
{
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &out = tensor(a[4]), &lse = tensor(a[5]), &d_out = tensor(a[6]);
    const Dims m = dims(q, k, v);
    like_q(out, q, "out and d_out must match q_seg in shape and dtype and be contiguous");
    like_q(d_out, q, "out and d_out must match q_seg in shape and dtype and be contiguous");
    check_lse(lse, m);
    const at::Tensor dq = none(a[8]) ? at::empty_like(q) : tensor(a[8]);
    const at::Tensor dk = output_as_is(a[9], k.sizes(), kF32, k), dv = output_as_is(a[10], k.sizes(), kF32, k);
    size_t wn;
    void *wp = scratch_for(a[15], m, q, wn);
    invoke(lss_segment_attn_bwd_ex, ptr(q), ptr(k), ptr(v), integer(a[3]), m.l_s, m.l_x, m.B, m.H, m.d, truth(a[7]),
                                  none(a[12]) ? 0.0 : real(a[12]), seed_bits(a[13]), m.eb, truth(a[14]) ? LSS_FLAG_SKIP_MASKED_TAIL : 0u,
                                  wp, wn, ptr(out), fptr(lse), ptr(d_out), ptr(dq), fptr(dk), fptr(dv), stream_of(a[11]));
    return pack({give(a[8], dq), give(a[9], dk), give(a[10], dv)});
}
// q_seg k v seg_offset out lse d_out causal dq dk_partial dv_partial stream
PyObject *attn_bwd_noalloc(PyObject *const *a)
{
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &out = tensor(a[4]), &lse = tensor(a[5]), &d_out = tensor(a[6]);
    const at::Tensor &dq = tensor(a[8]), &dk = tensor(a[9]), &dv = tensor(a[10]);
    const Dims m = dims(q, k, v);
    require(m.eb == 2, "bf16 only");
    for (const at::Tensor *t : {&out, &d_out, &dq}) like_q(*t, q, "out, d_out and dq must match q_seg in shape and dtype and be contiguous");
    check_lse(lse, m);
    for (const at::Tensor *t : {&dk, &dv})
        require(t->sizes() == k.sizes() && t->scalar_type() == kF32 && t->is_contiguous(), "partials must be contiguous float32 [B, l_x, H, d]");
    invoke(lss_segment_attn_bwd_noalloc, ptr(q), ptr(k), ptr(v), integer(a[3]), m.l_s, m.l_x, m.B, m.H, m.d, truth(a[7]), ptr(out), fptr(lse),
                                       ptr(d_out), ptr(dq), fptr(dk), fptr(dv), stream_of(a[11]));
    return pack({give(a[8], dq), give(a[9], dk), give(a[10], dv)});
}
// parts (list) rows_valid (list or None) out stream
PyObject *reduce_partials(PyObject *const *a)
{
    const Py_ssize_t n = PyList_GET_SIZE(a[0]);
    require(n > 0, "need at least one partial");
    const at::Tensor &p0 = tensor(PyList_GET_ITEM(a[0], 0));
    require(p0.dim() == 4, "partials must be [B, l_x, H, d]");
    std::vector<const float *> parts(n);
    std::vector<int64_t> rows;
    for (Py_ssize_t i = 0; i < n; ++i) {
        const at::Tensor &p = tensor(PyList_GET_ITEM(a[0], i));
        require(p.sizes() == p0.sizes() && plain(p, kF32), "partials must be contiguous float32 device tensors of one shape");
        parts[i] = fptr(p);
    }
    if (!none(a[1])) {
        require(PyList_GET_SIZE(a[1]) == n, "rows_valid must have one entry per partial");
        rows.resize(n);
        for (Py_ssize_t i = 0; i < n; ++i) rows[i] = integer(PyList_GET_ITEM(a[1], i));
    }
    const at::Tensor out = none(a[2]) ? at::empty_like(p0) : tensor(a[2]);
    invoke(lss_reduce_partials, parts.data(), (int)n, rows.empty() ? nullptr : rows.data(), p0.size(1), p0.size(0), p0.size(2), p0.size(3),
                              fptr(out), stream_of(a[3]));
    return give(a[2], out);
}

// ------------------------------------------------------------------------------------ projections
// x w_q w_kv seg_offset l_s H q_seg k v stream
PyObject *project_qkv(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]), &wq = tensor(a[1]), &wkv = tensor(a[2]);
    require(x.dim() == 3 && x.scalar_type() == kBf16, "x must be bf16 [B, l_x, E]");
    const int64_t B = x.size(0), l_x = x.size(1), E = x.size(2), s0 = integer(a[3]), l_s = integer(a[4]), H = integer(a[5]);
    require(H > 0 && E % H == 0, "E must be a multiple of H");
    const int64_t d = E / H;
    require(shaped(wq, {E, E}) && shaped(wkv, {E, 2 * E}), "w_q must be [E, E] and w_kv [E, 2E]");
    const at::Tensor q = output_as_is(a[6], {B, l_s, H, d}, kBf16, x), k = output_as_is(a[7], {B, l_x, H, d}, kBf16, x),
                     v = output_as_is(a[8], {B, l_x, H, d}, kBf16, x);
    require(shaped(q, {B, l_s, H, d}) && shaped(k, {B, l_x, H, d}) && shaped(v, {B, l_x, H, d}), "output shapes disagree with x, l_s and H");
    for (const at::Tensor *t : {&x, &wq, &wkv, &q, &k, &v}) require(plain(*t, kBf16), "tensors must be contiguous bf16 device tensors");
    invoke(lss_project_qkv, ptr(x), ptr(wq), ptr(wkv), s0, l_s, l_x, B, H, d, ptr(q), ptr(k), ptr(v), stream_of(a[9]));
    return pack({give(a[6], q), give(a[7], k), give(a[8], v)});
}
// dq dk_partial dv_partial w_q w_kv rows_valid dx_q dx_partial stream skip_masked_tail
PyObject *project_bwd(PyObject *const *a)
{
    const at::Tensor &dq = tensor(a[0]), &dk = tensor(a[1]), &dv = tensor(a[2]), &wq = tensor(a[3]), &wkv = tensor(a[4]);
    require(dq.dim() == 4 && dk.dim() == 4 && dk.sizes() == dv.sizes(), "dq must be [B,l_s,H,d]; partials [B,l_x,H,d]");
    const int64_t B = dq.size(0), l_s = dq.size(1), H = dq.size(2), d = dq.size(3), l_x = dk.size(1), E = H * d;
    require(shaped(dk, {B, l_x, H, d}) && shaped(wq, {E, E}) && shaped(wkv, {E, 2 * E}), "shapes disagree");
    const int64_t rows = none(a[5]) ? l_x : integer(a[5]);
    const at::Tensor dxq = output_as_is(a[6], {B, l_s, E}, kF32, dq), dxp = output_as_is(a[7], {B, l_x, E}, kF32, dq);
    require(shaped(dxq, {B, l_s, E}) && shaped(dxp, {B, l_x, E}), "output shapes disagree");
    require(plain(dq, kBf16) && plain(wq, kBf16) && plain(wkv, kBf16) && plain(dk, kF32) && plain(dv, kF32) && plain(dxq, kF32) &&
            plain(dxp, kF32), "tensors must be contiguous device tensors of the documented types");
    invoke(lss_project_bwd_ex, ptr(dq), fptr(dk), fptr(dv), ptr(wq), ptr(wkv), l_s, l_x, rows, B, H, d,
                             truth(a[9]) ? LSS_FLAG_SKIP_MASKED_TAIL : 0u, fptr(dxq), fptr(dxp), stream_of(a[8]));
    return pack({give(a[6], dxq), give(a[7], dxp)});
}
// x dq dk_partial dv_partial seg_offset rows_valid dw_q dw_kv scratch stream
PyObject *project_bwd_weight(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]), &dq = tensor(a[1]), &dk = tensor(a[2]), &dv = tensor(a[3]);
    require(x.dim() == 3 && dq.dim() == 4 && dk.dim() == 4 && dk.sizes() == dv.sizes(), "x must be [B,l_x,E]; dq [B,l_s,H,d]; partials [B,l_x,H,d]");
    const int64_t B = dq.size(0), l_s = dq.size(1), H = dq.size(2), d = dq.size(3), l_x = x.size(1), E = H * d;
    require(shaped(x, {B, l_x, E}) && shaped(dk, {B, l_x, H, d}), "shapes disagree");
    const int64_t rows = none(a[5]) ? l_x : integer(a[5]);
    require(plain(x, kBf16) && plain(dq, kBf16) && plain(dk, kF32) && plain(dv, kF32), "tensors must be contiguous device tensors of the documented types");
    const at::Tensor wq = output_as_is(a[6], {E, E}, kF32, x), wkv = output_as_is(a[7], {E, 2 * E}, kF32, x);
    require(shaped(wq, {E, E}) && shaped(wkv, {E, 2 * E}) && wq.scalar_type() == kF32 && wkv.scalar_type() == kF32,
            "dw_q must be float32 [E, E] and dw_kv float32 [E, 2E]");
    const int64_t need = (int64_t)lss_project_bwd_weight_scratch_bytes(l_s, l_x, B, H, d);
    const at::Tensor scratch = output_as_is(a[8], {need > 16 ? need : 16}, at::kByte, x);
    invoke(lss_project_bwd_weight, ptr(x), ptr(dq), fptr(dk), fptr(dv), integer(a[4]), l_s, l_x, rows, B, H, d, fptr(wq), fptr(wkv),
                                 ptr(scratch), (size_t)scratch.numel(), stream_of(a[9]));
    return pack({give(a[6], wq), give(a[7], wkv)});
}

// ------------------------------------------------------------------------------------ row operations
// tok pe_table seg_offset x stream
PyObject *embed_pe_fwd(PyObject *const *a)
{
    const at::Tensor &tok = tensor(a[0]), &pe = tensor(a[1]);
    require(tok.dim() == 3 && pe.dim() == 2 && pe.size(1) == tok.size(2), "tok must be [B, l_s, E] and pe_table [l_x, E]");
    dev(tok, kBf16, "tok"); dev(pe, kBf16, "pe_table");
    const at::Tensor x = output(a[3], tok.sizes(), kBf16, tok);
    invoke(lss_embed_pe_fwd, ptr(tok), ptr(pe), integer(a[2]), tok.size(1), pe.size(0), tok.size(0), tok.size(2), ptr(x), stream_of(a[4]));
    return give(a[3], x);
}
// dx dpe_rows stream
PyObject *embed_pe_bwd(PyObject *const *a)
{
    const at::Tensor &dx = tensor(a[0]);
    require(dx.dim() == 3, "dx must be [B, l_s, E]");
    dev(dx, kBf16, "dx");
    const at::Tensor o = output(a[1], {dx.size(1), dx.size(2)}, kF32, dx);
    invoke(lss_embed_pe_bwd, ptr(dx), dx.size(1), dx.size(0), dx.size(2), fptr(o), stream_of(a[2]));
    return give(a[1], o);
}
// x delta seg_offset p_drop seed out stream
PyObject *residual_dropout_add(PyObject *const *a)
{
    const at::Tensor &delta = tensor(a[1]);
    require(delta.dim() == 3 && (none(a[0]) || tensor(a[0]).sizes() == delta.sizes()), "delta must be [B, l_s, E] and x, if given, of the same shape");
    dev(delta, kBf16, "delta");
    if (!none(a[0])) dev(tensor(a[0]), kBf16, "x");
    const at::Tensor out = output(a[5], delta.sizes(), kBf16, delta);
    invoke(lss_residual_dropout_add, none(a[0]) ? nullptr : ptr(tensor(a[0])), ptr(delta), integer(a[2]), delta.size(1), delta.size(0),
                                   delta.size(2), real(a[3]), seed_bits(a[4]), ptr(out), stream_of(a[6]));
    return give(a[5], out);
}
struct RowsOf { int64_t rows, E; };
RowsOf rows_of(const at::Tensor &t)
{
    require(t.dim() >= 1, "a tensor of rows needs at least one dimension");
    const int64_t E = t.size(-1);
    return {E ? t.numel() / E : 0, E};
}
std::vector<int64_t> with_columns(const at::Tensor &t, int64_t n)
{
    std::vector<int64_t> s(t.sizes().begin(), t.sizes().end());
    s.back() = n;
    return s;
}
// x gamma beta eps y mean rstd stream
PyObject *layernorm_fwd(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]), &g = tensor(a[1]), &b = tensor(a[2]);
    const RowsOf m = rows_of(x);
    dev(x, kBf16, "x"); dev(g, kF32, "gamma"); dev(b, kF32, "beta");
    require(g.numel() == m.E && b.numel() == m.E, "gamma and beta must have E elements");
    const at::Tensor y = output(a[4], x.sizes(), kBf16, x), mean = output(a[5], {m.rows}, kF32, x), rstd = output(a[6], {m.rows}, kF32, x);
    invoke(lss_layernorm_fwd, ptr(x), fptr(g), fptr(b), real(a[3]), m.rows, m.E, ptr(y), fptr(mean), fptr(rstd), stream_of(a[7]));
    return pack({give(a[4], y), give(a[5], mean), give(a[6], rstd)});
}
// x gamma mean rstd dy dx dgamma dbeta scratch stream
PyObject *layernorm_bwd(PyObject *const *a)
{
    const at::Tensor &x = tensor(a[0]), &g = tensor(a[1]), &mean = tensor(a[2]), &rstd = tensor(a[3]), &dy = tensor(a[4]);
    const RowsOf m = rows_of(x);
    dev(x, kBf16, "x"); dev(dy, kBf16, "dy"); dev(g, kF32, "gamma"); dev(mean, kF32, "mean"); dev(rstd, kF32, "rstd");
    require(dy.sizes() == x.sizes() && g.numel() == m.E && mean.numel() == m.rows && rstd.numel() == m.rows, "shapes disagree");
    const at::Tensor dx = output(a[5], x.sizes(), kBf16, x), dg = output(a[6], {m.E}, kF32, x), db = output(a[7], {m.E}, kF32, x);
    const int64_t need = (int64_t)lss_layernorm_bwd_scratch_bytes(m.rows, m.E);
    const at::Tensor scratch = output_as_is(a[8], {need > 16 ? need : 16}, at::kByte, x);
    dev(scratch, at::kByte, "scratch");
    invoke(lss_layernorm_bwd, ptr(x), fptr(g), fptr(mean), fptr(rstd), ptr(dy), m.rows, m.E, ptr(dx), fptr(dg), fptr(db), ptr(scratch),
                            (size_t)scratch.numel(), stream_of(a[9]));
    return pack({give(a[5], dx), give(a[6], dg), give(a[7], db)});
}

// ------------------------------------------------------------------------------------ linear maps, GeLU
void check_linear(const at::Tensor &a, const at::Tensor &w, bool wide_side, const char *nm, const char *msg)
{
    require(w.dim() == 2 && a.dim() >= 1 && a.size(-1) == w.size(wide_side ? 1 : 0), msg);
    dev(a, kBf16, nm); dev(w, kBf16, "w");
}
// a w c stream
PyObject *linear_fwd(PyObject *const *p)
{
    const at::Tensor &a = tensor(p[0]), &w = tensor(p[1]);
    check_linear(a, w, false, "a", "a's last dimension must equal w's rows");
    const at::Tensor c = output(p[2], with_columns(a, w.size(1)), kBf16, a);
    invoke(lss_linear_fwd, ptr(a), ptr(w), rows_of(a).rows, w.size(0), w.size(1), ptr(c), stream_of(p[3]));
    return give(p[2], c);
}
// dc w da stream
PyObject *linear_bwd_input(PyObject *const *p)
{
    const at::Tensor &dc = tensor(p[0]), &w = tensor(p[1]);
    check_linear(dc, w, true, "dc", "dc's last dimension must equal w's columns");
    const at::Tensor da = output(p[2], with_columns(dc, w.size(0)), kBf16, dc);
    invoke(lss_linear_bwd_input, ptr(dc), ptr(w), rows_of(dc).rows, w.size(0), w.size(1), ptr(da), stream_of(p[3]));
    return give(p[2], da);
}
// a dc dw scratch stream
PyObject *linear_bwd_weight(PyObject *const *p)
{
    const at::Tensor &a = tensor(p[0]), &dc = tensor(p[1]);
    require(a.dim() >= 1 && a.dim() == dc.dim() && a.sizes().slice(0, a.dim() - 1) == dc.sizes().slice(0, dc.dim() - 1), "a and dc must have the same rows");
    dev(a, kBf16, "a"); dev(dc, kBf16, "dc");
    const RowsOf m = rows_of(a);
    const int64_t K = m.E, N = dc.size(-1);
    const at::Tensor dw = output(p[2], {K, N}, kF32, a);
    const int64_t need = (int64_t)lss_linear_bwd_weight_scratch_bytes(m.rows, K, N);
    const at::Tensor scratch = output_as_is(p[3], {need > 16 ? need : 16}, at::kByte, a);
    dev(scratch, at::kByte, "scratch");
    invoke(lss_linear_bwd_weight, ptr(a), ptr(dc), m.rows, K, N, fptr(dw), ptr(scratch), (size_t)scratch.numel(), stream_of(p[4]));
    return give(p[2], dw);
}
// a w u g stream
PyObject *linear_gelu_fwd(PyObject *const *p)
{
    const at::Tensor &a = tensor(p[0]), &w = tensor(p[1]);
    check_linear(a, w, false, "a", "a's last dimension must equal w's rows");
    const auto shape = with_columns(a, w.size(1));
    const at::Tensor u = output(p[2], shape, kBf16, a), g = output(p[3], shape, kBf16, a);
    invoke(lss_linear_gelu_fwd, ptr(a), ptr(w), rows_of(a).rows, w.size(0), w.size(1), ptr(u), ptr(g), stream_of(p[4]));
    return pack({give(p[2], u), give(p[3], g)});
}
// dc w u du stream
PyObject *linear_bwd_input_gelu(PyObject *const *p)
{
    const at::Tensor &dc = tensor(p[0]), &w = tensor(p[1]), &u = tensor(p[2]);
    require(w.dim() == 2 && dc.dim() >= 1 && u.dim() >= 1 && dc.size(-1) == w.size(1) && u.size(-1) == w.size(0) && rows_of(u).rows == rows_of(dc).rows, "shapes disagree");
    dev(dc, kBf16, "dc"); dev(w, kBf16, "w"); dev(u, kBf16, "u");
    const at::Tensor du = output(p[3], u.sizes(), kBf16, u);
    invoke(lss_linear_bwd_input_gelu, ptr(dc), ptr(w), ptr(u), rows_of(dc).rows, w.size(0), w.size(1), ptr(du), stream_of(p[4]));
    return give(p[3], du);
}
// u g stream
PyObject *gelu_fwd(PyObject *const *p)
{
    const at::Tensor &u = tensor(p[0]);
    dev(u, kBf16, "u");
    const at::Tensor g = output(p[1], u.sizes(), kBf16, u);
    invoke(lss_gelu_fwd, ptr(u), u.numel(), ptr(g), stream_of(p[2]));
    return give(p[1], g);
}
// u dg du stream
PyObject *gelu_bwd(PyObject *const *p)
{
    const at::Tensor &u = tensor(p[0]), &dg = tensor(p[1]);
    dev(u, kBf16, "u"); dev(dg, kBf16, "dg");
    require(dg.sizes() == u.sizes(), "u and dg must have the same shape");
    const at::Tensor du = output(p[2], u.sizes(), kBf16, u);
    invoke(lss_gelu_bwd, ptr(u), ptr(dg), u.numel(), ptr(du), stream_of(p[3]));
    return give(p[2], du);
}
PyObject *set_error_type(PyObject *const *p)
{
    Py_INCREF(p[0]);
    Py_XDECREF(g_error_type);
    g_error_type = p[0];
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *const *), int N>
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    HANDLE_TH_ERRORS
    try {
        return F(args);
    } catch (const PythonError &) {
        return nullptr;
    } catch (const ValueError &e) {
        PyErr_SetString(PyExc_ValueError, e.what());
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}
#define LSS_FN(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&call<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    LSS_FN(attn_fwd, 11), LSS_FN(attn_bwd, 16), LSS_FN(attn_bwd_noalloc, 12), LSS_FN(reduce_partials, 4), LSS_FN(project_qkv, 10),
    LSS_FN(project_bwd, 10), LSS_FN(project_bwd_weight, 10), LSS_FN(embed_pe_fwd, 5), LSS_FN(embed_pe_bwd, 3),
    LSS_FN(residual_dropout_add, 7), LSS_FN(layernorm_fwd, 8), LSS_FN(layernorm_bwd, 10), LSS_FN(linear_fwd, 4),
    LSS_FN(linear_bwd_input, 4), LSS_FN(linear_bwd_weight, 5), LSS_FN(linear_gelu_fwd, 5), LSS_FN(linear_bwd_input_gelu, 5),
    LSS_FN(gelu_fwd, 3), LSS_FN(gelu_bwd, 4), LSS_FN(set_error_type, 1), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_lss_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__lss_torch()
{
    PyObject *m = PyModule_Create(&g_module);
    // tensors cross this interface as C++ objects: lss.py refuses any torch but the one whose headers were used
    if (m && PyModule_AddStringConstant(m, "torch_version", LSS_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
