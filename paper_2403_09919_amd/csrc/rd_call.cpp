// rd_call: the tensor-facing half of the Python binding as a CPython extension (host code only).
//
// A decoding step makes a few dozen library calls of a few microseconds of GPU work each, so the host's share of a
// call decides how fast a program that launches from Python can go.  Checking 8 to 16 tensors (device, layout, type,
// shape), reading their addresses and looking up the stream from Python took 9 to 12 us per call, the launch included;
// here the tensors are inspected through torch's C++ interface and rd.h is called directly (3 to 4 us, nearly all of it
// the HIP launch).  The functions of binding.py keep their arguments, defaults and errors: they allocate what the caller
// left out, call the function here of the same name with everything in place, and turn a status code into RdError.
// The GIL is released around the library call, which can block when the GPU's queue is full.
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <initializer_list>
#include <limits.h>
#include <string>
#include "rd.h"

namespace {

struct PyError {};                      // a Python exception is set

constexpr int kAnyType = -1;

std::string shape_text(const int64_t *s, size_t n)
{
    std::string t = "(";
    for (size_t i = 0; i < n; ++i) t += (i ? ", " : "") + std::to_string(s[i]);
    return t + (n == 1 ? ",)" : ")");
}

std::string type_text(at::ScalarType t)
{
    std::string out = "?";
    if (PyObject *s = PyObject_Str(reinterpret_cast<PyObject *>(torch::getTHPDtype(t)))) {
        if (const char *c = PyUnicode_AsUTF8(s)) out = c;
        Py_DECREF(s);
    }
    return out;
}

[[noreturn]] void bad(const std::string &text)
{
    PyErr_SetString(PyExc_ValueError, text.c_str());
    throw PyError();
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_AttributeError, "%s: '%s' object is not a tensor", name, Py_TYPE(o)->tp_name);
        throw PyError();
    }
    return THPVariable_Unpack(o);
}

// Device address of a dense tensor on the GPU with this element type (kAnyType: any) and, where given, shape;
// None is a null pointer.
void *ptr(PyObject *o, int type, const std::initializer_list<int64_t> *shape, const char *name)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    if (!t.is_cuda()) bad(std::string(name) + " must live in device memory");
    if (!t.is_contiguous()) bad(std::string(name) + " must be contiguous");
    if (type != kAnyType && (int)t.scalar_type() != type)
        bad(std::string(name) + " must be " + type_text((at::ScalarType)type) + ", got " + type_text(t.scalar_type()));
    if (shape) {
        const auto got = t.sizes();
        if (got.size() != shape->size() || !std::equal(got.begin(), got.end(), shape->begin()))
            bad(std::string(name) + " must have shape " + shape_text(shape->begin(), shape->size()) + ", got " + shape_text(got.data(), got.size()));
    }
    return t.data_ptr();
}

void *dev(PyObject *o, int type, std::initializer_list<int64_t> shape, const char *name) { return ptr(o, type, &shape, name); }
const int32_t *i32(PyObject *o, std::initializer_list<int64_t> shape, const char *name)
{
    return static_cast<const int32_t *>(ptr(o, (int)at::kInt, &shape, name));
}
int32_t *i32_out(PyObject *o, std::initializer_list<int64_t> shape, const char *name) { return const_cast<int32_t *>(i32(o, shape, name)); }
float *f32(PyObject *o, std::initializer_list<int64_t> shape, const char *name)
{
    return static_cast<float *>(ptr(o, (int)at::kFloat, &shape, name));
}
uint64_t *bits(PyObject *o, std::initializer_list<int64_t> shape, const char *name)
{
    return static_cast<uint64_t *>(ptr(o, (int)at::kLong, &shape, name));
}

template <size_t R>
std::array<int, R> sizes(const at::Tensor &t, const char *name)
{
    std::array<int, R> s;
    if (t.dim() != (int64_t)R) bad(std::string(name) + " must have " + std::to_string(R) + " dimensions, got " + std::to_string(t.dim()));
    for (size_t i = 0; i < R; ++i) s[i] = (int)t.size((int64_t)i);
    return s;
}

struct Scratch { void *p; size_t bytes; };
Scratch scratch(PyObject *o)
{
    void *p = ptr(o, (int)at::kByte, nullptr, "workspace");
    return {p, p ? (size_t)THPVariable_Unpack(o).numel() : 0};
}

int integer(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyError();
    if (v != (long)(int)v) { PyErr_SetString(PyExc_OverflowError, "value does not fit a C int"); throw PyError(); }
    return (int)v;
}
// What int(o) accepts, moved into a C int's range where it lies outside (a context bound above every capacity is one)
int bound(PyObject *o)
{
    PyObject *n = PyNumber_Long(o);
    if (!n) throw PyError();
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(n, &over);
    Py_DECREF(n);
    if (over > 0 || v > INT_MAX) return INT_MAX;
    return over < 0 || v < INT_MIN ? INT_MIN : (int)v;
}
// What float(o) accepts
float real(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject *f = PyNumber_Float(o);
    if (!f) throw PyError();
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}

rd_dtype dtype_of(const at::Tensor &t)
{
    switch (t.scalar_type()) {
    case at::kFloat: return RD_F32;
    case at::kBFloat16: return RD_BF16;
    case at::kHalf: return RD_F16;
    default: bad("unsupported element type " + type_text(t.scalar_type()) + " (float32, bfloat16 or float16)");
    }
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs `body` (which returns an rd_status) with the GIL released.
template <typename F>
PyObject *status(F body)
{
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = body();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(code);
}

typedef PyObject *const *Args;
template <PyObject *(*Fn)(Args), int Count>
PyObject *entry(PyObject *, Args a, Py_ssize_t n)
{
    if (n != Count) return PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", Count, n);
    try {
        return Fn(a);
    } catch (const PyError &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// beams, ctx_len, prefix_tree, packed_tokens, n_packed, unpack_index, parent, position_ids, tree_mask, tree_mask_bits
PyObject *dedup(Args a)
{
    const auto [B, W, L] = sizes<3>(tensor(a[0], "beams"), "beams");
    const int64_t N = (int64_t)W * L;
    const int32_t *beams = i32(a[0], {B, W, L}, "beams"), *ctx = i32(a[1], {B}, "ctx_len");
    int32_t *prefix = i32_out(a[2], {B, W, L}, "prefix_tree"), *packed = i32_out(a[3], {B, N}, "packed_tokens");
    int32_t *n_packed = i32_out(a[4], {B}, "n_packed"), *unpack = i32_out(a[5], {B, W, L}, "unpack_index");
    int32_t *parent = i32_out(a[6], {B, N}, "parent"), *pos = i32_out(a[7], {B, N}, "position_ids");
    uint8_t *mask = static_cast<uint8_t *>(dev(a[8], (int)at::kByte, {B, N, N}, "tree_mask"));
    uint64_t *mb = bits(a[9], {B, N, (N + 63) / 64}, "tree_mask_bits");
    void *s = stream();
    return status([&, B = B, W = W, L = L] { return rd_dedup(beams, ctx, B, W, L, prefix, packed, n_packed, unpack, parent, pos, mask, mb, s); });
}

// What the attention entry points share: q, ctx_len, k_new, v_new, n_packed, tree_mask_bits, out, workspace.
struct Attn {
    int B, H, N, D;
    rd_dtype dt;
    int type;
    const void *q, *k_new, *v_new;
    const int32_t *ctx_len, *n_packed;
    const uint64_t *mask;
    void *out;
    Scratch ws;
    Attn(PyObject *q_, PyObject *ctx_, PyObject *k_, PyObject *v_, PyObject *n_, PyObject *m_, PyObject *out_, PyObject *ws_)
    {
        const at::Tensor &t = tensor(q_, "q");
        const auto s = sizes<4>(t, "q");
        B = s[0]; H = s[1]; N = s[2]; D = s[3];
        dt = dtype_of(t);
        type = (int)t.scalar_type();
        q = dev(q_, type, {B, H, N, D}, "q");
        ctx_len = i32(ctx_, {B}, "ctx_len");
        k_new = dev(k_, type, {B, H, N, D}, "k_new");
        v_new = dev(v_, type, {B, H, N, D}, "v_new");
        n_packed = i32(n_, {B}, "n_packed");
        mask = bits(m_, {B, N, (N + 63) / 64}, "tree_mask_bits");
        out = dev(out_, type, {B, H, N, D}, "out");
        ws = scratch(ws_);
    }
    const void *cache(PyObject *o, int Cmax, const char *name) const
    {
        return Cmax > 0 ? dev(o, type, {B, H, Cmax, D}, name) : nullptr;
    }
};

int capacity(PyObject *k_cache)
{
    const at::Tensor &t = tensor(k_cache, "k_cache");
    if (t.dim() < 3) bad("k_cache must have 4 dimensions, got " + std::to_string(t.dim()));     // (the whole shape is checked where keys are held)
    return (int)t.size(2);
}

// q, k_cache, v_cache, ctx_len, k_new, v_new, n_packed, tree_mask_bits, scale, out, workspace, ctx_bound or None
PyObject *tree_attn(Args a)
{
    const Attn t(a[0], a[3], a[4], a[5], a[6], a[7], a[9], a[10]);
    const int Cmax = capacity(a[1]);
    const void *kc = t.cache(a[1], Cmax, "k_cache"), *vc = t.cache(a[2], Cmax, "v_cache");
    const float scale = real(a[8]);
    void *s = stream();
    if (a[11] == Py_None)
        return status([&] { return rd_tree_attn(t.q, kc, vc, t.ctx_len, t.k_new, t.v_new, t.n_packed, t.mask, t.B, t.H, t.N, t.D, Cmax, t.dt, scale, t.out, t.ws.p, t.ws.bytes, s); });
    const int most = bound(a[11]);
    return status([&] { return rd_tree_attn_bounded(t.q, kc, vc, t.ctx_len, t.k_new, t.v_new, t.n_packed, t.mask, t.B, t.H, t.N, t.D, Cmax, most, t.dt, scale, t.out, t.ws.p, t.ws.bytes, s); });
}

// q, k_cache, v_cache, ctx_len, k_new, v_new, n_packed, tree_mask_bits, position_ids, cos_tab, sin_tab, scale, out,
// k_new_rot, workspace
PyObject *tree_attn_rope(Args a)
{
    const Attn t(a[0], a[3], a[4], a[5], a[6], a[7], a[12], a[14]);
    const int Cmax = capacity(a[1]);
    const void *kc = t.cache(a[1], Cmax, "k_cache"), *vc = t.cache(a[2], Cmax, "v_cache");
    const int32_t *pos = i32(a[8], {t.B, t.N}, "position_ids");
    const int max_pos = (int)tensor(a[9], "cos_tab").size(0);
    const float *ct = f32(a[9], {max_pos, t.D / 2}, "cos_tab"), *st = f32(a[10], {max_pos, t.D / 2}, "sin_tab");
    const float scale = real(a[11]);
    void *rot = dev(a[13], t.type, {t.B, t.H, t.N, t.D}, "k_new_rot");
    void *s = stream();
    return status([&] { return rd_tree_attn_rope(t.q, kc, vc, t.ctx_len, t.k_new, t.v_new, t.n_packed, t.mask, pos, ct, st, max_pos, t.B, t.H, t.N, t.D, Cmax, t.dt, scale, t.out, rot, t.ws.p, t.ws.bytes, s); });
}

// q, k_pages, v_pages, block_table, ctx_len, k_new, v_new, n_packed, tree_mask_bits, scale, out, workspace
PyObject *tree_attn_paged(Args a)
{
    const Attn t(a[0], a[4], a[5], a[6], a[7], a[8], a[10], a[11]);
    const auto [n_pages, Hp, page, Dp] = sizes<4>(tensor(a[1], "k_pages"), "k_pages");
    const auto [rows, max_pages] = sizes<2>(tensor(a[3], "block_table"), "block_table");
    (void)Hp; (void)Dp; (void)rows;
    const void *kp = dev(a[1], t.type, {n_pages, t.H, page, t.D}, "k_pages"), *vp = dev(a[2], t.type, {n_pages, t.H, page, t.D}, "v_pages");
    const int32_t *table = i32(a[3], {t.B, max_pages}, "block_table");
    const float scale = real(a[9]);
    void *s = stream();
    return status([&, n_pages = n_pages, page = page, max_pages = max_pages] {
        return rd_tree_attn_paged(t.q, kp, vp, table, page, max_pages, n_pages, t.ctx_len, t.k_new, t.v_new, t.n_packed, t.mask, t.B, t.H, t.N, t.D, t.dt, scale, t.out, t.ws.p, t.ws.bytes, s);
    });
}

// logits, beams, unpack_index, n_packed, root_token, argmax, n_accept, best_beam, best_len, next_token, accepted_idx,
// then workspace unless the call is rd_accept_static
template <bool STATIC>
PyObject *accept(Args a)
{
    const auto [B, W, L] = sizes<3>(tensor(a[1], "beams"), "beams");
    const int64_t N = (int64_t)W * L;
    const int V = sizes<3>(tensor(a[0], "logits"), "logits")[2];
    const float *logits = f32(a[0], {B, N, V}, "logits");
    const int32_t *beams = i32(a[1], {B, W, L}, "beams"), *unpack = i32(a[2], {B, W, L}, "unpack_index");
    const int32_t *n_packed = i32(a[3], {B}, "n_packed"), *root = i32(a[4], {B}, "root_token");
    int32_t *am = i32_out(a[5], {B, N}, "argmax"), *na = i32_out(a[6], {B, W}, "n_accept"), *bb = i32_out(a[7], {B}, "best_beam");
    int32_t *bl = i32_out(a[8], {B}, "best_len"), *nt = i32_out(a[9], {B}, "next_token"), *ai = i32_out(a[10], {B, L}, "accepted_idx");
    void *s = stream();
    if constexpr (STATIC) {
        return status([&, B = B, W = W, L = L] { return rd_accept_static(logits, beams, unpack, n_packed, root, B, W, L, V, am, na, bb, bl, nt, ai, s); });
    } else {
        const Scratch ws = scratch(a[11]);
        return status([&, B = B, W = W, L = L] { return rd_accept(logits, beams, unpack, n_packed, root, B, W, L, V, am, na, bb, bl, nt, ai, ws.p, ws.bytes, s); });
    }
}

// logits, draft_logits, step_row, beams, unpack_index, n_packed, root_token, u_accept, u_next, temperature, n_accept,
// best_beam, best_len, next_token, accepted_idx, workspace
PyObject *accept_sample(Args a)
{
    const auto [B, W, L] = sizes<3>(tensor(a[3], "beams"), "beams");
    const int64_t N = (int64_t)W * L;
    const int V = sizes<3>(tensor(a[0], "logits"), "logits")[2];
    const float *logits = f32(a[0], {B, N, V}, "logits");
    const bool record = a[2] != Py_None;
    const int rows = record ? sizes<3>(tensor(a[1], "draft_logits"), "draft_logits")[1] : 0;
    const float *draft = record ? f32(a[1], {L - 1, rows, V}, "draft_logits") : f32(a[1], {B, N, V}, "draft_logits");
    const int32_t *step_row = i32(a[2], {B, W, L - 1}, "step_row");
    const int32_t *beams = i32(a[3], {B, W, L}, "beams"), *unpack = i32(a[4], {B, W, L}, "unpack_index");
    const int32_t *n_packed = i32(a[5], {B}, "n_packed"), *root = i32(a[6], {B}, "root_token");
    const float *ua = f32(a[7], {B, N}, "u_accept"), *un = f32(a[8], {B}, "u_next");
    const float temperature = real(a[9]);
    int32_t *na = i32_out(a[10], {B, W}, "n_accept"), *bb = i32_out(a[11], {B}, "best_beam"), *bl = i32_out(a[12], {B}, "best_len");
    int32_t *nt = i32_out(a[13], {B}, "next_token"), *ai = i32_out(a[14], {B, L}, "accepted_idx");
    const Scratch ws = scratch(a[15]);
    void *s = stream();
    return status([&, B = B, W = W, L = L] { return rd_accept_sample(logits, draft, step_row, rows, beams, unpack, n_packed, root, ua, un, temperature, B, W, L, V, na, bb, bl, nt, ai, ws.p, ws.bytes, s); });
}

// k_new, v_new, accepted_idx, best_len, ctx_len, k_cache, v_cache, ctx_len_out, n_committed, hidden, hidden_last
PyObject *commit(Args a)
{
    const at::Tensor &k = tensor(a[0], "k_new");
    const auto [B, H, N, D] = sizes<4>(k, "k_new");
    const int type = (int)k.scalar_type();
    const rd_dtype dt = dtype_of(k);
    const int Cmax = capacity(a[5]), L = sizes<2>(tensor(a[2], "accepted_idx"), "accepted_idx")[1];
    const void *kn = dev(a[0], type, {B, H, N, D}, "k_new"), *vn = dev(a[1], type, {B, H, N, D}, "v_new");
    const int32_t *ai = i32(a[2], {B, L}, "accepted_idx"), *bl = i32(a[3], {B}, "best_len"), *ctx = i32(a[4], {B}, "ctx_len");
    void *kc = dev(a[5], type, {B, H, Cmax, D}, "k_cache"), *vc = dev(a[6], type, {B, H, Cmax, D}, "v_cache");
    int32_t *next = i32_out(a[7], {B}, "ctx_len_out"), *nc = i32_out(a[8], {B}, "n_committed");
    int Dh = 0;
    const void *hidden = nullptr;
    void *last = nullptr;
    if (a[9] != Py_None) {
        Dh = sizes<3>(tensor(a[9], "hidden"), "hidden")[2];
        hidden = dev(a[9], type, {B, N, Dh}, "hidden");
        last = dev(a[10], type, {B, Dh}, "hidden_last");
    }
    void *s = stream();
    return status([&, B = B, H = H, N = N, D = D] { return rd_commit(kn, vn, ai, bl, ctx, B, H, N, D, Cmax, L, dt, kc, vc, next, nc, hidden, Dh, last, s); });
}

// k_new, v_new, accepted_idx, best_len, ctx_len, k_pages, v_pages, block_table, ctx_len_out, n_committed
PyObject *commit_paged(Args a)
{
    const at::Tensor &k = tensor(a[0], "k_new");
    const auto [B, H, N, D] = sizes<4>(k, "k_new");
    const int type = (int)k.scalar_type();
    const rd_dtype dt = dtype_of(k);
    const auto [n_pages, Hp, page, Dp] = sizes<4>(tensor(a[5], "k_pages"), "k_pages");
    const int max_pages = sizes<2>(tensor(a[7], "block_table"), "block_table")[1];
    const int L = sizes<2>(tensor(a[2], "accepted_idx"), "accepted_idx")[1];
    (void)Hp; (void)Dp;
    const void *kn = dev(a[0], type, {B, H, N, D}, "k_new"), *vn = dev(a[1], type, {B, H, N, D}, "v_new");
    const int32_t *ai = i32(a[2], {B, L}, "accepted_idx"), *bl = i32(a[3], {B}, "best_len"), *ctx = i32(a[4], {B}, "ctx_len");
    void *kp = dev(a[5], type, {n_pages, H, page, D}, "k_pages"), *vp = dev(a[6], type, {n_pages, H, page, D}, "v_pages");
    const int32_t *table = i32(a[7], {B, max_pages}, "block_table");
    int32_t *next = i32_out(a[8], {B}, "ctx_len_out"), *nc = i32_out(a[9], {B}, "n_committed");
    void *s = stream();
    return status([&, B = B, H = H, N = N, D = D, n_pages = n_pages, page = page] {
        return rd_commit_paged(kn, vn, ai, bl, ctx, B, H, N, D, L, dt, kp, vp, table, page, max_pages, n_pages, next, nc, nullptr, 0, nullptr, s);
    });
}

// q or None, k_new or None, position_ids, n_packed, cos_tab, sin_tab
PyObject *rope(Args a)
{
    const at::Tensor &ref = tensor(a[0] != Py_None ? a[0] : a[1], "q");
    const auto [B, H, N, D] = sizes<4>(ref, "q");
    const int type = (int)ref.scalar_type();
    const rd_dtype dt = dtype_of(ref);
    const int max_pos = (int)tensor(a[4], "cos_tab").size(0);
    void *q = dev(a[0], type, {B, H, N, D}, "q"), *k = dev(a[1], type, {B, H, N, D}, "k_new");
    const int32_t *pos = i32(a[2], {B, N}, "position_ids"), *n_packed = i32(a[3], {B}, "n_packed");
    const float *ct = f32(a[4], {max_pos, D / 2}, "cos_tab"), *st = f32(a[5], {max_pos, D / 2}, "sin_tab");
    void *s = stream();
    return status([&, B = B, H = H, N = N, D = D] { return rd_rope(q, k, pos, n_packed, ct, st, max_pos, B, H, N, D, dt, s); });
}

PyObject *item(PyObject *dict, const char *key)
{
    PyObject *o = PyDict_GetItemString(dict, key);             // borrowed
    if (!o) { PyErr_SetString(PyExc_KeyError, key); throw PyError(); }
    return o;
}

// params (a dict), h, last_token, W, L, beams, beam_logp, step_logits, step_row, workspace
PyObject *draft(Args a)
{
    PyObject *params = a[0];
    if (!PyDict_Check(params)) { PyErr_SetString(PyExc_TypeError, "params must be a dict"); throw PyError(); }
    const at::Tensor &emb = tensor(item(params, "emb"), "emb");
    const int type = (int)emb.scalar_type();
    if (type != (int)at::kBFloat16 && type != (int)at::kHalf)
        bad("draft model weights must be bfloat16 or float16, got " + type_text(emb.scalar_type()));
    const auto [V, Dm] = sizes<2>(emb, "emb");
    PyObject *mark = PyDict_GetItemString(params, "tiled");     // matrices packed by rd_draft_pack: flat tensors
    const int tiled = mark ? PyObject_IsTrue(mark) : 0;
    if (tiled < 0) throw PyError();
    const int K = tiled ? integer(item(params, "n_mlp")) : (int)tensor(item(params, "mlp_w"), "mlp_w").size(0);
    const int64_t G = 2 * (int64_t)Dm;
    const int W = integer(a[3]), L = integer(a[4]);
    const at::Tensor &h = tensor(a[1], "h");
    if (h.dim() < 1) bad("h must have 2 dimensions, got 0");
    const int64_t B = h.size(0), T = L > 1 ? L - 1 : 0;
    auto square = [&](const char *name, int64_t n, int64_t k) -> const void * {
        PyObject *o = item(params, name);
        return tiled ? dev(o, type, {(int64_t)rd_draft_packed_elems((int)n, (int)k)}, name) : dev(o, type, {n, k}, name);
    };
    rd_draft_params p = {};
    p.emb = dev(item(params, "emb"), type, {V, Dm}, "emb");
    p.rnn_u = square("rnn_u", Dm, Dm);
    p.rnn_w = square("rnn_w", Dm, Dm);
    p.rnn_b = f32(item(params, "rnn_b"), {Dm}, "rnn_b");
    if (K) {
        PyObject *o = item(params, "mlp_w");
        p.mlp_w = tiled ? dev(o, type, {(int64_t)K * (int64_t)rd_draft_packed_elems((int)G, (int)G)}, "mlp_w") : dev(o, type, {K, G, G}, "mlp_w");
        p.mlp_b = f32(item(params, "mlp_b"), {K, G}, "mlp_b");
    }
    p.head_w = square("head_w", V, G);
    p.n_mlp = K; p.Dm = Dm; p.V = V; p.dtype = type == (int)at::kBFloat16 ? RD_BF16 : RD_F16; p.tiled = tiled;
    const void *hp = dev(a[1], type, {B, Dm}, "h");
    const int32_t *lt = i32(a[2], {B}, "last_token");
    int32_t *beams = i32_out(a[5], {B, W, L}, "beams");
    float *logp = f32(a[6], {B, W}, "beam_logp"), *sl = f32(a[7], {T, B * W, V}, "step_logits");
    int32_t *sr = i32_out(a[8], {B, W, T}, "step_row");
    const Scratch ws = scratch(a[9]);
    void *s = stream();
    return status([&] { return rd_draft(&p, hp, lt, (int)B, W, L, beams, logp, sl, sr, ws.p, ws.bytes, s); });
}

#define RD_ENTRY(name, fn, count) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<fn, count>)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    RD_ENTRY("dedup", dedup, 10),
    RD_ENTRY("tree_attn", tree_attn, 12),
    RD_ENTRY("tree_attn_rope", tree_attn_rope, 15),
    RD_ENTRY("tree_attn_paged", tree_attn_paged, 12),
    RD_ENTRY("accept", accept<false>, 12),
    RD_ENTRY("accept_static", accept<true>, 11),
    RD_ENTRY("accept_sample", accept_sample, 16),
    RD_ENTRY("commit", commit, 11),
    RD_ENTRY("commit_paged", commit_paged, 10),
    RD_ENTRY("rope", rope, 6),
    RD_ENTRY("draft", draft, 10),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_rdcall", "Tensor checks and calls of librd for binding.py.", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rdcall(void) { return PyModule_Create(&kModule); }
