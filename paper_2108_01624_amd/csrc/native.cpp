// Argument marshalling of the calls that a training step makes many times, and the walk over a micro-batch's layers, as a
// Python extension: tensors are read through libtorch instead of through one Python attribute after the other, and the library is called
// directly.  Host time of a call, by ctypes and here: a fill, of which 2.8 us are the launch, 4.2 | 3.1 us; an update 6.8 | 4.4; both passes over the 72 dense
// layers and 24 LayerNorms of twelve blocks (14 launches) 254 | 88: small micro-batches are over on the GPU before Python has described them.
//
// Nothing is decided here that the Python functions of binding.py and step.py decide differently: whatever these functions do not
// expect - another type, a shape that does not fit, an address in place of a tensor - they leave alone (None), before the library has been
// called, and the Python function of the same name does the work or raises.  Otherwise: the library's status, and its entry point where several are called.
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include <new>
#include <string>
#include <utility>
#include <vector>

#include <torch/csrc/autograd/python_variable.h>

#include "dpclip.h"

namespace {

constexpr int OTHER = -1;

struct Arr {
    void* p = nullptr;
    int dim = 0;
    int64_t s[4] = {0, 0, 0, 0};
    int64_t numel = 0;
    int type = OTHER;  // DP_F32, DP_BF16
    bool i32 = false;
    bool same_shape(const Arr& o) const { return dim == o.dim && !memcmp(s, o.s, sizeof(s)); }
};

// A plain tensor of at most four dimensions.
bool get(PyObject* o, Arr& a) {
    if (!o || !THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.has_storage() || t.dim() > 4) return false;
        a.dim = (int)t.dim();
        for (int k = 0; k < a.dim; ++k) a.s[k] = t.size(k);
        a.numel = t.numel();
        const auto st = t.scalar_type();
        a.type = st == at::kFloat ? (int)DP_F32 : st == at::kBFloat16 ? (int)DP_BF16 : OTHER;
        a.i32 = st == at::kInt;
        a.p = t.data_ptr();
        return true;
    } catch (...) {
        return false;
    }
}
bool get_f32(PyObject* o, Arr& a) { return get(o, a) && a.type == DP_F32; }
bool get_data(PyObject* o, Arr& a) { return get(o, a) && a.type != OTHER; }

bool fits(int64_t v) { return v >= 0 && v <= INT32_MAX; }
bool fits(const Arr& a) {
    for (int k = 0; k < a.dim; ++k)
        if (!fits(a.s[k])) return false;
    return true;
}

// Python number -> C number; false (no error pending) for anything else.
bool num(PyObject* o, int64_t& v) {
    if (!PyLong_Check(o)) return false;
    v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) return PyErr_Clear(), false;
    return true;
}
bool num(PyObject* o, int& v) {
    int64_t x;
    if (!num(o, x) || x < INT32_MIN || x > INT32_MAX) return false;
    v = (int)x;
    return true;
}
bool num(PyObject* o, uint64_t& v) {
    if (!PyLong_Check(o)) return false;
    v = PyLong_AsUnsignedLongLong(o);
    if (v == (uint64_t)-1 && PyErr_Occurred()) return PyErr_Clear(), false;
    return true;
}
bool num(PyObject* o, float& v) {
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
    const double d = PyFloat_AsDouble(o);
    if (d == -1.0 && PyErr_Occurred()) return PyErr_Clear(), false;
    v = (float)d;
    return true;
}
// A flag: True, False, 1 or 0 (whatever else has a truth value need not be a number to Python's int()).
bool truth(PyObject* o, bool& v) {
    int64_t x;
    if (!num(o, x) || (x != 0 && x != 1)) return false;
    v = x != 0;
    return true;
}
bool context(PyObject* o, dp_ctx*& ctx) {
    if (!PyLong_Check(o)) return false;
    ctx = (dp_ctx*)PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) return PyErr_Clear(), false;
    return ctx != nullptr;
}

template <typename F>
int call(F f) {
    int st;
    Py_BEGIN_ALLOW_THREADS st = (int)f();
    Py_END_ALLOW_THREADS return st;
}

#define LEAVE Py_RETURN_NONE
#define NEED(cond) \
    if (!(cond)) LEAVE
#define STATUS(expr) return PyLong_FromLong(call([&] { return (expr); }))
#define ARGS(count) NEED(n == (count))

typedef PyObject* const* Args;

PyObject* zero_f32(PyObject*, Args a, Py_ssize_t n) {  // ctx, p, n
    dp_ctx* ctx;
    Arr p;
    uint64_t len;
    ARGS(3);
    NEED(context(a[0], ctx) && get_f32(a[1], p));
    if (a[2] == Py_None) len = (uint64_t)p.numel;
    else NEED(num(a[2], len));
    STATUS(dp_zero_f32(ctx, (float*)p.p, len));
}

PyObject* sqnorms_dense(PyObject*, Args a, Py_ssize_t n) {  // ctx, A, G, has_bias, path, sqnorms
    dp_ctx* ctx;
    Arr A, G, sq;
    bool bias;
    int path;
    ARGS(6);
    NEED(context(a[0], ctx) && get_data(a[1], A) && get_data(a[2], G) && A.dim == 3 && G.dim >= 1 && fits(A) && fits(G) && truth(a[3], bias) && num(a[4], path) && get_f32(a[5], sq));
    STATUS(dp_sqnorms_dense(ctx, A.p, G.p, (dp_dtype)A.type, (int)A.s[0], (int)A.s[1], (int)A.s[2], (int)G.s[G.dim - 1], bias, (dp_path)path, (float*)sq.p));
}

PyObject* clip_accumulate_dense(PyObject*, Args a, Py_ssize_t n) {  // ctx, A, G, C, sqnorms, sum_W, sum_b
    dp_ctx* ctx;
    Arr A, G, sq, W, b;
    float C;
    ARGS(7);
    NEED(context(a[0], ctx) && get_data(a[1], A) && get_data(a[2], G) && A.dim == 3 && G.dim >= 1 && fits(A) && fits(G) && num(a[3], C) && get_f32(a[4], sq) && get_f32(a[5], W));
    if (a[6] != Py_None) NEED(get_f32(a[6], b));
    STATUS(dp_clip_accumulate_dense(ctx, A.p, G.p, (dp_dtype)A.type, (int)A.s[0], (int)A.s[1], (int)A.s[2], (int)G.s[G.dim - 1], C, (float*)sq.p, (float*)W.p, (float*)b.p));
}

// A list of tensors.
bool list_of(PyObject* o, std::vector<Arr>& out) {
    if (!PyList_CheckExact(o)) return false;
    out.resize((size_t)PyList_GET_SIZE(o));
    for (size_t k = 0; k < out.size(); ++k)
        if (!get(PyList_GET_ITEM(o, k), out[k])) return false;
    return true;
}
std::vector<const void*> addresses(const std::vector<Arr>& v) {
    std::vector<const void*> p;
    p.reserve(v.size());
    for (const Arr& a : v) p.push_back(a.p);
    return p;
}
// Layers of one shape (B, T, d_in), (B, T, d_out) and type.
bool same_layers(const std::vector<Arr>& A, const std::vector<Arr>& G) {
    if (A.empty() || A.size() != G.size()) return false;
    for (size_t k = 0; k < A.size(); ++k)
        if (A[k].dim != 3 || G[k].dim != 3 || A[k].type == OTHER || A[k].type != A[0].type || G[k].type != A[0].type || !A[k].same_shape(A[0]) ||
            !G[k].same_shape(G[0]) || G[k].s[0] != A[0].s[0] || G[k].s[1] != A[0].s[1] || !fits(A[k]) || !fits(G[k]))
            return false;
    return true;
}

PyObject* sqnorms_dense_batched(PyObject*, Args a, Py_ssize_t n) {  // ctx, As, Gs, has_bias, path, sqnorms
    dp_ctx* ctx;
    std::vector<Arr> A, G;
    Arr sq;
    bool bias;
    int path;
    ARGS(6);
    NEED(context(a[0], ctx) && list_of(a[1], A) && list_of(a[2], G) && same_layers(A, G) && truth(a[3], bias) && num(a[4], path) && get_f32(a[5], sq));
    const auto pa = addresses(A), pg = addresses(G);
    STATUS(dp_sqnorms_dense_batched(ctx, (int)A.size(), pa.data(), pg.data(), (dp_dtype)A[0].type, (int)A[0].s[0], (int)A[0].s[1], (int)A[0].s[2], (int)G[0].s[2], bias,
                                    (dp_path)path, (float*)sq.p));
}

PyObject* clip_accumulate_dense_batched(PyObject*, Args a, Py_ssize_t n) {  // ctx, As, Gs, C, sqnorms, sum_Ws, sum_bs
    dp_ctx* ctx;
    std::vector<Arr> A, G, W;
    Arr sq;
    float C;
    ARGS(7);
    NEED(context(a[0], ctx) && list_of(a[1], A) && list_of(a[2], G) && same_layers(A, G) && num(a[3], C) && get_f32(a[4], sq) && list_of(a[5], W) && W.size() == A.size());
    std::vector<float*> pw, pb;
    for (const Arr& w : W) {
        NEED(w.type == DP_F32);
        pw.push_back((float*)w.p);
    }
    if (a[6] != Py_None) {
        NEED(PyList_CheckExact(a[6]) && (size_t)PyList_GET_SIZE(a[6]) == A.size());
        for (size_t k = 0; k < A.size(); ++k) {
            PyObject* o = PyList_GET_ITEM(a[6], k);
            Arr b;
            NEED(o == Py_None || get_f32(o, b));
            pb.push_back((float*)b.p);
        }
    }
    const auto pa = addresses(A), pg = addresses(G);
    STATUS(dp_clip_accumulate_dense_batched(ctx, (int)A.size(), pa.data(), pg.data(), (dp_dtype)A[0].type, (int)A[0].s[0], (int)A[0].s[1], (int)A[0].s[2], (int)G[0].s[2], C,
                                            (float*)sq.p, pw.data(), pb.empty() ? nullptr : pb.data()));
}

PyObject* sqnorms_embedding(PyObject*, Args a, Py_ssize_t n) {  // ctx, ids, G, V, distinct, sqnorms
    dp_ctx* ctx;
    Arr ids, G, sq;
    int V;
    bool distinct;
    ARGS(6);
    NEED(context(a[0], ctx) && get(a[1], ids) && ids.i32 && get_data(a[2], G) && G.dim == 3 && fits(G) && num(a[3], V) && truth(a[4], distinct) && get_f32(a[5], sq));
    STATUS(dp_sqnorms_embedding(ctx, (int32_t*)ids.p, G.p, (dp_dtype)G.type, (int)G.s[0], (int)G.s[1], (int)G.s[2], V, distinct, (float*)sq.p));
}

PyObject* clip_accumulate_embedding(PyObject*, Args a, Py_ssize_t n) {  // ctx, ids, G, V, C, sqnorms, sum_E
    dp_ctx* ctx;
    Arr ids, G, sq, E;
    int V;
    float C;
    ARGS(7);
    NEED(context(a[0], ctx) && get(a[1], ids) && ids.i32 && get_data(a[2], G) && G.dim == 3 && fits(G) && num(a[3], V) && num(a[4], C) && get_f32(a[5], sq) && get_f32(a[6], E));
    STATUS(dp_clip_accumulate_embedding(ctx, (int32_t*)ids.p, G.p, (dp_dtype)G.type, (int)G.s[0], (int)G.s[1], (int)G.s[2], V, C, (float*)sq.p, (float*)E.p));
}

struct Tied {
    Arr ids, dY, H, dL;
    bool get_all(PyObject* i, PyObject* y, PyObject* h, PyObject* l) {
        return get(i, ids) && ids.i32 && get_data(y, dY) && get_data(h, H) && get_data(l, dL) && dY.dim == 3 && dL.dim == 3 && H.dim == 3 && ids.dim == 2 &&
               H.type == dY.type && dL.type == dY.type && ids.s[0] == dY.s[0] && ids.s[1] == dY.s[1] && H.s[0] == dY.s[0] && H.s[1] == dL.s[1] && H.s[2] == dY.s[2] &&
               dL.s[0] == dY.s[0] && fits(dY) && fits(H) && fits(dL);
    }
    int norms(dp_ctx* ctx, float* sq) const {
        return dp_sqnorms_tied_embedding(ctx, (int32_t*)ids.p, dY.p, H.p, dL.p, (dp_dtype)dY.type, (int)dY.s[0], (int)dY.s[1], (int)dL.s[1], (int)dY.s[2], (int)dL.s[2], sq);
    }
    int sums(dp_ctx* ctx, float C, const float* sq, float* E) const {
        return dp_clip_accumulate_tied_embedding(ctx, (int32_t*)ids.p, dY.p, H.p, dL.p, (dp_dtype)dY.type, (int)dY.s[0], (int)dY.s[1], (int)dL.s[1], (int)dY.s[2],
                                                 (int)dL.s[2], C, sq, E);
    }
};

PyObject* sqnorms_tied_embedding(PyObject*, Args a, Py_ssize_t n) {  // ctx, ids, dY, H, dL, sqnorms
    dp_ctx* ctx;
    Tied t;
    Arr sq;
    ARGS(6);
    NEED(context(a[0], ctx) && t.get_all(a[1], a[2], a[3], a[4]) && get_f32(a[5], sq));
    STATUS(t.norms(ctx, (float*)sq.p));
}

PyObject* clip_accumulate_tied_embedding(PyObject*, Args a, Py_ssize_t n) {  // ctx, ids, dY, H, dL, C, sqnorms, sum_E
    dp_ctx* ctx;
    Tied t;
    Arr sq, E;
    float C;
    ARGS(8);
    NEED(context(a[0], ctx) && t.get_all(a[1], a[2], a[3], a[4]) && num(a[5], C) && get_f32(a[6], sq) && get_f32(a[7], E) && E.numel == t.dL.s[2] * t.dY.s[2]);
    STATUS(t.sums(ctx, C, (float*)sq.p, (float*)E.p));
}

// ctx, params, m, v, sum, n, elem_offset, sigma, C, seed, step, batch_size, lr, beta1, beta2, eps, weight_decay, zero_sum[, snr_sq]
PyObject* noise_adamw(PyObject*, Args a, Py_ssize_t n) {
    dp_ctx* ctx;
    Arr p, m, v, s, q;
    uint64_t len, off, seed, step, batch;
    float sigma, C, lr, b1, b2, eps, wd;
    bool zero;
    NEED(n == 18 || n == 19);
    NEED(context(a[0], ctx) && get_f32(a[1], p) && get_f32(a[2], m) && get_f32(a[3], v) && get_f32(a[4], s));
    if (a[5] == Py_None) len = (uint64_t)p.numel;
    else NEED(num(a[5], len));
    NEED(num(a[6], off) && num(a[7], sigma) && num(a[8], C) && num(a[9], seed) && num(a[10], step) && num(a[11], batch) && num(a[12], lr) && num(a[13], b1) &&
         num(a[14], b2) && num(a[15], eps) && num(a[16], wd) && truth(a[17], zero));
    if (n == 18)
        STATUS(dp_noise_adamw(ctx, (float*)p.p, (float*)m.p, (float*)v.p, (float*)s.p, len, off, sigma, C, seed, step, batch, lr, b1, b2, eps, wd, zero));
    NEED(get_f32(a[18], q) && q.numel >= 2);
    STATUS(dp_noise_adamw_snr(ctx, (float*)p.p, (float*)m.p, (float*)v.p, (float*)s.p, len, off, sigma, C, seed, step, batch, lr, b1, b2, eps, wd, zero, (float*)q.p));
}

// ---------------------------------------------------------------------------------------------------------------------
// A micro-batch's layers
// ---------------------------------------------------------------------------------------------------------------------
PyObject *s_kind, *s_A, *s_G, *s_X, *s_H, *s_dL, *s_ids, *s_V, *s_distinct, *s_has_bias, *s_dense, *s_layernorm, *s_tied;

enum Kind { DENSE, LAYERNORM, TIED, EMBEDDING };

struct Layer {
    Kind kind;
    Arr A, G;  // LAYERNORM: A is X; EMBEDDING: A is ids
    Tied tied;
    bool flag = false;  // DENSE: has_bias; EMBEDDING: distinct
    int V = 0;
};

bool parse(PyObject* list, std::vector<Layer>& out) {
    if (!PyList_CheckExact(list) || PyList_GET_SIZE(list) == 0) return false;
    out.resize((size_t)PyList_GET_SIZE(list));
    for (size_t k = 0; k < out.size(); ++k) {
        PyObject* d = PyList_GET_ITEM(list, k);
        if (!PyDict_CheckExact(d)) return false;
        auto item = [&](PyObject* key) { return PyDict_GetItemWithError(d, key); };
        PyObject *kind = item(s_kind), *o;
        if (!kind || !PyUnicode_CheckExact(kind)) return PyErr_Clear(), false;
        Layer& l = out[k];
        l.kind = PyUnicode_Compare(kind, s_dense) == 0 ? DENSE : PyUnicode_Compare(kind, s_layernorm) == 0 ? LAYERNORM : PyUnicode_Compare(kind, s_tied) == 0 ? TIED : EMBEDDING;
        bool ok;
        if (l.kind == DENSE) {
            ok = get_data(item(s_A), l.A) && get_data(item(s_G), l.G) && l.A.type == l.G.type && l.A.dim == 3 && l.G.dim == 3 && l.A.s[0] == l.G.s[0] && l.A.s[1] == l.G.s[1] &&
                 fits(l.A) && fits(l.G) && (o = item(s_has_bias)) && truth(o, l.flag);
        } else if (l.kind == LAYERNORM) {
            ok = get_data(item(s_X), l.A) && get_data(item(s_G), l.G) && l.A.type == l.G.type && l.A.dim == 3 && l.A.same_shape(l.G) && fits(l.A);
        } else if (l.kind == TIED) {
            ok = l.tied.get_all(item(s_ids), item(s_G), item(s_H), item(s_dL));
            l.G = l.tied.dY;
        } else {
            ok = get(item(s_ids), l.A) && l.A.i32 && get_data(item(s_G), l.G) && l.G.dim == 3 && fits(l.G) && (o = item(s_V)) && num(o, l.V) && (o = item(s_distinct)) && truth(o, l.flag);
        }
        if (!ok) return PyErr_Clear(), false;
        if (l.G.s[0] != out[0].G.s[0] || (l.kind == EMBEDDING && (l.A.dim != 2 || l.A.s[0] != l.G.s[0] || l.A.s[1] != l.G.s[1]))) return false;
    }
    return true;
}

// Whether there are norms, and room for kept LayerNorm gradients, for as many examples as the layers (all the same) have.
bool holds(const std::vector<Layer>& layers, const Arr& sqnorms, int64_t max_batch) { return layers[0].G.s[0] <= max_batch && layers[0].G.s[0] <= sqnorms.numel; }

// The groups of same-shaped layers of a kind, in order of their first layer.
std::vector<std::vector<int>> group(const std::vector<Layer>& layers, Kind kind, bool by_bias) {
    std::vector<std::vector<int>> out;
    for (int k = 0; k < (int)layers.size(); ++k) {
        const Layer& l = layers[k];
        if (l.kind != kind) continue;
        std::vector<int>* to = nullptr;
        for (auto& g : out) {
            const Layer& h = layers[g[0]];
            if (h.A.type == l.A.type && h.A.same_shape(l.A) && h.G.same_shape(l.G) && (!by_bias || h.flag == l.flag)) to = &g;
        }
        if (!to) {
            out.emplace_back();
            to = &out.back();
        }
        to->push_back(k);
    }
    return out;
}

// Identifies the micro-batch whose LayerNorm gradients the keep buffers hold: batch size and input buffers.
std::string token(const std::vector<Layer>& layers, int64_t nB) {
    std::string t((const char*)&nB, sizeof(nB));
    for (const Layer& l : layers)
        if (l.kind == LAYERNORM) {
            t.append((const char*)&l.A.p, sizeof(void*));
            t.append((const char*)&l.G.p, sizeof(void*));
        }
    return t;
}

// The keep buffers of the LayerNorms `sel`, through `make(k, d)` where there is none of that size yet.
bool keeps(PyObject* dict, PyObject* make, const std::vector<Layer>& layers, const std::vector<int>& sel, int64_t max_batch, std::vector<float*>& out) {
    for (int k : sel) {
        const int64_t d = layers[k].A.s[2], need = max_batch * 2 * d;
        PyObject* key = PyLong_FromLong(k);
        if (!key) return false;
        PyObject* o = PyDict_GetItemWithError(dict, key);
        Py_DECREF(key);
        Arr a;
        if (o && get_f32(o, a) && a.numel >= need) {
            out.push_back((float*)a.p);
            continue;
        }
        if (!make) return PyErr_Clear(), false;
        PyObject* made = PyObject_CallFunction(make, "iL", k, (long long)d);  // (the dictionary holds it)
        const bool ok = made && get_f32(made, a) && a.numel >= layers[k].A.s[0] * 2 * d;
        Py_XDECREF(made);
        if (!ok) return PyErr_Clear(), false;
        out.push_back((float*)a.p);
    }
    return true;
}

PyObject* failed(int st, const char* where) { return Py_BuildValue("is", st, where); }
#define CALL(name, ...)                                            \
    do {                                                           \
        const int st__ = call([&] { return (name)(__VA_ARGS__); }); \
        if (st__ != DP_OK) return failed(st__, #name);             \
    } while (0)

// ctx, layers, sqnorms, ln_keep, keep_buffer, max_batch -> None: left alone; (status, entry point): an error; bytes: done, and the
// micro-batch whose LayerNorm gradients were kept (empty: none were)
PyObject* pass1(PyObject*, Args a, Py_ssize_t n) {
    dp_ctx* ctx;
    std::vector<Layer> layers;
    Arr sq;
    int64_t max_batch;
    ARGS(6);
    NEED(context(a[0], ctx) && get_f32(a[2], sq) && PyDict_CheckExact(a[3]) && num(a[5], max_batch) && parse(a[1], layers) && holds(layers, sq, max_batch));
    float* const out = (float*)sq.p;
    const auto norms = group(layers, LAYERNORM, false), dense = group(layers, DENSE, true);
    std::vector<std::vector<float*>> kept(norms.size());
    bool all_kept = !norms.empty();
    for (size_t g = 0; g < norms.size(); ++g) {
        if (layers[norms[g][0]].A.s[2] % 4) all_kept = false;
        else NEED(keeps(a[3], a[4], layers, norms[g], max_batch, kept[g]));
    }
    for (const Layer& l : layers) {
        if (l.kind == TIED) {
            const int st = call([&] { return l.tied.norms(ctx, out); });
            if (st != DP_OK) return failed(st, "dp_sqnorms_tied_embedding");
        } else if (l.kind == EMBEDDING) {
            CALL(dp_sqnorms_embedding, ctx, (int32_t*)l.A.p, l.G.p, (dp_dtype)l.G.type, (int)l.G.s[0], (int)l.G.s[1], (int)l.G.s[2], l.V, l.flag, out);
        }
    }
    std::vector<const void*> pa, pg;
    auto take = [&](const std::vector<int>& sel) {
        pa.clear();
        pg.clear();
        for (int k : sel) {
            pa.push_back(layers[k].A.p);
            pg.push_back(layers[k].G.p);
        }
    };
    for (size_t g = 0; g < norms.size(); ++g) {
        const Arr& x = layers[norms[g][0]].A;
        take(norms[g]);
        if (!kept[g].empty())
            CALL(dp_sqnorms_layernorm_keep, ctx, (int)pa.size(), pa.data(), pg.data(), (dp_dtype)x.type, (int)x.s[0], (int)x.s[1], (int)x.s[2], out, kept[g].data());
        else
            CALL(dp_sqnorms_layernorm_batched, ctx, (int)pa.size(), pa.data(), pg.data(), (dp_dtype)x.type, (int)x.s[0], (int)x.s[1], (int)x.s[2], out);
    }
    for (const auto& sel : dense) {
        const Layer& f = layers[sel[0]];
        // layers reading the very same input tensor (query / key / value projections) share its Gram matrix
        std::vector<std::vector<int>> by_input;
        for (int k : sel) {
            std::vector<int>* to = nullptr;
            for (auto& g : by_input)
                if (layers[g[0]].A.p == layers[k].A.p) to = &g;
            if (!to) {
                by_input.emplace_back();
                to = &by_input.back();
            }
            to->push_back(k);
        }
        for (size_t width = 3; width >= 2; --width) {
            std::vector<const void*> in, gs;
            for (const auto& g : by_input)
                if (g.size() == width) {
                    in.push_back(layers[g[0]].A.p);
                    for (int k : g) gs.push_back(layers[k].G.p);
                }
            if (!in.empty())
                CALL(dp_sqnorms_dense_shared, ctx, (int)in.size(), in.data(), (int)width, gs.data(), (dp_dtype)f.A.type, (int)f.A.s[0], (int)f.A.s[1], (int)f.A.s[2],
                     (int)f.G.s[2], f.flag, out);
        }
        std::vector<int> rest;
        for (int k : sel)
            for (const auto& g : by_input)
                if (layers[g[0]].A.p == layers[k].A.p && g.size() != 2 && g.size() != 3) rest.push_back(k);
        if (rest.empty()) continue;
        take(rest);
        CALL(dp_sqnorms_dense_batched, ctx, (int)pa.size(), pa.data(), pg.data(), (dp_dtype)f.A.type, (int)f.A.s[0], (int)f.A.s[1], (int)f.A.s[2], (int)f.G.s[2], f.flag,
             DP_PATH_AUTO, out);
    }
    const std::string t = all_kept ? token(layers, layers[0].G.s[0]) : std::string();
    return PyBytes_FromStringAndSize(t.data(), (Py_ssize_t)t.size());
}

// ctx, layers, C, sqnorms, S, [[(byte offset, elements) of each tensor of a layer's parameters]], ln_keep, kept_for, max_batch
// -> None, (status, entry point) or True
PyObject* pass2(PyObject*, Args a, Py_ssize_t n) {
    dp_ctx* ctx;
    std::vector<Layer> layers;
    Arr sq, S;
    float C;
    int64_t max_batch;
    ARGS(9);
    NEED(context(a[0], ctx) && num(a[2], C) && get_f32(a[3], sq) && get_f32(a[4], S) && PyList_CheckExact(a[5]) && PyDict_CheckExact(a[6]) && num(a[8], max_batch) && parse(a[1], layers) && holds(layers, sq, max_batch));
    const float* const norms = (float*)sq.p;
    // where the layers' sums lie
    NEED(PyList_GET_SIZE(a[5]) >= (Py_ssize_t)layers.size());
    std::vector<std::pair<float*, float*>> at(layers.size());
    for (size_t k = 0; k < layers.size(); ++k) {
        PyObject* t = PyList_GET_ITEM(a[5], k);
        NEED(PyList_CheckExact(t));
        const Layer& l = layers[k];
        const Py_ssize_t need = l.kind == LAYERNORM || (l.kind == DENSE && l.flag) ? 2 : 1;
        NEED(PyList_GET_SIZE(t) >= need);
        int64_t off[2] = {0, 0}, elems[2] = {0, 0};
        for (Py_ssize_t j = 0; j < need; ++j) {
            PyObject* e = PyList_GET_ITEM(t, j);
            NEED(PyTuple_CheckExact(e) && PyTuple_GET_SIZE(e) == 2 && num(PyTuple_GET_ITEM(e, 0), off[j]) && num(PyTuple_GET_ITEM(e, 1), elems[j]));
        }
        at[k] = {(float*)((char*)S.p + off[0]), need == 2 ? (float*)((char*)S.p + off[1]) : nullptr};
        if (l.kind == TIED) NEED(elems[0] == l.tied.dL.s[2] * l.tied.dY.s[2]);
        if (l.kind == EMBEDDING && l.flag) NEED(elems[0] >= l.G.s[1] * l.G.s[2]);
    }
    const auto lns = group(layers, LAYERNORM, false), dense = group(layers, DENSE, false);
    bool kept = !lns.empty() && PyBytes_CheckExact(a[7]) && PyBytes_GET_SIZE(a[7]) > 0;
    if (kept) {
        const std::string t = token(layers, layers[0].G.s[0]);
        kept = (size_t)PyBytes_GET_SIZE(a[7]) == t.size() && !memcmp(PyBytes_AS_STRING(a[7]), t.data(), t.size());
    }
    NEED(kept || a[7] == Py_None || PyBytes_CheckExact(a[7]));
    std::vector<std::vector<float*>> bufs(lns.size());
    for (size_t g = 0; kept && g < lns.size(); ++g) NEED(keeps(a[6], nullptr, layers, lns[g], max_batch, bufs[g]));
    for (size_t k = 0; k < layers.size(); ++k) {
        const Layer& l = layers[k];
        if (l.kind == TIED) {
            const int st = call([&] { return l.tied.sums(ctx, C, norms, at[k].first); });
            if (st != DP_OK) return failed(st, "dp_clip_accumulate_tied_embedding");
        } else if (l.kind == EMBEDDING && l.flag) {  // position ids: no sort needed
            CALL(dp_clip_accumulate_positions, ctx, l.G.p, (dp_dtype)l.G.type, (int)l.G.s[0], (int)l.G.s[1], (int)l.G.s[2], C, norms, at[k].first);
        } else if (l.kind == EMBEDDING) {
            CALL(dp_clip_accumulate_embedding, ctx, (int32_t*)l.A.p, l.G.p, (dp_dtype)l.G.type, (int)l.G.s[0], (int)l.G.s[1], (int)l.G.s[2], l.V, C, norms, at[k].first);
        }
    }
    std::vector<const void*> pa, pg;
    std::vector<float*> p1, p2;
    auto take = [&](const std::vector<int>& sel) {
        pa.clear(), pg.clear(), p1.clear(), p2.clear();
        for (int k : sel) {
            pa.push_back(layers[k].A.p);
            pg.push_back(layers[k].G.p);
            p1.push_back(at[k].first);
            p2.push_back(at[k].second);
        }
    };
    for (size_t g = 0; g < lns.size(); ++g) {
        const Arr& x = layers[lns[g][0]].A;
        take(lns[g]);
        if (kept)
            CALL(dp_clip_accumulate_layernorm_kept, ctx, (int)p1.size(), bufs[g].data(), (int)x.s[0], (int)x.s[2], C, norms, p1.data(), p2.data());
        else
            CALL(dp_clip_accumulate_layernorm_batched, ctx, (int)p1.size(), pa.data(), pg.data(), (dp_dtype)x.type, (int)x.s[0], (int)x.s[1], (int)x.s[2], C, norms,
                 p1.data(), p2.data());
    }
    for (const auto& sel : dense) {
        const Layer& f = layers[sel[0]];
        take(sel);
        CALL(dp_clip_accumulate_dense_batched, ctx, (int)p1.size(), pa.data(), pg.data(), (dp_dtype)f.A.type, (int)f.A.s[0], (int)f.A.s[1], (int)f.A.s[2], (int)f.G.s[2], C,
             norms, p1.data(), p2.data());
    }
    Py_RETURN_TRUE;
}

// No exception leaves the extension.
template <PyObject* (*F)(PyObject*, Args, Py_ssize_t)>
PyObject* guarded(PyObject* self, Args a, Py_ssize_t n) {
    try {
        return F(self, a, n);
    } catch (const std::bad_alloc&) {
        return PyErr_NoMemory();
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unexpected exception in the native call layer");
        return nullptr;
    }
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))guarded<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(zero_f32), METHOD(sqnorms_dense), METHOD(clip_accumulate_dense), METHOD(sqnorms_dense_batched), METHOD(clip_accumulate_dense_batched),
                         METHOD(sqnorms_embedding), METHOD(clip_accumulate_embedding), METHOD(sqnorms_tied_embedding), METHOD(clip_accumulate_tied_embedding),
                         METHOD(noise_adamw), METHOD(pass1), METHOD(pass2), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    const std::pair<PyObject**, const char*> names[] = {{&s_kind, "kind"}, {&s_A, "A"}, {&s_G, "G"}, {&s_X, "X"}, {&s_H, "H"}, {&s_dL, "dL"}, {&s_ids, "ids"}, {&s_V, "V"},
                                                        {&s_distinct, "distinct"}, {&s_has_bias, "has_bias"}, {&s_dense, "dense"}, {&s_layernorm, "layernorm"},
                                                        {&s_tied, "tied_embedding"}};
    for (const auto& x : names)
        if (!(*x.first = PyUnicode_InternFromString(x.second))) return nullptr;
    return PyModule_Create(&module);
}
