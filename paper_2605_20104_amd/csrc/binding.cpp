// Native half of the Python binding: tensor -> pointer marshalling, output allocation and the
// call into libgraft.so, one C function per entry point.
//
// A decoding round of a small model is bound by the host: the kernels of a call take 4 to 10 us.
// The same marshalling through ctypes cost 8 to 10 us per call (17 foreign-function arguments
// converted one by one, data_ptr() and is_contiguous() as Python method calls, torch.empty() at
// 1.5 us each, the current stream looked up through Python); here a call costs what its launches
// cost.  The library stays a plain C ABI without any knowledge of PyTorch: this file resolves its
// functions from the path the Python side hands to bind().
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "graft.h"

namespace {

// ---- the library's entry points ------------------------------------------------------------
#define GRAFT_ENTRY_POINTS(X)                                                                       \
    X(graft_retrieve) X(graft_build_tree_mask) X(graft_tree_attn_workspace_bytes) X(graft_tree_attn) \
    X(graft_accept_workspace_bytes) X(graft_accept) X(graft_accept_noalloc) X(graft_matrix_retrieve) \
    X(graft_matrix_update_workspace_bytes) X(graft_matrix_update) X(graft_kv_compact) X(graft_prune_select) \
    X(graft_last_hip_error)
struct Library {
#define X(name) decltype(&::name) name = nullptr;
    GRAFT_ENTRY_POINTS(X)
#undef X
};
Library lib;
PyObject* graft_error = nullptr;         // the GraftError class
PyObject *s_page, *s_token, *s_head, *s_cuda_stream;

// Thrown after a Python error has been set.
struct PythonError {};

// ---- arguments -----------------------------------------------------------------------------
const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    return THPVariable_Unpack(o);
}

template <class T> T* ptr(const at::Tensor& t) {
    if (!t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "tensors cross the C ABI as dense row-major arrays");
        throw PythonError();
    }
    return static_cast<T*>(t.data_ptr());
}
template <class T> T* ptr(PyObject* o) { return o == Py_None ? nullptr : ptr<T>(tensor(o)); }

int32_t to_i32(PyObject* o) {
    const unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (v == static_cast<unsigned long>(-1) && PyErr_Occurred()) throw PythonError();
    return static_cast<int32_t>(v);
}
int64_t to_i64(PyObject* o) {
    PyObject* i = PyNumber_Long(o);
    if (!i) throw PythonError();
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw PythonError();
    return v;
}

void sizes2(const at::Tensor& t, int32_t& a, int32_t& b) {
    if (t.dim() != 2) {
        PyErr_Format(PyExc_ValueError, "expected a tensor of 2 dimensions, got %d", static_cast<int>(t.dim()));
        throw PythonError();
    }
    a = static_cast<int32_t>(t.size(0));
    b = static_cast<int32_t>(t.size(1));
}
int32_t size_at(const at::Tensor& t, int64_t dim) {
    if (t.dim() <= dim) {
        PyErr_SetString(PyExc_IndexError, "a tensor argument has too few dimensions");
        throw PythonError();
    }
    return static_cast<int32_t>(t.size(dim));
}

// A reference held for as long as the object is looked at.
struct Ref {
    PyObject* o;
    explicit Ref(PyObject* owned) : o(owned) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref&) = delete;
    operator PyObject*() const { return o; }
};

// KeyError if the key is missing.  The reference is held: a mapping other than a dict may make its
// values on the fly.
Ref item(PyObject* dict, PyObject* key) {
    PyObject* v;
    if (PyDict_CheckExact(dict)) {
        v = PyDict_GetItemWithError(dict, key);
        Py_XINCREF(v);
        if (!v && !PyErr_Occurred()) PyErr_SetObject(PyExc_KeyError, key);
    } else v = PyObject_GetItem(dict, key);
    if (!v) throw PythonError();
    return Ref(v);
}

struct Strides { int64_t page, token, head; };
Strides strides_of(PyObject* d) {
    return {to_i64(item(d, s_page)), to_i64(item(d, s_token)), to_i64(item(d, s_head))};
}

at::Tensor empty_bytes(size_t n, const at::Device& dev);

// The stream a call launches on: the given one (an object with a cuda_stream attribute, or the handle
// itself), else the current stream of the current device.
class LaunchStream {
public:
    LaunchStream(PyObject* given, const at::Device& dev) : dev_(dev), given_(given != Py_None) {
        if (!given_) {
            handle_ = c10::hip::getCurrentHIPStream().stream();
            return;
        }
        PyObject* h = PyObject_GetAttr(given, s_cuda_stream);
        if (!h) {
            PyErr_Clear();
            handle_ = reinterpret_cast<void*>(to_i64(given));
            return;
        }
        PyObject* i = PyNumber_Long(h);
        Py_DECREF(h);
        if (!i) throw PythonError();
        handle_ = PyLong_AsVoidPtr(i);
        Py_DECREF(i);
    }
    void* handle() const { return handle_; }
    // Scratch memory of the call.  It is given back when the call returns, with its kernels still to run, so
    // it has to belong to the stream they run on: the allocator hands a block out again in the order of the
    // stream it was taken for.  Taken for the current stream, two calls on two other streams get the
    // same block, and so does whatever is allocated next.
    at::Tensor scratch(size_t n) const {
        if (!given_ || !dev_.is_cuda()) return empty_bytes(n, dev_);
        struct Restore {
            c10::hip::HIPStream before;
            ~Restore() { c10::hip::setCurrentHIPStream(before); }
        } restore{c10::hip::getCurrentHIPStream(dev_.index())};
        c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(static_cast<hipStream_t>(handle_), dev_.index()));
        return empty_bytes(n, dev_);
    }

private:
    at::Device dev_;
    bool given_;
    void* handle_;
};

// ---- results -------------------------------------------------------------------------------
at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Device& dev) {
    if (dev.is_cuda()) return at::Tensor(at::detail::empty_cuda(shape, type, dev, std::nullopt));
    return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
}
at::Tensor empty_i32(at::IntArrayRef shape, const at::Device& dev) { return empty(shape, at::kInt, dev); }
at::Tensor empty_bytes(size_t n, const at::Device& dev) { return empty({static_cast<int64_t>(n)}, at::kByte, dev); }

// A dict of result tensors: either the caller's (no allocation) or a new one.
class Outputs {
public:
    Outputs(PyObject* given, const at::Device& dev) : dev_(dev) {
        if (given != Py_None) {
            Py_INCREF(given);
            dict_ = given;
        } else {
            dict_ = PyDict_New();
            fresh_ = true;
            if (!dict_) throw PythonError();
        }
    }
    ~Outputs() { Py_XDECREF(dict_); }
    Outputs(const Outputs&) = delete;
    template <class T = int32_t> T* get(PyObject* key, at::IntArrayRef shape, at::ScalarType type = at::kInt) {
        if (!fresh_) return ptr<T>(item(dict_, key));
        at::Tensor t = empty(shape, type, dev_);
        T* p = static_cast<T*>(t.data_ptr());
        put(key, THPVariable_Wrap(std::move(t)));
        return p;
    }
    void put(PyObject* key, PyObject* value) {                     // steals value
        const int bad = value ? PyObject_SetItem(dict_, key, value) : -1;
        Py_XDECREF(value);
        if (bad) throw PythonError();
    }
    bool fresh() const { return fresh_; }
    PyObject* release() {
        PyObject* d = dict_;
        dict_ = nullptr;
        return d;
    }

private:
    PyObject* dict_ = nullptr;
    bool fresh_ = false;
    at::Device dev_;
};

// GraftError on a return code other than GRAFT_OK.
void check(const char* fn, int32_t rc) {
    if (rc == GRAFT_OK) return;
    PyObject* e = PyObject_CallFunction(graft_error, "sii", fn, rc, lib.graft_last_hip_error());
    if (e) {
        PyErr_SetObject(graft_error, e);
        Py_DECREF(e);
    }
    throw PythonError();
}

// The library call, without the GIL (a launch waits when the stream's queue is full).
template <class F> int32_t unlocked(F&& f) {
    PyThreadState* st = PyEval_SaveThread();
    const int32_t rc = f();
    PyEval_RestoreThread(st);
    return rc;
}

void need_args(Py_ssize_t got, Py_ssize_t want) {
    if (!graft_error) {
        PyErr_SetString(PyExc_RuntimeError, "the library has not been bound");
        throw PythonError();
    }
    if (got != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
        throw PythonError();
    }
}

// ---- one function per entry point; arguments are those of the Python function, in order, all given
#define GRAFT_PY(name, n)                                                                 \
    PyObject* name##_body(PyObject* const* a);                                             \
    PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n_args) {                     \
        try {                                                                              \
            need_args(n_args, n);                                                          \
            return name##_body(a);                                                         \
        } catch (const PythonError&) {                                                     \
            return nullptr;                                                                \
        } catch (...) { /* as torch raises it: out of memory is torch.OutOfMemoryError */  \
            torch::translate_exception_to_python(std::current_exception());                \
            return nullptr;                                                                \
        }                                                                                  \
    }                                                                                      \
    PyObject* name##_body(PyObject* const* a)
#define GRAFT_KEY(name) static PyObject* const k_##name = PyUnicode_InternFromString(#name)

// ctx, ctx_len, n_min, n_max, C, m, tail, tail_len, out, stream
GRAFT_PY(py_retrieve, 10) {
    GRAFT_KEY(chain_tok); GRAFT_KEY(chain_len); GRAFT_KEY(chain_pos); GRAFT_KEY(chain_match); GRAFT_KEY(n_hits); GRAFT_KEY(status);
    const at::Tensor& ctx = tensor(a[0]);
    int32_t B, L_max;
    sizes2(ctx, B, L_max);
    const int32_t n_min = to_i32(a[2]), n_max = to_i32(a[3]), C = to_i32(a[4]), m = to_i32(a[5]);
    Outputs out(a[8], ctx.device());
    int32_t* tok = out.get(k_chain_tok, {B, C, m});
    int32_t* len = out.get(k_chain_len, {B, C});
    int32_t* pos = out.get(k_chain_pos, {B, C});
    int32_t* match = out.get(k_chain_match, {B, C});
    int32_t* hits = out.get(k_n_hits, {B});
    int32_t* status = out.get(k_status, {B});
    const int32_t tail_max = a[6] == Py_None ? 0 : size_at(tensor(a[6]), 1);
    const int32_t *c = ptr<int32_t>(ctx), *cl = ptr<int32_t>(a[1]), *t = ptr<int32_t>(a[6]), *tl = ptr<int32_t>(a[7]);
    void* s = LaunchStream(a[9], ctx.device()).handle();
    check("graft_retrieve", unlocked([&] {
        return lib.graft_retrieve(c, cl, B, L_max, t, tl, tail_max, n_min, n_max, C, m, tok, len, pos, match, hits, status, s);
    }));
    return out.release();
}

// parent, n_nodes, prefix_len, n_leaf_max, depth_cap, out, stream
GRAFT_PY(py_build_tree_mask, 7) {
    GRAFT_KEY(mask); GRAFT_KEY(pos); GRAFT_KEY(depth); GRAFT_KEY(paths); GRAFT_KEY(status);
    const at::Tensor& parent = tensor(a[0]);
    int32_t B, K;
    sizes2(parent, B, K);
    const int32_t n_leaf_max = to_i32(a[3]), depth_cap = to_i32(a[4]);
    Outputs out(a[5], parent.device());
    uint64_t* mask = out.get<uint64_t>(k_mask, {B, K, GRAFT_MASK_WORDS}, at::kLong);
    int32_t* pos = out.get(k_pos, {B, K});
    int32_t* depth = out.get(k_depth, {B, K});
    int32_t* paths = nullptr;
    if (!out.fresh() || n_leaf_max > 0) paths = out.get(k_paths, {B, n_leaf_max, depth_cap + 1});
    else {
        Py_INCREF(Py_None);
        out.put(k_paths, Py_None);
    }
    int32_t* status = out.get(k_status, {B});
    const int32_t *p = ptr<int32_t>(parent), *n = ptr<int32_t>(a[1]), *pl = ptr<int32_t>(a[2]);
    void* s = LaunchStream(a[6], parent.device()).handle();
    check("graft_build_tree_mask", unlocked([&] {
        return lib.graft_build_tree_mask(p, n, pl, B, K, mask, pos, depth, paths, n_leaf_max, depth_cap, status, s);
    }));
    return out.release();
}

// q, k_cache, v_cache, strides, block_table, prefix_len, n_nodes, mask, Hkv, scale, out, workspace, stream
GRAFT_PY(py_tree_attn, 13) {
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &table = tensor(a[4]);
    if (q.dim() != 4) {
        PyErr_Format(PyExc_ValueError, "expected a query tensor of 4 dimensions, got %d", static_cast<int>(q.dim()));
        throw PythonError();
    }
    const at::ScalarType type = q.scalar_type();
    if ((type != at::kFloat && type != at::kBFloat16) || k.scalar_type() != type || v.scalar_type() != type) {
        PyErr_SetString(PyExc_AssertionError, "queries, keys and values are all float32 or all bfloat16");
        throw PythonError();
    }
    const int32_t dtype = type == at::kFloat ? GRAFT_F32 : GRAFT_BF16;
    const int32_t B = static_cast<int32_t>(q.size(0)), K = static_cast<int32_t>(q.size(1)),
                  Hq = static_cast<int32_t>(q.size(2)), D = static_cast<int32_t>(q.size(3));
    const int32_t max_pages = size_at(table, 1), Hkv = to_i32(a[8]);
    const double scale = PyFloat_AsDouble(a[9]);
    if (scale == -1.0 && PyErr_Occurred()) throw PythonError();
    const Strides st = strides_of(a[3]);
    const LaunchStream stream(a[12], q.device());
    at::Tensor new_out, new_ws;
    void* out;
    if (a[10] == Py_None) {
        new_out = empty(q.sizes(), type, q.device());
        out = new_out.data_ptr();
    } else out = ptr<void>(a[10]);
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (a[11] == Py_None) {
        ws_bytes = lib.graft_tree_attn_workspace_bytes(B, K, Hq, Hkv, D, max_pages, dtype);
        if (ws_bytes > 0) {
            new_ws = stream.scratch(ws_bytes);
            ws = new_ws.data_ptr();
        }
    } else {
        const at::Tensor& w = tensor(a[11]);
        ws = ptr<void>(w);
        ws_bytes = static_cast<size_t>(w.numel());
    }
    const void *qp = ptr<void>(q), *kp = ptr<void>(k), *vp = ptr<void>(v);
    const int32_t *tp = ptr<int32_t>(table), *pl = ptr<int32_t>(a[5]), *n = ptr<int32_t>(a[6]);
    const uint64_t* mask = ptr<uint64_t>(a[7]);
    void* s = stream.handle();
    check("graft_tree_attn", unlocked([&] {
        return lib.graft_tree_attn(qp, kp, vp, st.page, st.token, st.head, tp, max_pages, pl, n, mask, B, K, Hq, Hkv, D,
                                   GRAFT_PAGE_SIZE, static_cast<float>(scale), dtype, out, ws, ws_bytes, s);
    }));
    if (new_out.defined()) return THPVariable_Wrap(std::move(new_out));
    Py_INCREF(a[10]);
    return a[10];
}

// parent, tokens, n_nodes, depth_cap, target_ids, logits, out, workspace, stream
GRAFT_PY(py_accept, 9) {
    GRAFT_KEY(accept_len); GRAFT_KEY(best_node); GRAFT_KEY(path); GRAFT_KEY(out_tokens); GRAFT_KEY(status); GRAFT_KEY(target_ids);
    const at::Tensor& parent = tensor(a[0]);
    int32_t B, K, V = 0;
    sizes2(parent, B, K);
    const int32_t depth_cap = to_i32(a[3]);
    const at::Device dev = parent.device();
    const LaunchStream stream(a[8], dev);
    const float* logits = nullptr;
    int32_t* ids;
    PyObject* ids_obj = a[4];
    at::Tensor new_ws;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (a[5] != Py_None) {
        const at::Tensor& lg = tensor(a[5]);
        V = size_at(lg, 2);
        logits = ptr<float>(lg);
        at::Tensor t = empty_i32({B, K}, dev);
        ids = static_cast<int32_t*>(t.data_ptr());
        ids_obj = THPVariable_Wrap(std::move(t));
        if (!ids_obj) throw PythonError();
    } else {
        ids = ptr<int32_t>(a[4]);
        Py_INCREF(ids_obj);
    }
    const Ref ids_held(ids_obj);
    Outputs out(a[6], dev);
    int32_t* len = out.get(k_accept_len, {B});
    int32_t* best = out.get(k_best_node, {B});
    int32_t* path = out.get(k_path, {B, depth_cap + 1});
    int32_t* toks = out.get(k_out_tokens, {B, depth_cap + 1});
    int32_t* status = out.get(k_status, {B});
    Py_INCREF(ids_obj);
    out.put(k_target_ids, ids_obj);
    if (a[7] != Py_None) {
        const at::Tensor& w = tensor(a[7]);
        ws = ptr<void>(w);
        ws_bytes = static_cast<size_t>(w.numel());
    } else if (logits) {
        ws_bytes = lib.graft_accept_workspace_bytes(B, K, V);
        new_ws = stream.scratch(ws_bytes);
        ws = new_ws.data_ptr();
    }
    const int32_t *p = ptr<int32_t>(parent), *tk = ptr<int32_t>(a[1]), *n = ptr<int32_t>(a[2]);
    void* s = stream.handle();
    check("graft_accept", unlocked([&] {
        return lib.graft_accept(p, tk, n, logits, V, ids, B, K, depth_cap, len, best, path, toks, status, ws, ws_bytes, s);
    }));
    return out.release();
}

// parent, tokens, n_nodes, depth_cap, out, target_ids, logits, stream
GRAFT_PY(py_accept_noalloc, 8) {
    GRAFT_KEY(accept_len); GRAFT_KEY(best_node); GRAFT_KEY(path); GRAFT_KEY(out_tokens); GRAFT_KEY(status);
    const at::Tensor& parent = tensor(a[0]);
    int32_t B, K;
    sizes2(parent, B, K);
    const int32_t depth_cap = to_i32(a[3]), V = a[6] == Py_None ? 0 : size_at(tensor(a[6]), 2);
    const float* logits = ptr<float>(a[6]);
    int32_t* ids = ptr<int32_t>(a[5]);
    int32_t *len = ptr<int32_t>(item(a[4], k_accept_len)), *best = ptr<int32_t>(item(a[4], k_best_node)),
            *path = ptr<int32_t>(item(a[4], k_path)), *toks = ptr<int32_t>(item(a[4], k_out_tokens)),
            *status = ptr<int32_t>(item(a[4], k_status));
    const int32_t *p = ptr<int32_t>(parent), *tk = ptr<int32_t>(a[1]), *n = ptr<int32_t>(a[2]);
    void* s = LaunchStream(a[7], parent.device()).handle();
    check("graft_accept_noalloc", unlocked([&] {
        return lib.graft_accept_noalloc(p, tk, n, logits, V, ids, B, K, depth_cap, len, best, path, toks, status, s);
    }));
    Py_INCREF(a[4]);
    return a[4];
}

// M, tpl_parent, tpl_rank, n_ret, tokens, parent, n_nodes, status, stream
GRAFT_PY(py_matrix_retrieve, 9) {
    int32_t V, k, B, K;
    sizes2(tensor(a[0]), V, k);
    const at::Tensor& tokens = tensor(a[4]);
    sizes2(tokens, B, K);
    at::Tensor fresh;
    int32_t* status;
    if (a[7] == Py_None) {
        fresh = empty_i32({B}, tokens.device());
        status = static_cast<int32_t*>(fresh.data_ptr());
    } else status = ptr<int32_t>(a[7]);
    const int32_t *M = ptr<int32_t>(a[0]), *tp = ptr<int32_t>(a[1]), *tr = ptr<int32_t>(a[2]), *nr = ptr<int32_t>(a[3]);
    const int32_t N = size_at(tensor(a[1]), 0);
    int32_t *tk = ptr<int32_t>(tokens), *p = ptr<int32_t>(a[5]), *n = ptr<int32_t>(a[6]);
    void* s = LaunchStream(a[8], tokens.device()).handle();
    check("graft_matrix_retrieve", unlocked([&] {
        return lib.graft_matrix_retrieve(M, V, k, tp, tr, N, nr, B, K, tk, p, n, status, s);
    }));
    if (fresh.defined()) return THPVariable_Wrap(std::move(fresh));
    Py_INCREF(a[7]);
    return a[7];
}

// tokens, n_nodes, logits, M, target_ids, workspace, stream
GRAFT_PY(py_matrix_update, 7) {
    const at::Tensor &lg = tensor(a[2]), &M = tensor(a[3]);
    if (lg.dim() != 3) {
        PyErr_Format(PyExc_ValueError, "expected logits of 3 dimensions, got %d", static_cast<int>(lg.dim()));
        throw PythonError();
    }
    const int32_t B = size_at(lg, 0), K = size_at(lg, 1), V = size_at(lg, 2), k = size_at(M, 1);
    const LaunchStream stream(a[6], lg.device());
    at::Tensor fresh, new_ws;
    int32_t* ids;
    if (a[4] == Py_None) {
        fresh = empty_i32({B, K}, lg.device());
        ids = static_cast<int32_t*>(fresh.data_ptr());
    } else ids = ptr<int32_t>(a[4]);
    void* ws;
    size_t ws_bytes;
    if (a[5] == Py_None) {
        ws_bytes = lib.graft_matrix_update_workspace_bytes(B, K, V, k);
        ws_bytes = ws_bytes > 8 ? ws_bytes : 8;
        new_ws = stream.scratch(ws_bytes);
        ws = new_ws.data_ptr();
    } else {
        const at::Tensor& w = tensor(a[5]);
        ws = ptr<void>(w);
        ws_bytes = static_cast<size_t>(w.numel());
    }
    const int32_t *tk = ptr<int32_t>(a[0]), *n = ptr<int32_t>(a[1]);
    const float* logits = ptr<float>(lg);
    int32_t* Mp = ptr<int32_t>(M);
    void* s = stream.handle();
    check("graft_matrix_update", unlocked([&] {
        return lib.graft_matrix_update(tk, n, logits, V, B, K, Mp, k, ids, ws, ws_bytes, s);
    }));
    if (fresh.defined()) return THPVariable_Wrap(std::move(fresh));
    Py_INCREF(a[4]);
    return a[4];
}

// k_cache, v_cache, layer_stride, n_layers, strides, block_table, prefix_len, path, accept_len, K_max, Hkv, D, out, stream
GRAFT_PY(py_kv_compact, 14) {
    GRAFT_KEY(new_prefix_len); GRAFT_KEY(status);
    const at::Tensor &k = tensor(a[0]), &v = tensor(a[1]), &table = tensor(a[5]), &path = tensor(a[7]);
    int32_t B, width;
    sizes2(path, B, width);
    const at::ScalarType type = k.scalar_type();
    if ((type != at::kFloat && type != at::kBFloat16) || v.scalar_type() != type) {
        PyErr_SetString(PyExc_AssertionError, "the caches are both float32 or both bfloat16");
        throw PythonError();
    }
    const int64_t layer_stride = to_i64(a[2]);
    const int32_t n_layers = to_i32(a[3]), K = to_i32(a[9]), Hkv = to_i32(a[10]), D = to_i32(a[11]);
    const Strides st = strides_of(a[4]);
    Outputs out(a[12], path.device());
    int32_t* new_len = out.get(k_new_prefix_len, {B});
    int32_t* status = out.get(k_status, {B});
    void *kp = ptr<void>(k), *vp = ptr<void>(v);
    const int32_t *tp = ptr<int32_t>(table), *pl = ptr<int32_t>(a[6]), *pp = ptr<int32_t>(path), *al = ptr<int32_t>(a[8]);
    const int32_t max_pages = size_at(table, 1);
    void* s = LaunchStream(a[13], path.device()).handle();
    check("graft_kv_compact", unlocked([&] {
        return lib.graft_kv_compact(kp, vp, layer_stride, n_layers, st.page, st.token, st.head, tp, max_pages, pl, pp, al, B,
                                    width - 1, K, Hkv, D, type == at::kFloat ? GRAFT_F32 : GRAFT_BF16, new_len, status, s);
    }));
    return out.release();
}

// parent, tokens, logq, n_nodes, chk_depth, chk_log_tau, chk_keep, chk_ret, out, stream
GRAFT_PY(py_prune_select, 10) {
    GRAFT_KEY(parent); GRAFT_KEY(tokens); GRAFT_KEY(index); GRAFT_KEY(n_nodes); GRAFT_KEY(stage); GRAFT_KEY(n_ret); GRAFT_KEY(status);
    const at::Tensor& parent = tensor(a[0]);
    int32_t B, K;
    sizes2(parent, B, K);
    Outputs out(a[8], parent.device());
    int32_t* op = out.get(k_parent, {B, K});
    int32_t* ot = out.get(k_tokens, {B, K});
    int32_t* oi = out.get(k_index, {B, K});
    int32_t* on = out.get(k_n_nodes, {B});
    int32_t* stage = out.get(k_stage, {B});
    int32_t* nr = out.get(k_n_ret, {B});
    int32_t* status = out.get(k_status, {B});
    const int32_t *p = ptr<int32_t>(parent), *tk = ptr<int32_t>(a[1]), *n = ptr<int32_t>(a[3]), *cd = ptr<int32_t>(a[4]),
                  *ck = ptr<int32_t>(a[6]), *cr = ptr<int32_t>(a[7]);
    const float *lq = ptr<float>(a[2]), *ct = ptr<float>(a[5]);
    const int32_t n_chk = size_at(tensor(a[4]), 0);
    void* s = LaunchStream(a[9], parent.device()).handle();
    check("graft_prune_select", unlocked([&] {
        return lib.graft_prune_select(p, tk, lq, n, B, K, cd, ct, ck, cr, n_chk, op, ot, oi, on, stage, nr, status, s);
    }));
    return out.release();
}

// path of the library, GraftError
PyObject* py_bind(PyObject*, PyObject* args) {
    const char* path;
    PyObject* error;
    if (!PyArg_ParseTuple(args, "sO", &path, &error)) return nullptr;
    void* h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!h) return PyErr_Format(PyExc_OSError, "%s", dlerror());
    Library l;
#define X(name)                                                                      \
    l.name = reinterpret_cast<decltype(&::name)>(dlsym(h, #name));                    \
    if (!l.name) return PyErr_Format(PyExc_OSError, "%s does not export " #name, path);
    GRAFT_ENTRY_POINTS(X)
#undef X
    lib = l;
    Py_INCREF(error);
    Py_XDECREF(graft_error);
    graft_error = error;
    Py_RETURN_NONE;
}

#define GRAFT_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, "bind(path, error_class): resolve the library's entry points"},
    GRAFT_METHOD(retrieve), GRAFT_METHOD(build_tree_mask), GRAFT_METHOD(tree_attn), GRAFT_METHOD(accept),
    GRAFT_METHOD(accept_noalloc), GRAFT_METHOD(matrix_retrieve), GRAFT_METHOD(matrix_update), GRAFT_METHOD(kv_compact),
    GRAFT_METHOD(prune_select), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", "Marshalling of the graft_* calls.", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    s_page = PyUnicode_InternFromString("page");
    s_token = PyUnicode_InternFromString("token");
    s_head = PyUnicode_InternFromString("head");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return PyModule_Create(&module_def);
}
