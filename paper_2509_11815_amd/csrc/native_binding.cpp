// Argument marshalling of the Python binding in C++ (host code only, a CPython extension module).
//
// Eager callers make one to seven library calls of 3 - 20 us of GPU time each per round, so the host
// time of a call decides how fast they run: marshalled in Python (ctypes objects, tensor attributes
// one by one, a stream look-up) a call cost 9 - 17 us, here it costs 3 - 8 us, most of it the
// launch itself (a step of 32 layers: 316 -> 144 us of host time per pass, six levels of tree growth
// 113 -> 56 us, and with it the growth itself 122 -> 78 us).  Every function takes its arguments by position, None for an omitted one; names, defaults
// and documentation are binding.py's.  The library's entry points arrive as addresses (bind()), so that
// the library binding.py has loaded is the one that is called.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <array>
#include <optional>
#include <string>

#include "specvlm.h"

namespace {

// ---- the library's entry points ------------------------------------------------------------------
#define SPECVLM_NATIVE_ENTRIES(X)                                                                          \
    X(specvlm_last_hip_error) X(specvlm_tree_verify_attn_workspace_bytes) X(specvlm_tree_verify_attn_num_splits) X(specvlm_tree_verify_attn)      \
    X(specvlm_tree_verify_attn_static) X(specvlm_tree_verify_attn_vector_alu) X(specvlm_node_argmax)       \
    X(specvlm_tree_accept) X(specvlm_node_argmax_accept) X(specvlm_tree_accept_sample) X(specvlm_kv_compact) \
    X(specvlm_draft_topk) X(specvlm_draft_topk_select) X(specvlm_draft_select) X(specvlm_draft_finalize)   \
    X(specvlm_head_argmax_workspace_bytes) X(specvlm_head_argmax) X(specvlm_visual_pool) X(specvlm_visual_prune)  \
    X(specvlm_visual_pool_padded) X(specvlm_visual_prune_padded)
#define SPECVLM_DECLARE(name) decltype(&::name) name;
struct Entries { SPECVLM_NATIVE_ENTRIES(SPECVLM_DECLARE) } lib;
#undef SPECVLM_DECLARE
PyObject* g_error = nullptr;                     // binding.SpecvlmError

template <typename... A>
[[noreturn]] void fail(PyObject* type, const char* format, A... args) {
    PyErr_Format(type, format, args...);
    throw python_error();
}

// ---- arguments -----------------------------------------------------------------------------------
struct Arguments {
    PyObject* const* a;
    Py_ssize_t n;
    const char* what;
    PyObject* obj(int i) const {
        if (i >= n) fail(PyExc_TypeError, "%s: too few arguments", what);
        return a[i];
    }
    bool given(int i) const { return obj(i) != Py_None; }
    const at::Tensor& tensor(int i, const char* name) const {
        PyObject* o = obj(i);
        if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s: %s must be a tensor", what, name);
        return THPVariable_Unpack(o);
    }
    void* ptr(int i, const char* name) const { return given(i) ? tensor(i, name).data_ptr() : nullptr; }
    int32_t* i32_unchecked(int i, const char* name) const { return static_cast<int32_t*>(ptr(i, name)); }
    // a contiguous int32 device tensor or None
    int32_t* i32(int i, const char* name) const {
        if (!given(i)) return nullptr;
        const at::Tensor& t = tensor(i, name);
        if (!t.is_cuda() || t.scalar_type() != at::kInt || !t.is_contiguous())
            fail(PyExc_TypeError, "%s must be a contiguous int32 device tensor", name);
        return static_cast<int32_t*>(t.data_ptr());
    }
    // a float32 device tensor with a contiguous last dimension, or None
    float* f32(int i, const char* name) const {
        if (!given(i)) return nullptr;
        const at::Tensor& t = tensor(i, name);
        if (!t.is_cuda() || t.scalar_type() != at::kFloat || t.stride(-1) != 1)
            fail(PyExc_TypeError, "%s must be a float32 device tensor with a contiguous last dimension", name);
        return static_cast<float*>(t.data_ptr());
    }
    int64_t integer(int i) const {
        const long long v = PyLong_AsLongLong(obj(i));
        if (v == -1 && PyErr_Occurred()) throw python_error();
        return v;
    }
    // what int() / float() make of the argument
    int64_t as_int(int i) const {
        THPObjectPtr number(PyNumber_Long(obj(i)));
        const long long v = number ? PyLong_AsLongLong(number) : -1;
        if (v == -1 && PyErr_Occurred()) throw python_error();
        return v;
    }
    float as_float(int i) const {
        THPObjectPtr number(PyNumber_Float(obj(i)));
        const double v = number ? PyFloat_AsDouble(number) : -1.0;
        if (v == -1.0 && PyErr_Occurred()) throw python_error();
        return static_cast<float>(v);
    }
    float real(int i) const {
        const double v = PyFloat_AsDouble(obj(i));
        if (v == -1.0 && PyErr_Occurred()) throw python_error();
        return static_cast<float>(v);
    }
    // a torch stream, or None for the current one
    void* stream(int i) const {
        if (!given(i)) return c10::hip::getCurrentHIPStream().stream();
        THPObjectPtr handle(PyObject_GetAttrString(obj(i), "cuda_stream"));
        if (!handle) throw python_error();
        void* s = PyLong_AsVoidPtr(handle);
        if (!s && PyErr_Occurred()) throw python_error();
        return s;
    }
};

int32_t dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kBFloat16) return SPECVLM_BF16;
    if (t.scalar_type() == at::kFloat) return SPECVLM_F32;
    fail(PyExc_TypeError, "bfloat16 or float32 expected, got %s", c10::toString(t.scalar_type()));
}

void check(int32_t rc, const char* what) {
    if (rc == SPECVLM_OK) return;
    static const char* const names[] = {"OK", "INVALID_ARG", "UNSUPPORTED", "WORKSPACE_TOO_SMALL", "HIP_ERROR"};
    std::string msg = std::string(what) + ": " + (rc >= 0 && rc < 5 ? names[rc] : std::to_string(rc).c_str());
    if (rc == SPECVLM_HIP_ERROR) msg += " (hipError " + std::to_string(lib.specvlm_last_hip_error()) + ")";
    fail(g_error, "%s", msg.c_str());
}

// A library call without the interpreter lock: a launch can block on a full queue, and other threads go on meanwhile.
// (The caller's frame holds the tensors; arguments are taken from Python objects before the lock is given up.)
template <typename F, typename... A>
int32_t unlocked(F* entry, A... args) {
    PyThreadState* const state = PyEval_SaveThread();
    const int32_t rc = entry(args...);
    PyEval_RestoreThread(state);
    return rc;
}

void want(bool ok, const char* message) {
    if (!ok) fail(PyExc_ValueError, "%s", message);
}

// The stream of a call: argument i, or the current one.  Tensors that the call allocates or zeroes belong to it: an
// explicit stream is made the current one of `like`'s device for the length of the call, so that a zero fill comes before
// the kernel, and memory given back meanwhile is not handed to other streams' work.  A returned tensor is recorded on the
// stream that was current, where the caller is likely to use it.
class CallStream {
public:
    CallStream(const Arguments& a, int i, const at::Tensor& like) : a_(a), i_(i) {
        if (!a.given(i) || !like.is_cuda()) return;
        void* const handle = a.stream(i);
        const auto device = like.device().index();
        const auto current = c10::hip::getCurrentHIPStream(device);
        if (current.stream() == handle) return;
        before_ = current;
        device_ = like.device();
        c10::hip::setCurrentHIPStream(handle ? c10::hip::getStreamFromExternal(static_cast<hipStream_t>(handle), device)
                                             : c10::hip::getDefaultHIPStream(device));
    }
    void* handle() const { return a_.stream(i_); }
    ~CallStream() { if (before_) c10::hip::setCurrentHIPStream(*before_); }
    CallStream(const CallStream&) = delete;
    CallStream& operator=(const CallStream&) = delete;
    PyObject* wrap(const at::Tensor& made) const {
        if (before_ && made.defined()) made.record_stream(c10::Stream(c10::Stream::UNSAFE, *device_, before_->id()));
        return THPVariable_Wrap(made);
    }
    // The given tensor as a new reference, or a new one wrapped.
    PyObject* keep(PyObject* given, const at::Tensor& made) const {
        if (given != Py_None) { Py_INCREF(given); return given; }
        return wrap(made);
    }

private:
    const Arguments& a_;
    const int i_;
    std::optional<c10::hip::HIPStream> before_;
    std::optional<c10::Device> device_;
};

at::Tensor new_i32(const at::Tensor& like, at::IntArrayRef size) { return at::empty(size, like.options().dtype(at::kInt)); }
at::Tensor new_f32(const at::Tensor& like, at::IntArrayRef size) { return at::empty(size, like.options().dtype(at::kFloat)); }

template <size_t N>
PyObject* tuple_of(const std::array<PyObject*, N>& items) {
    PyObject* t = PyTuple_New(N);
    for (size_t i = 0; i < N; ++i) PyTuple_SET_ITEM(t, i, items[i]);
    return t;
}

// Per-request arrival counters of the fused calls: zeroed when omitted, else checked.
at::Tensor counters_of(const Arguments& a, int i, const at::Tensor& like, int64_t B) {
    if (!a.given(i)) return at::zeros({B * SPECVLM_COUNTER_STRIDE}, like.options().dtype(at::kInt));
    a.i32(i, "counters");
    const at::Tensor& t = a.tensor(i, "counters");
    if (t.numel() < B * SPECVLM_COUNTER_STRIDE)
        fail(PyExc_ValueError, "counters must hold B * COUNTER_STRIDE = %lld int32 words", static_cast<long long>(B * SPECVLM_COUNTER_STRIDE));
    return t;
}

// The four outputs of an acceptance walk: argument i's tuple, which has the path capacity of its path, or new tensors
// with that of argument cap.
struct WalkOutputs {
    THPObjectPtr seq;                                // keeps the given tensors (the argument may be any iterable)
    at::Tensor accept_len, path, bonus, committed;
    PyObject* given[4] = {Py_None, Py_None, Py_None, Py_None};
    int64_t path_cap;
    WalkOutputs(const Arguments& a, int i, const at::Tensor& like, int64_t B, int cap_arg) {
        if (!a.given(i)) {
            const int64_t cap = path_cap = a.integer(cap_arg);
            accept_len = new_i32(like, {B}); path = new_i32(like, {B, cap});
            bonus = new_i32(like, {B}); committed = new_i32(like, {B, cap});
            return;
        }
        seq = PySequence_Fast(a.obj(i), "out must be a sequence");
        if (!seq) throw python_error();
        want(PySequence_Fast_GET_SIZE(seq.get()) == 4, "out must hold accept_len, path, bonus_tok and committed_tok");
        at::Tensor* to[4] = {&accept_len, &path, &bonus, &committed};
        for (int x = 0; x < 4; ++x) {
            given[x] = PySequence_Fast_GET_ITEM(seq.get(), x);
            if (!THPVariable_Check(given[x])) fail(PyExc_TypeError, "out must hold tensors");
            *to[x] = THPVariable_Unpack(given[x]);
        }
        path_cap = path.size(1);
    }
    static int32_t* p(const at::Tensor& t) { return static_cast<int32_t*>(t.data_ptr()); }
    std::array<PyObject*, 4> take(const CallStream& on) const {
        return {on.keep(given[0], accept_len), on.keep(given[1], path), on.keep(given[2], bonus), on.keep(given[3], committed)};
    }
};

// ---- attention and compaction --------------------------------------------------------------------
// (q, k, v, prefix_len, parent, num_nodes, block_table, out, lse, workspace, err_flag, softmax_scale, num_splits, desc,
//  stream, entry): entry 0 caller's workspace, 1 static scratch, 2 vector-ALU kernel
PyObject* tree_verify_attn(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const int entry = nargs > 15 ? static_cast<int>(PyLong_AsLong(args[15])) : 0;
    const char* const what = entry == 0 ? "specvlm_tree_verify_attn"
                             : entry == 1 ? "specvlm_tree_verify_attn_static" : "specvlm_tree_verify_attn_vector_alu";
    const Arguments a{args, nargs, what};
    const at::Tensor &q = a.tensor(0, "q"), &k = a.tensor(1, "k_cache"), &v = a.tensor(2, "v_cache");
    const CallStream on(a, 14, q);
    at::Tensor made;
    if (!a.given(7)) made = at::zeros_like(q);       // rows past num_nodes are not written
    const at::Tensor& out = a.given(7) ? a.tensor(7, "out") : made;
    specvlm_attn_desc local{};
    const specvlm_attn_desc* desc = &local;
    Py_buffer view{};
    struct Release { Py_buffer* v; ~Release() { if (v->obj) PyBuffer_Release(v); } } release{&view};
    if (a.given(13)) {
        if (PyObject_GetBuffer(a.obj(13), &view, PyBUF_SIMPLE)) throw python_error();
        if (view.len != static_cast<Py_ssize_t>(sizeof(specvlm_attn_desc))) fail(PyExc_TypeError, "desc must be an AttnDesc");
        desc = static_cast<const specvlm_attn_desc*>(view.buf);
    } else {
        want(q.dim() == 4 && k.dim() == 4, "q and k_cache must have four dimensions");
        want(q.stride(3) == 1 && k.stride(3) == 1, "innermost dimension must be contiguous");
        specvlm_attn_desc& d = local;
        d.dtype = dtype_code(q);
        d.B = q.size(0); d.N_max = q.size(1); d.H_q = q.size(2); d.D = q.size(3);
        d.H_kv = k.size(1);
        d.softmax_scale = a.as_float(11);
        d.num_splits = static_cast<int32_t>(a.as_int(12));
        d.q_stride_b = q.stride(0); d.q_stride_n = q.stride(1); d.q_stride_h = q.stride(2);
        d.o_stride_b = out.stride(0); d.o_stride_n = out.stride(1); d.o_stride_h = out.stride(2);
        d.kv_stride_b = k.stride(0); d.kv_stride_h = k.stride(1); d.kv_stride_t = k.stride(2);
        d.kv_capacity = k.size(2);
        if (a.given(6)) {
            d.paged = 1;
            d.block_size = k.size(2);
            d.max_blocks_per_req = a.tensor(6, "block_table").size(1);
            d.num_blocks = k.size(0);
            d.kv_capacity = d.max_blocks_per_req * d.block_size;
        }
    }
    want(k.strides() == v.strides() && k.sizes() == v.sizes(), "K and V caches must share one geometry");
    const int32_t *table = a.i32(6, "block_table"), *prefix = a.i32(3, "prefix_len"), *nn = a.i32(5, "num_nodes"),
                  *parent = a.i32(4, "parent");
    float* lse = static_cast<float*>(a.ptr(8, "lse"));
    int32_t* err = a.i32_unchecked(10, "err_flag");
    int32_t rc;
    at::Tensor scratch;                              // (of the call's stream: may be given back as soon as the call is enqueued)
    if (entry == 0) {
        void* ws = nullptr;
        size_t bytes = 0;
        if (a.given(9)) {
            const at::Tensor& t = a.tensor(9, "workspace");
            ws = t.data_ptr();
            bytes = t.numel() * t.element_size();
        } else if (lib.specvlm_tree_verify_attn_num_splits(desc) > 1) {       // (others need none; filling one costs more than it gains)
            bytes = lib.specvlm_tree_verify_attn_workspace_bytes(desc);
            scratch = at::zeros({static_cast<int64_t>(bytes)}, q.options().dtype(at::kByte));   // zero-filled once, as the ABI asks
            ws = scratch.data_ptr();
        }
        rc = unlocked(lib.specvlm_tree_verify_attn, desc, q.data_ptr(), k.data_ptr(), v.data_ptr(), table, prefix, nn, parent,
                                          out.data_ptr(), lse, ws, bytes, err, on.handle());
    } else {
        auto* fn = entry == 1 ? lib.specvlm_tree_verify_attn_static : lib.specvlm_tree_verify_attn_vector_alu;
        rc = unlocked(fn, desc, q.data_ptr(), k.data_ptr(), v.data_ptr(), table, prefix, nn, parent, out.data_ptr(), lse, err, on.handle());
    }
    check(rc, what);
    return on.keep(a.obj(7), made);
    END_HANDLE_TH_ERRORS
}

// (k_caches, v_caches, prefix_len, path, accept_len, block_table, new_prefix_len, moved_idx, k_ptrs, v_ptrs, err_flag, stream)
PyObject* kv_compact(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_kv_compact"};
    const at::Tensor &k = a.tensor(0, "k_caches"), &path = a.tensor(3, "path");
    want(path.dim() == 2, "path must have two dimensions");
    const CallStream on(a, 11, path);
    const int64_t B = path.size(0), cap = path.size(1);
    const bool by_ptr = a.given(8);
    const int x = by_ptr ? 0 : 1;                    // first per-layer dimension
    want(k.dim() == 4 + x, "k_caches must be [L, <cache dims>], or one layer's cache beside layer_ptrs");
    void *kb = nullptr, *vb = nullptr;
    int64_t L, layer_stride = 0;
    if (by_ptr) {
        L = a.tensor(8, "layer_ptrs").numel();
    } else {
        const at::Tensor& v = a.tensor(1, "v_caches");
        want(k.strides() == v.strides(), "K and V caches must share one geometry");
        L = k.size(0);
        layer_stride = k.stride(0);
        kb = k.data_ptr();
        vb = v.data_ptr();
    }
    specvlm_attn_desc d{};
    d.dtype = dtype_code(k);
    d.B = B; d.H_q = d.H_kv = k.size(x + 1); d.D = k.size(x + 3); d.N_max = SPECVLM_MAX_NODES;
    d.kv_stride_b = k.stride(x); d.kv_stride_h = k.stride(x + 1); d.kv_stride_t = k.stride(x + 2);
    d.kv_capacity = k.size(x + 2);
    if (a.given(5)) {
        d.paged = 1;
        d.block_size = k.size(x + 2);
        d.max_blocks_per_req = a.tensor(5, "block_table").size(1);
        d.num_blocks = k.size(x);
        d.kv_capacity = d.max_blocks_per_req * d.block_size;
    }
    at::Tensor made;
    if (!a.given(6)) made = new_i32(path, {B});
    int32_t* new_prefix = static_cast<int32_t*>(a.given(6) ? a.ptr(6, "new_prefix_len") : made.data_ptr());
    check(unlocked(lib.specvlm_kv_compact, &d, static_cast<int32_t>(L), kb, vb, layer_stride,
                                 static_cast<void* const*>(a.ptr(8, "layer_ptrs")), static_cast<void* const*>(a.ptr(9, "layer_ptrs")),
                                 a.i32(5, "block_table"), a.i32(2, "prefix_len"), a.i32(3, "path"), static_cast<int32_t>(cap),
                                 a.i32(4, "accept_len"), new_prefix, a.i32_unchecked(7, "moved_idx"),
                                 a.i32_unchecked(10, "err_flag"), on.handle()),
          a.what);
    Py_INCREF(a.obj(7));                             // (moved_idx is None where it is not given)
    return tuple_of<2>({on.keep(a.obj(6), made), a.obj(7)});
    END_HANDLE_TH_ERRORS
}

// ---- arg-max and acceptance ----------------------------------------------------------------------
const at::Tensor& logits_of(const Arguments& a, int i) {
    const at::Tensor& t = a.tensor(i, "logits");
    want(t.dim() == 3, "logits must have three dimensions");
    want(t.stride(2) == 1, "vocab dimension must be contiguous");
    return t;
}

// (logits, num_nodes, out, stream)
PyObject* node_argmax(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_node_argmax"};
    const at::Tensor& l = logits_of(a, 0);
    const CallStream on(a, 3, l);
    at::Tensor made;
    if (!a.given(2)) made = new_i32(l, {l.size(0), l.size(1)});
    check(unlocked(lib.specvlm_node_argmax, dtype_code(l), l.size(0), l.size(1), l.size(2), l.data_ptr(), l.stride(0), l.stride(1),
                                  a.i32(1, "num_nodes"),
                                  static_cast<int32_t*>(a.given(2) ? a.ptr(2, "out") : made.data_ptr()), on.handle()),
          a.what);
    return on.keep(a.obj(2), made);
    END_HANDLE_TH_ERRORS
}

// (parent, draft_tok, amax, num_nodes, path_cap, err_flag, out, stream)
PyObject* tree_accept(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_tree_accept"};
    const at::Tensor& parent = a.tensor(0, "parent");
    want(parent.dim() == 2, "parent must have two dimensions");
    const CallStream on(a, 7, parent);
    const int64_t B = parent.size(0);
    const WalkOutputs o(a, 6, parent, B, 4);
    check(unlocked(lib.specvlm_tree_accept, B, parent.size(1), o.path_cap, a.i32(0, "parent"), a.i32(1, "draft_tok"), a.i32(2, "amax"),
                                  a.i32(3, "num_nodes"), o.p(o.accept_len), o.p(o.path), o.p(o.bonus), o.p(o.committed),
                                  a.i32_unchecked(5, "err_flag"), on.handle()),
          a.what);
    return tuple_of<4>(o.take(on));
    END_HANDLE_TH_ERRORS
}

// (logits, parent, draft_tok, num_nodes, path_cap, counters, amax, err_flag, out, stream)
PyObject* node_argmax_accept(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_node_argmax_accept"};
    const at::Tensor& l = logits_of(a, 0);
    const CallStream on(a, 9, l);
    const int64_t B = l.size(0), N = l.size(1);
    const WalkOutputs o(a, 8, l, B, 4);
    at::Tensor made;
    if (!a.given(6)) made = new_i32(l, {B, N});
    int32_t* amax = a.given(6) ? a.i32(6, "amax") : static_cast<int32_t*>(made.data_ptr());
    const at::Tensor counters = counters_of(a, 5, l, B);
    check(unlocked(lib.specvlm_node_argmax_accept, dtype_code(l), B, N, l.size(2), o.path_cap, l.data_ptr(), l.stride(0), l.stride(1),
                                         a.i32(3, "num_nodes"), a.i32(1, "parent"), a.i32(2, "draft_tok"), amax,
                                         o.p(o.accept_len), o.p(o.path), o.p(o.bonus), o.p(o.committed), o.p(counters),
                                         a.i32_unchecked(7, "err_flag"), on.handle()),
          a.what);
    const auto w = o.take(on);
    return tuple_of<5>({on.keep(a.obj(6), made), w[0], w[1], w[2], w[3]});
    END_HANDLE_TH_ERRORS
}

// (parent, draft_tok, logits, u_accept, u_bonus, temperature, num_nodes, path_cap, err_flag, out, stream)
PyObject* tree_accept_sample(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_tree_accept_sample"};
    const at::Tensor& l = logits_of(a, 2);
    const CallStream on(a, 10, l);
    const int64_t B = l.size(0), N = l.size(1);
    const at::Tensor &ua = a.tensor(3, "u_accept"), &ub = a.tensor(4, "u_bonus");
    if (ua.scalar_type() != at::kFloat || ua.dim() != 2 || ua.size(0) != B || ua.size(1) != N || !ua.is_contiguous())
        fail(PyExc_ValueError, "u_accept must be a contiguous float32 tensor of shape (%lld, %lld)", static_cast<long long>(B), static_cast<long long>(N));
    if (ub.scalar_type() != at::kFloat || ub.dim() != 1 || ub.size(0) != B || !ub.is_contiguous())
        fail(PyExc_ValueError, "u_bonus must be a contiguous float32 tensor of shape (%lld,)", static_cast<long long>(B));
    const WalkOutputs o(a, 9, l, B, 7);
    check(unlocked(lib.specvlm_tree_accept_sample, dtype_code(l), B, N, l.size(2), o.path_cap, a.i32(0, "parent"), a.i32(1, "draft_tok"),
                                         l.data_ptr(), l.stride(0), l.stride(1), a.i32(6, "num_nodes"), a.real(5),
                                         static_cast<const float*>(ua.data_ptr()), static_cast<const float*>(ub.data_ptr()),
                                         o.p(o.accept_len), o.p(o.path), o.p(o.bonus), o.p(o.committed),
                                         a.i32_unchecked(8, "err_flag"), on.handle()),
          a.what);
    return tuple_of<4>(o.take(on));
    END_HANDLE_TH_ERRORS
}

// ---- draft growth --------------------------------------------------------------------------------
// A level's inputs and outputs: arguments first .. first + 5 are cum, parent_idx, score_out, token_out, parent_out, lse_out.
struct Level {
    at::Tensor score, token, parent_made;
    const float* cum;
    const int32_t* parent_idx;
    int64_t cum_stride, parent_stride;
    int32_t* parent_out;
    float* lse;
    Level(const Arguments& a, int first, const at::Tensor& l, int64_t K) {
        const int64_t B = l.size(0), want_n = l.size(1) * K;
        score = a.given(first + 2) ? a.tensor(first + 2, "score_out") : new_f32(l, {B, want_n});
        token = a.given(first + 3) ? a.tensor(first + 3, "token_out") : new_i32(l, {B, want_n});
        const bool has_parent = a.given(first + 4) || a.given(first + 1);
        if (!a.given(first + 4) && has_parent) parent_made = new_i32(l, {B, want_n});
        const at::Tensor& par = a.given(first + 4) ? a.tensor(first + 4, "parent_out") : parent_made;
        auto fits = [&](const at::Tensor& t) { return t.dim() == 2 && t.stride(0) == score.stride(0) && t.stride(1) == 1 && t.size(1) >= want_n; };
        want(fits(score) && fits(token) && (!has_parent || fits(par)),
             "score_out / token_out / parent_out must share one row stride and hold W*K entries");
        if (token.scalar_type() != at::kInt || (has_parent && par.scalar_type() != at::kInt))
            fail(PyExc_TypeError, "token_out / parent_out must be int32");
        a.f32(first + 2, "score_out");
        cum = a.f32(first, "cum");
        cum_stride = cum ? a.tensor(first, "cum").stride(0) : 0;
        parent_idx = a.i32_unchecked(first + 1, "parent_idx");
        parent_stride = parent_idx ? a.tensor(first + 1, "parent_idx").stride(0) : 0;
        parent_out = has_parent ? static_cast<int32_t*>(par.data_ptr()) : nullptr;
        lse = a.f32(first + 5, "lse_out");
    }
    PyObject* parent(const CallStream& on, const Arguments& a, int first) const {
        if (a.given(first + 4) || !parent_made.defined()) { Py_INCREF(a.obj(first + 4)); return a.obj(first + 4); }
        return on.wrap(parent_made);
    }
};

// (logits, K, cum, parent_idx, score_out, token_out, parent_out, lse_out, stream)
PyObject* draft_topk(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_draft_topk"};
    const at::Tensor& l = logits_of(a, 0);
    const CallStream on(a, 8, l);
    const int64_t K = a.integer(1);
    const Level v(a, 2, l, K);
    check(unlocked(lib.specvlm_draft_topk, dtype_code(l), l.size(0), l.size(1), l.size(2), K, l.data_ptr(), l.stride(0), l.stride(1),
                                 v.cum, v.cum_stride, v.parent_idx, v.parent_stride, static_cast<float*>(v.score.data_ptr()),
                                 static_cast<int32_t*>(v.token.data_ptr()), v.parent_out, v.score.stride(0), v.lse, on.handle()),
          a.what);
    return tuple_of<3>({on.keep(a.obj(4), v.score), on.keep(a.obj(5), v.token), v.parent(on, a, 2)});
    END_HANDLE_TH_ERRORS
}

// The outputs of a selection: arguments first .. first + 2 are sel_out, sel_score_out, count_out.
struct Selection {
    at::Tensor sel, score, count;
    Selection(const Arguments& a, int first, const at::Tensor& like, int64_t B, int64_t M) {
        sel = a.given(first) ? a.tensor(first, "sel_out") : new_i32(like, {B, M});
        score = a.given(first + 1) ? a.tensor(first + 1, "sel_score_out") : new_f32(like, {B, M});
        count = a.given(first + 2) ? a.tensor(first + 2, "count_out") : new_i32(like, {B});
        a.i32(first, "sel_out");
        a.f32(first + 1, "sel_score_out");
        a.i32(first + 2, "count_out");
    }
};

// (logits, K, M, cum, parent_idx, score_out, token_out, parent_out, lse_out, index_base, sel_out, sel_score_out, count_out,
//  counters, stream)
PyObject* draft_topk_select(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_draft_topk_select"};
    const at::Tensor& l = logits_of(a, 0);
    const CallStream on(a, 14, l);
    const int64_t K = a.integer(1), M = a.integer(2), B = l.size(0);
    const Level v(a, 3, l, K);
    const Selection s(a, 10, l, B, M);
    const at::Tensor counters = counters_of(a, 13, l, B);
    check(unlocked(lib.specvlm_draft_topk_select, dtype_code(l), B, l.size(1), l.size(2), K, l.data_ptr(), l.stride(0), l.stride(1),
                                        v.cum, v.cum_stride, v.parent_idx, v.parent_stride, static_cast<float*>(v.score.data_ptr()),
                                        static_cast<int32_t*>(v.token.data_ptr()), v.parent_out, v.score.stride(0), v.lse, M,
                                        a.integer(9), static_cast<int32_t*>(s.sel.data_ptr()), static_cast<float*>(s.score.data_ptr()),
                                        static_cast<int32_t*>(s.count.data_ptr()), static_cast<int32_t*>(counters.data_ptr()), on.handle()),
          a.what);
    return tuple_of<6>({on.keep(a.obj(5), v.score), on.keep(a.obj(6), v.token), v.parent(on, a, 3), on.keep(a.obj(10), s.sel),
                        on.keep(a.obj(11), s.score), on.keep(a.obj(12), s.count)});
    END_HANDLE_TH_ERRORS
}

// (score, M, num_cand, index_base, sel_out, sel_score_out, count_out, stream)
PyObject* draft_select(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_draft_select"};
    const at::Tensor& score = a.tensor(0, "score");
    want(score.dim() == 2, "score must have two dimensions");
    const CallStream on(a, 7, score);
    a.f32(0, "score");
    const int64_t B = score.size(0), M = a.integer(1);
    const Selection s(a, 4, score, B, M);
    check(unlocked(lib.specvlm_draft_select, B, score.size(1), M, static_cast<const float*>(score.data_ptr()), score.stride(0), a.i32(2, "num_cand"),
                                   a.integer(3), static_cast<int32_t*>(s.sel.data_ptr()), static_cast<float*>(s.score.data_ptr()),
                                   static_cast<int32_t*>(s.count.data_ptr()), on.handle()),
          a.what);
    return tuple_of<3>({on.keep(a.obj(4), s.sel), on.keep(a.obj(5), s.score), on.keep(a.obj(6), s.count)});
    END_HANDLE_TH_ERRORS
}

// (cand_score, cand_parent, cand_token, root_token, N_max, num_cand, err_flag, out, stream)
PyObject* draft_finalize(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_draft_finalize"};
    const at::Tensor &score = a.tensor(0, "cand_score"), &par = a.tensor(1, "cand_parent"), &tok = a.tensor(2, "cand_token");
    want(score.dim() == 2, "cand_score must have two dimensions");
    const CallStream on(a, 8, score);
    a.f32(0, "cand_score");
    const int64_t B = score.size(0), N = a.integer(4);
    for (const at::Tensor* t : {&par, &tok})
        want(t->scalar_type() == at::kInt && t->strides() == score.strides(), "cand_parent / cand_token must be int32 with cand_score's strides");
    at::Tensor t[4];
    PyObject* given[4] = {Py_None, Py_None, Py_None, Py_None};
    THPObjectPtr seq;
    if (a.given(7)) {
        seq = PySequence_Fast(a.obj(7), "out must be a sequence");
        if (!seq) throw python_error();
        want(PySequence_Fast_GET_SIZE(seq.get()) == 4, "out must hold parent, draft_tok, node_cand and num_nodes");
        for (int x = 0; x < 4; ++x) {
            given[x] = PySequence_Fast_GET_ITEM(seq.get(), x);
            if (x == 2 && given[x] == Py_None) continue;             // node_cand may be left out
            if (!THPVariable_Check(given[x])) fail(PyExc_TypeError, "out must hold tensors");
            t[x] = THPVariable_Unpack(given[x]);
            if (x != 2 && (!t[x].is_cuda() || t[x].scalar_type() != at::kInt || !t[x].is_contiguous()))
                fail(PyExc_TypeError, "%s must be a contiguous int32 device tensor", x == 0 ? "parent" : x == 1 ? "draft_tok" : "num_nodes");
        }
    } else {
        for (int x = 0; x < 3; ++x) t[x] = new_i32(score, {B, N});
        t[3] = new_i32(score, {B});
    }
    auto p = [&](int x) { return t[x].defined() ? static_cast<int32_t*>(t[x].data_ptr()) : nullptr; };
    check(unlocked(lib.specvlm_draft_finalize, B, score.size(1), N, static_cast<const float*>(score.data_ptr()),
                                     static_cast<const int32_t*>(par.data_ptr()), static_cast<const int32_t*>(tok.data_ptr()),
                                     score.stride(0), a.i32(5, "num_cand"), a.i32(3, "root_token"), p(0), p(1), p(2), p(3),
                                     a.i32_unchecked(6, "err_flag"), on.handle()),
          a.what);
    std::array<PyObject*, 4> r;
    for (int x = 0; x < 4; ++x) {
        if (t[x].defined()) { r[x] = on.keep(given[x], t[x]); continue; }
        Py_INCREF(Py_None);
        r[x] = Py_None;
    }
    return tuple_of<4>(r);
    END_HANDLE_TH_ERRORS
}

// ---- head and compressors ------------------------------------------------------------------------
// (hidden, weight, num_nodes, out, max_logit, workspace, stream)
PyObject* head_argmax(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_head_argmax"};
    const at::Tensor &h = a.tensor(0, "hidden"), &w = a.tensor(1, "weight");
    const CallStream on(a, 6, h);
    want(h.dim() == 3 && w.dim() == 2 && h.stride(2) == 1 && w.stride(1) == 1 && w.size(1) == h.size(2),
         "hidden [B,N_max,E] and weight [V,E] need a contiguous last dimension of equal size");
    const int64_t B = h.size(0), N = h.size(1), V = w.size(0);
    at::Tensor made, scratch;
    if (!a.given(3)) made = new_i32(h, {B, N});
    int32_t* out = a.given(3) ? a.i32(3, "out") : static_cast<int32_t*>(made.data_ptr());
    if (!a.given(5))                                 // zero-filled once, as the ABI asks
        scratch = at::zeros({static_cast<int64_t>(lib.specvlm_head_argmax_workspace_bytes(B, N, V))}, h.options().dtype(at::kByte));
    const at::Tensor& ws = a.given(5) ? a.tensor(5, "workspace") : scratch;
    check(unlocked(lib.specvlm_head_argmax, dtype_code(h), B, N, h.size(2), V, h.data_ptr(), h.stride(0), h.stride(1), w.data_ptr(), w.stride(0),
                                  a.i32(2, "num_nodes"), out, a.f32(4, "max_logit"), ws.data_ptr(),
                                  static_cast<size_t>(ws.numel() * ws.element_size()), on.handle()),
          a.what);
    return on.keep(a.obj(3), made);
    END_HANDLE_TH_ERRORS
}

// (x, ratio, num_tokens, out, out_tokens, err_flag, stream)
PyObject* visual_pool(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_visual_pool"};
    const at::Tensor& x = a.tensor(0, "x");
    const CallStream on(a, 6, x);
    want(x.dim() == 3, "x must have three dimensions");
    const int64_t B = x.size(0), T = x.size(1), E = x.size(2), ratio = a.integer(1);
    const int64_t Tp = ratio > 0 ? (T + ratio - 1) / ratio : T;      // (the library rejects ratio < 1)
    at::Tensor made, made_n;
    // a given result keeps its rows past a request's own, in a new one the call makes them zeros
    if (!a.given(3)) made = at::empty({B, Tp, E}, x.options());
    if (!a.given(4)) made_n = new_i32(x, {B});
    const at::Tensor& out = a.given(3) ? a.tensor(3, "out") : made;
    want(out.dim() == 3 && x.stride(2) == 1 && out.stride(2) == 1, "feature dimension must be contiguous");
    auto* const fn = a.given(3) ? lib.specvlm_visual_pool : lib.specvlm_visual_pool_padded;
    check(unlocked(fn, dtype_code(x), B, T, E, ratio, x.data_ptr(), x.stride(0), x.stride(1), a.i32(2, "num_tokens"),
                                  out.data_ptr(), out.stride(0), out.stride(1),
                                  a.given(4) ? a.i32(4, "out_tokens") : static_cast<int32_t*>(made_n.data_ptr()),
                                  a.i32_unchecked(5, "err_flag"), on.handle()),
          a.what);
    return tuple_of<2>({on.keep(a.obj(3), made), on.keep(a.obj(4), made_n)});
    END_HANDLE_TH_ERRORS
}

// (x, keep, out, err_flag, stream)
PyObject* visual_prune(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "specvlm_visual_prune"};
    const at::Tensor &x = a.tensor(0, "x"), &kept = a.tensor(1, "keep");
    const CallStream on(a, 4, x);
    want(x.dim() == 3 && kept.dim() == 2, "x must have three dimensions and keep two");
    const int64_t B = x.size(0), T = x.size(1), E = x.size(2), Tk = kept.size(1);
    at::Tensor made;
    if (!a.given(2)) made = at::empty({B, Tk, E}, x.options());      // (the call makes the rows of padding entries zeros)
    const at::Tensor& out = a.given(2) ? a.tensor(2, "out") : made;
    want(out.dim() == 3 && x.stride(2) == 1 && out.stride(2) == 1, "feature dimension must be contiguous");
    auto* const fn = a.given(2) ? lib.specvlm_visual_prune : lib.specvlm_visual_prune_padded;
    check(unlocked(fn, dtype_code(x), B, T, Tk, E, x.data_ptr(), x.stride(0), x.stride(1), a.i32(1, "keep"),
                                   out.data_ptr(), out.stride(0), out.stride(1), a.i32_unchecked(3, "err_flag"), on.handle()),
          a.what);
    return on.keep(a.obj(2), made);
    END_HANDLE_TH_ERRORS
}

// bind({entry point: address}, SpecvlmError)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    const Arguments a{args, nargs, "bind"};
    Entries e{};
#define SPECVLM_TAKE(name)                                                                             \
    {                                                                                                  \
        PyObject* o = PyDict_GetItemString(a.obj(0), #name);                                           \
        if (!o) fail(PyExc_ValueError, "bind: no address for %s", #name);                             \
        void* p = PyLong_AsVoidPtr(o);                                                                 \
        if (!p) fail(PyExc_ValueError, "bind: no address for %s", #name);                             \
        e.name = reinterpret_cast<decltype(e.name)>(p);                                                \
    }
    SPECVLM_NATIVE_ENTRIES(SPECVLM_TAKE)
#undef SPECVLM_TAKE
    Py_INCREF(a.obj(1));
    Py_XDECREF(g_error);
    g_error = a.obj(1);
    lib = e;
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

#define SPECVLM_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SPECVLM_METHOD(bind), SPECVLM_METHOD(tree_verify_attn), SPECVLM_METHOD(kv_compact), SPECVLM_METHOD(node_argmax),
    SPECVLM_METHOD(tree_accept), SPECVLM_METHOD(node_argmax_accept), SPECVLM_METHOD(tree_accept_sample),
    SPECVLM_METHOD(draft_topk), SPECVLM_METHOD(draft_topk_select), SPECVLM_METHOD(draft_select), SPECVLM_METHOD(draft_finalize),
    SPECVLM_METHOD(head_argmax), SPECVLM_METHOD(visual_pool), SPECVLM_METHOD(visual_prune),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_specvlm_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__specvlm_native() { return PyModule_Create(&module_def); }
