// Native marshalling of torch tensors into the C ABI (the Python package's
// fast path): a call checks its tensors, takes torch's current stream and
// calls the library without a Python-level check or a ctypes conversion per
// argument, and a round or a draft stage runs its layers or steps in one call.
// A small round spends its time here: submitting one attention call took 16.6
// us through ctypes (the kernel of a short batch takes 5 to 12), a four-call
// round 42 us.
//
// Every function returns None, having enqueued nothing, for arguments it does
// not take (another type of argument, a tensor that fails a check); the Python
// caller then goes through its own checks, which name the fault.  Library
// errors come back as (entry point, status).
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "nebulasd.h"

namespace {

using at::Tensor;

// Entry points of the loaded library, set once by bind().
struct Api {
  decltype(&nsd_kv_gather) kv_gather;
  decltype(&nsd_verify_attention) verify_attention;
  decltype(&nsd_gather_verify_attention) gather_verify_attention;
  decltype(&nsd_verify_attention_workspace_size) attention_ws;
  decltype(&nsd_spec_accept) spec_accept;
  decltype(&nsd_spec_accept_workspace_size) accept_ws;
  decltype(&nsd_sample) sample;
  decltype(&nsd_kv_append) kv_append;
  decltype(&nsd_commit_lengths) commit_lengths;
  decltype(&nsd_kv_append_layers) kv_append_layers;
  decltype(&nsd_spec_accept_commit) spec_accept_commit;
  decltype(&nsd_sample_steps) sample_steps;
} api;

// Thrown (before anything is enqueued) for arguments the Python path handles.
struct NotHere {};
// A library call's error.
struct Failed {
  const char* fn;
  nsd_status status;
};

void check(const char* fn, nsd_status st) {
  if (st != NSD_OK) throw Failed{fn, st};
}

const Tensor& any_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotHere();
  return THPVariable_Unpack(o);
}

const Tensor& tensor(PyObject* o, at::ScalarType type) {
  const Tensor& t = any_tensor(o);
  if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous()) throw NotHere();
  return t;
}

const Tensor& bf16(PyObject* o) { return tensor(o, at::kBFloat16); }
const Tensor& i32(PyObject* o) { return tensor(o, at::kInt); }
const Tensor& f32(PyObject* o) { return tensor(o, at::kFloat); }

int32_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw NotHere();
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) throw NotHere();
  return (int32_t)v;
}

void need(bool ok) {
  if (!ok) throw NotHere();
}

int32_t small(int64_t v) {
  need(v >= 0 && v <= INT32_MAX);
  return (int32_t)v;
}

void* stream_of(const Tensor& t) {
  return (void*)c10::hip::getCurrentHIPStream(t.device().index()).stream();
}

float scale_of(PyObject* o, int64_t head_dim) {
  if (o == Py_None) return (float)(1.0 / std::sqrt((double)head_dim));
  if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
  throw NotHere();
}

// The caller's workspace, or a new one of `bytes`, kept alive by `own`.
const Tensor& workspace(PyObject* o, const Tensor& like, size_t bytes, Tensor& own) {
  if (o == Py_None) {
    own = at::empty({(int64_t)std::max<size_t>(bytes, 16)}, like.options().dtype(at::kByte));
    return own;
  }
  const Tensor& t = tensor(o, at::kByte);
  need(t.device() == like.device());
  return t;
}

// The caller's output, or a new one like `like`.
Tensor output(PyObject* o, at::ScalarType type, at::IntArrayRef shape, const Tensor& like) {
  if (o == Py_None) return at::empty(shape, like.options().dtype(type));
  const Tensor& t = tensor(o, type);
  need(t.sizes() == shape);
  return t;
}

// One layer's paged planes.
struct Planes {
  char* k;
  char* v;
  int64_t blocks;
  int64_t layer_bytes;   // between layers of a stacked pool
};

// Batch metadata and head geometry of an attention call, checked.
struct Batch {
  const int32_t *table, *stage, *lens, *indptr;
  int32_t bs, width, hq, hkv, d, max_q, max_len;
  float scale;
  char* ws;
  size_t ws_bytes;
  void* stream;
};

// Pool planes [layers][blocks][Hkv][D/8][16][8] and [layers][blocks][Hkv][D][16]
// (stacked) or one layer's, as head geometry hkv, d.
Planes planes(const Tensor& k, const Tensor& v, bool stacked, int64_t hkv, int64_t d) {
  const int o = stacked ? 1 : 0;
  need(k.dim() == 5 + o && v.dim() == 4 + o);
  if (stacked) need(k.size(0) == v.size(0));
  need(k.size(o) == v.size(o) && k.size(o + 1) == hkv && v.size(o + 1) == hkv &&
       k.size(o + 2) * k.size(o + 4) == d && k.size(o + 3) == NSD_BLOCK_SIZE &&
       k.size(o + 4) == 8 && v.size(o + 2) == d && v.size(o + 3) == NSD_BLOCK_SIZE);
  return Planes{(char*)k.data_ptr(), (char*)v.data_ptr(), k.size(o),
                k.size(o) * hkv * d * NSD_BLOCK_SIZE * 2};
}

Planes at_layer(const Planes& p, int64_t layer) {
  return Planes{p.k + layer * p.layer_bytes, p.v + layer * p.layer_bytes, p.blocks,
                p.layer_bytes};
}

void metadata(Batch& b, PyObject* table, PyObject* lens, PyObject* indptr, PyObject* max_q,
              PyObject* max_len) {
  const Tensor &t = i32(table), &l = i32(lens), &q = i32(indptr);
  b.bs = small(l.numel());
  need(t.dim() == 2 && t.size(0) == b.bs && q.numel() == (int64_t)b.bs + 1);
  b.width = small(t.size(1));
  b.table = t.data_ptr<int32_t>();
  b.stage = nullptr;
  b.lens = l.data_ptr<int32_t>();
  b.indptr = q.data_ptr<int32_t>();
  b.max_q = integer(max_q);
  b.max_len = integer(max_len);
}

void stage_table(Batch& b, PyObject* o) {
  const Tensor& t = i32(o);
  need(t.dim() == 2 && t.size(0) == b.bs && t.size(1) == b.width);
  b.stage = t.data_ptr<int32_t>();
}

size_t attention_ws(const Batch& b) {
  return api.attention_ws(b.bs, b.hq, b.hkv, b.d, b.max_q, b.max_len);
}

void attend(const Batch& b, const char* q, const Planes& pool, char* out) {
  check("verify_attention",
        api.verify_attention(q, pool.k, pool.v, pool.blocks, b.table, b.width, b.lens, b.indptr,
                             b.bs, b.hq, b.hkv, b.d, NSD_BLOCK_SIZE, b.max_q, b.max_len, b.scale,
                             out, b.ws, b.ws_bytes, b.stream));
}

void attend_fused(const Batch& b, const char* q, const Planes& pool, const Planes& stage,
                  char* out) {
  check("gather_verify_attention",
        api.gather_verify_attention(q, pool.k, pool.v, pool.blocks, stage.k, stage.v, stage.blocks,
                                    b.table, b.stage, b.width, b.lens, b.indptr, b.bs, b.hq,
                                    b.hkv, b.d, NSD_BLOCK_SIZE, b.max_q, b.max_len, b.scale, out,
                                    b.ws, b.ws_bytes, b.stream));
}

void append(const Planes& pool, const char* kn, const char* vn, const int32_t* table,
            int32_t width, const int32_t* lens, const Batch& b, int32_t total_q) {
  check("kv_append",
        api.kv_append(pool.k, pool.v, pool.blocks, kn, vn, table, width, lens, b.indptr, b.bs,
                      total_q, b.hkv, NSD_BLOCK_SIZE, b.d, b.stream));
}

// The window rows of a round's layers, into the pool and (fused preparation) the
// staging bank.
void append_layers(const Batch& b, const Planes& pool, const int32_t* pool_table,
                   const Planes& stage, const int32_t* stage_rows, int32_t layers,
                   const void* const* kn, const void* const* vn, int32_t total_q) {
  check("kv_append_layers",
        api.kv_append_layers(pool.k, pool.v, pool.blocks, pool_table, stage.k, stage.v,
                             stage.blocks, stage_rows, layers, kn, vn, b.width, b.lens, b.indptr,
                             b.bs, total_q, b.hkv, NSD_BLOCK_SIZE, b.d, b.stream));
}

// Runs f without the interpreter lock; library errors become (entry point, status).
template <class F>
PyObject* unlocked(F f, PyObject* (*result)(void*), void* arg) {
  Failed failed{nullptr, NSD_OK};
  Py_BEGIN_ALLOW_THREADS
  try {
    f();
  } catch (const Failed& e) {
    failed = e;
  }
  Py_END_ALLOW_THREADS
  if (failed.fn) return Py_BuildValue("(si)", failed.fn, (int)failed.status);
  return result(arg);
}

PyObject* yes(void*) { Py_RETURN_TRUE; }
PyObject* wrap(void* t) { return THPVariable_Wrap(*(Tensor*)t); }
PyObject* wrap2(void* t) {
  PyObject* a = THPVariable_Wrap(((Tensor*)t)[0]);
  PyObject* b = THPVariable_Wrap(((Tensor*)t)[1]);
  return Py_BuildValue("[NN]", a, b);
}

// The body of an entry point: whatever it does not take comes back as None.
template <class F>
PyObject* entry(F f) {
  try {
    return f();
  } catch (const NotHere&) {
  } catch (const std::exception&) {   // torch's own checks: the Python path reports them
  }
  Py_RETURN_NONE;
}

PyObject* py_verify_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // q, k, v, table, lens, indptr, max_q, max_len, scale, out, workspace
  return entry([&]() -> PyObject* {
    need(n == 11);
    const Tensor& q = bf16(a[0]);
    need(q.dim() == 3);
    const Tensor& k = bf16(a[1]);
    need(k.dim() == 5);
    Batch b;
    b.hq = small(q.size(1));
    b.d = small(q.size(2));
    b.hkv = small(k.size(1));
    const Planes pool = planes(k, bf16(a[2]), false, b.hkv, b.d);
    metadata(b, a[3], a[4], a[5], a[6], a[7]);
    b.scale = scale_of(a[8], b.d);
    Tensor out = output(a[9], at::kBFloat16, q.sizes(), q), own;
    const Tensor& ws = workspace(a[10], q, a[10] == Py_None ? attention_ws(b) : 0, own);
    b.ws = (char*)ws.data_ptr();
    b.ws_bytes = ws.numel();
    b.stream = stream_of(q);
    char *qp = (char*)q.data_ptr(), *op = (char*)out.data_ptr();
    return unlocked([&] { attend(b, qp, pool, op); }, wrap, &out);
  });
}

PyObject* py_gather_verify_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // q, k, v, k_stage, v_stage, table, stage_table, lens, indptr, max_q, max_len, scale, out, ws
  return entry([&]() -> PyObject* {
    need(n == 14);
    const Tensor& q = bf16(a[0]);
    need(q.dim() == 3);
    const Tensor& k = bf16(a[1]);
    need(k.dim() == 5);
    Batch b;
    b.hq = small(q.size(1));
    b.d = small(q.size(2));
    b.hkv = small(k.size(1));
    const Planes pool = planes(k, bf16(a[2]), false, b.hkv, b.d);
    const Planes stage = planes(bf16(a[3]), bf16(a[4]), false, b.hkv, b.d);
    metadata(b, a[5], a[7], a[8], a[9], a[10]);
    stage_table(b, a[6]);
    b.scale = scale_of(a[11], b.d);
    Tensor out = output(a[12], at::kBFloat16, q.sizes(), q), own;
    const Tensor& ws = workspace(a[13], q, a[13] == Py_None ? attention_ws(b) : 0, own);
    b.ws = (char*)ws.data_ptr();
    b.ws_bytes = ws.numel();
    b.stream = stream_of(q);
    char *qp = (char*)q.data_ptr(), *op = (char*)out.data_ptr();
    return unlocked([&] { attend_fused(b, qp, pool, stage, op); }, wrap, &out);
  });
}

// Acceptance inputs, checked.
struct Accept {
  const float *p, *q, *u;
  const int32_t *x, *indptr;
  int32_t bs, vocab, max_k;
  int32_t *len, *tok;
  void* ws;
  size_t ws_bytes;
  void* stream;
  Tensor out[2], own;
};

void accept_args(Accept& s, PyObject* p_, PyObject* q_, PyObject* x_, PyObject* u_,
                 const Tensor& indptr, PyObject* k_, PyObject* len_, PyObject* tok_,
                 PyObject* ws_) {
  const Tensor &p = f32(p_), &u = f32(u_);
  need(p.dim() == 2);
  s.max_k = integer(k_);
  s.vocab = small(p.size(1));
  s.bs = small(indptr.numel() - 1);
  const int64_t total = p.size(0);
  need(u.numel() == total);
  s.q = nullptr;
  s.x = nullptr;
  if (s.max_k > 0) {
    const Tensor &q = f32(q_), &x = i32(x_);
    need(q.dim() == 2 && q.size(0) == total - s.bs && q.size(1) == s.vocab &&
         x.numel() == total - s.bs);
    s.q = q.data_ptr<float>();
    s.x = x.data_ptr<int32_t>();
  }
  s.p = p.data_ptr<float>();
  s.u = u.data_ptr<float>();
  s.indptr = indptr.data_ptr<int32_t>();
  if (len_ != Py_None) need(any_tensor(len_).dim() == 1);
  if (tok_ != Py_None) need(any_tensor(tok_).dim() == 1);
  s.out[0] = output(len_, at::kInt, {s.bs}, p);
  s.out[1] = output(tok_, at::kInt, {total}, p);
  s.len = s.out[0].data_ptr<int32_t>();
  s.tok = s.out[1].data_ptr<int32_t>();
  const Tensor& ws = workspace(ws_, p, ws_ == Py_None ? api.accept_ws(s.bs, s.vocab) : 0, s.own);
  s.ws = ws.data_ptr();
  s.ws_bytes = ws.numel();
  s.stream = stream_of(p);
}

void accept(const Accept& s) {
  check("spec_accept", api.spec_accept(s.p, s.q, s.x, s.u, s.indptr, s.bs, s.vocab, s.max_k,
                                       s.len, s.tok, s.ws, s.ws_bytes, s.stream));
}

PyObject* py_spec_accept(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // p, q, x, u, indptr, max_k, accepted_len, out_tokens, workspace
  return entry([&]() -> PyObject* {
    need(n == 9);
    Accept s;
    accept_args(s, a[0], a[1], a[2], a[3], i32(a[4]), a[5], a[6], a[7], a[8]);
    return unlocked([&] { accept(s); }, wrap2, s.out);
  });
}

PyObject* py_sample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // probs, uniforms, out, workspace
  return entry([&]() -> PyObject* {
    need(n == 4);
    const Tensor& p = any_tensor(a[0]);
    need(p.scalar_type() == at::kFloat && p.is_cuda() && p.dim() == 2);
    const int32_t rows = small(p.size(0)), vocab = small(p.size(1));
    need((rows <= 1 || p.stride(0) >= vocab) && (vocab <= 1 || p.stride(1) == 1));
    const Tensor& u = f32(a[1]);
    need(u.numel() == rows);
    Tensor out, own;
    if (a[2] == Py_None) {
      out = at::empty({rows}, p.options().dtype(at::kInt));
    } else {
      out = any_tensor(a[2]);
      need(out.scalar_type() == at::kInt && out.is_cuda() && out.dim() == 1 &&
           out.numel() == rows);
    }
    const Tensor& ws = workspace(a[3], p, a[3] == Py_None ? api.accept_ws(rows, vocab) : 0, own);
    const float *pp = p.data_ptr<float>(), *up = u.data_ptr<float>();
    const int64_t stride = rows > 1 ? p.stride(0) : vocab;
    const int32_t ostride = small(std::max<int64_t>(1, out.stride(0)));
    int32_t* op = out.data_ptr<int32_t>();
    void *wp = ws.data_ptr(), *st = stream_of(p);
    const size_t wn = ws.numel();
    return unlocked(
        [&] { check("sample", api.sample(pp, stride, up, rows, vocab, op, ostride, wp, wn, st)); },
        wrap, &out);
  });
}

// Geometry of stacked gather planes.
struct Gather {
  Planes src, dst;
  int32_t layers, hkv, d;
  const int32_t *sid, *did;
  int64_t pairs;
};

Gather gather_args(const Tensor& sk, const Tensor& sv, const Tensor& dk, const Tensor& dv,
                   PyObject* src_ids, PyObject* dst_ids) {
  Gather g;
  const int o = dk.dim() == 6 ? 1 : 0;   // stacked, or one layer's planes
  need(dk.dim() == 5 + o && sk.dim() == 5 + o && (!o || sk.size(0) == dk.size(0)));
  g.layers = o ? small(dk.size(0)) : 1;
  g.hkv = small(dk.size(o + 1));
  g.d = small(dk.size(o + 2) * dk.size(o + 4));
  g.src = planes(sk, sv, o, g.hkv, g.d);
  g.dst = planes(dk, dv, o, g.hkv, g.d);
  const Tensor &s = i32(src_ids), &t = i32(dst_ids);
  need(s.numel() == t.numel());
  g.sid = s.data_ptr<int32_t>();
  g.did = t.data_ptr<int32_t>();
  g.pairs = s.numel();
  return g;
}

void gather(const Gather& g, int32_t layer0, int32_t n, void* stream) {
  check("kv_gather", api.kv_gather(g.src.k, g.src.v, g.src.blocks, g.dst.k, g.dst.v, g.dst.blocks,
                                   g.sid, g.did, g.pairs, g.layers, layer0, n, g.hkv,
                                   NSD_BLOCK_SIZE, g.d, stream));
}

PyObject* py_kv_gather(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // src_k, src_v, dst_k, dst_v, src_ids, dst_ids, layer0, n_layers
  return entry([&]() -> PyObject* {
    need(n == 8);
    const Gather g = gather_args(bf16(a[0]), bf16(a[1]), bf16(a[2]), bf16(a[3]), a[4], a[5]);
    const int32_t l0 = integer(a[6]);
    need(l0 >= 0);   // (g.layers - l0 cannot overflow; the Python path names the fault)
    const int32_t nl = a[7] == Py_None ? g.layers - l0 : integer(a[7]);
    void* st = stream_of(any_tensor(a[0]));
    return unlocked([&] { gather(g, l0, nl, st); }, yes, nullptr);
  });
}

PyObject* py_kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // k_pool, v_pool, k_new, v_new, table, lens, indptr
  return entry([&]() -> PyObject* {
    need(n == 7);
    const Tensor &kn = bf16(a[2]), &vn = bf16(a[3]), &k = bf16(a[0]);
    need(kn.dim() == 3 && vn.sizes() == kn.sizes());
    Batch b;
    b.hkv = small(kn.size(1));
    b.d = small(kn.size(2));
    const Planes pool = planes(k, bf16(a[1]), false, b.hkv, b.d);
    const Tensor &t = i32(a[4]), &l = i32(a[5]), &q = i32(a[6]);
    b.bs = small(l.numel());
    need(t.dim() == 2 && t.size(0) == b.bs && q.numel() == (int64_t)b.bs + 1);
    b.indptr = q.data_ptr<int32_t>();
    b.stream = stream_of(k);
    const int32_t total = small(kn.size(0)), width = small(t.size(1));
    char *kp = (char*)kn.data_ptr(), *vp = (char*)vn.data_ptr();
    const int32_t *tp = t.data_ptr<int32_t>(), *lp = l.data_ptr<int32_t>();
    return unlocked([&] { append(pool, kp, vp, tp, width, lp, b, total); }, yes, nullptr);
  });
}

PyObject* py_commit_lengths(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // lens, indptr, accepted_len, out
  return entry([&]() -> PyObject* {
    need(n == 4);
    const Tensor &l = i32(a[0]), &q = i32(a[1]), &acc = i32(a[2]);
    const int32_t bs = small(l.numel());
    need(q.numel() == (int64_t)bs + 1 && acc.numel() == bs);
    Tensor out = a[3] == Py_None ? at::empty_like(l) : i32(a[3]);
    need(out.numel() == bs);
    const int32_t *lp = l.data_ptr<int32_t>(), *qp = q.data_ptr<int32_t>(),
                  *ap = acc.data_ptr<int32_t>();
    int32_t* op = out.data_ptr<int32_t>();
    void* st = stream_of(l);
    return unlocked([&] { check("commit_lengths", api.commit_lengths(lp, qp, ap, op, bs, st)); },
                    wrap, &out);
  });
}

// References to the tensors inside a call's tuples and lists: the call runs without
// the interpreter lock, and a list's owner may change it meanwhile.
using Held = std::vector<Tensor>;

const Tensor& held(Held& h, const Tensor& t) {
  h.push_back(t);
  return t;
}

// A tuple or list of n items, or NotHere.
PyObject** items_of(PyObject* o, Py_ssize_t n) {
  if (!PyTuple_CheckExact(o) && !PyList_CheckExact(o)) throw NotHere();
  need(n < 0 || PySequence_Fast_GET_SIZE(o) == n);
  return PySequence_Fast_ITEMS(o);
}

PyObject* py_verify_round(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // 0 k_pool 1 v_pool 2 k_stage 3 v_stage 4 src_ids 5 dst_ids 6 q 7 table 8 lens 9 indptr
  // 10 max_q 11 max_len 12 accept 13 out 14 workspace 15 scale 16 stage_table (None: gather)
  // 17 window_kv 18 committed 19 append tables (fused window) 20 accept workspace
  return entry([&]() -> PyObject* {
    need(n == 21);
    const Tensor &k = bf16(a[0]), &v = bf16(a[1]), &q = bf16(a[6]), &out = bf16(a[13]);
    need(k.dim() == 6 && q.dim() == 4 && q.size(0) >= k.size(0) && out.sizes() == q.sizes());
    const int64_t layers = k.size(0);
    Batch b;
    b.hq = small(q.size(2));
    b.d = small(q.size(3));
    b.hkv = small(k.size(2));
    const int32_t total = small(q.size(1));
    const Planes pool = planes(k, v, true, b.hkv, b.d);
    metadata(b, a[7], a[8], a[9], a[10], a[11]);
    b.scale = scale_of(a[15], b.d);
    const Tensor& ws = tensor(a[14], at::kByte);
    need(ws.device() == q.device());
    b.ws = (char*)ws.data_ptr();
    b.ws_bytes = ws.numel();
    b.stream = stream_of(q);
    const bool fused = a[16] != Py_None;
    const Tensor &ks = bf16(a[2]), &vs = bf16(a[3]);
    need(k.device() == q.device() && ks.device() == q.device());
    Planes stage{nullptr, nullptr, 0, 0};
    Gather g;
    if (fused) {
      stage_table(b, a[16]);
      stage = planes(ks, vs, true, b.hkv, b.d);
      need(ks.size(0) >= layers);
    } else {
      g = gather_args(ks, vs, k, v, a[4], a[5]);
    }
    Held h;
    std::vector<const void*> k_new, v_new;
    const int32_t *pool_table = b.table, *stage_rows = nullptr;
    if (a[17] != Py_None) {
      PyObject** rows = items_of(a[17], -1);
      need(PySequence_Fast_GET_SIZE(a[17]) >= layers);
      for (int64_t l = 0; l < layers; ++l) {
        PyObject** kv = items_of(rows[l], 2);
        const Tensor &kn = held(h, bf16(kv[0])), &vn = held(h, bf16(kv[1]));
        need(kn.dim() == 3 && kn.size(0) == total && kn.size(1) == b.hkv && kn.size(2) == b.d &&
             vn.sizes() == kn.sizes());
        k_new.push_back(kn.data_ptr());
        v_new.push_back(vn.data_ptr());
      }
      if (fused) {
        PyObject** tables = items_of(a[19], 2);
        const Tensor &pt = held(h, i32(tables[0])), &sr = held(h, i32(tables[1]));
        need(pt.dim() == 2 && pt.size(0) == b.bs && pt.size(1) == b.width &&
             sr.sizes() == pt.sizes());
        pool_table = pt.data_ptr<int32_t>();
        stage_rows = sr.data_ptr<int32_t>();
      }
    }
    Accept s;
    const bool accepts = a[12] != Py_None;
    int32_t* committed = nullptr;
    if (accepts) {
      PyObject** in = items_of(a[12], 5);
      accept_args(s, in[0], in[1], in[2], in[3], i32(a[9]), in[4], Py_None, Py_None, a[20]);
      need(any_tensor(in[0]).device() == q.device());
      for (int i : {0, 1, 2, 3})
        if (s.max_k > 0 || i % 3 == 0) held(h, any_tensor(in[i]));   // (no draft rows without K)
      if (a[18] != Py_None) {
        const Tensor& c = i32(a[18]);
        need(c.numel() == b.bs);
        committed = c.data_ptr<int32_t>();
      }
    }
    const char* qp = (const char*)q.data_ptr();
    char* op = (char*)out.data_ptr();
    const int64_t rows = (int64_t)total * b.hq * b.d * 2;
    return unlocked(
        [&] {
          if (!fused) gather(g, 0, g.layers, b.stream);
          // every layer's rows are in hand: one launch appends them all
          if (!k_new.empty())
            append_layers(b, pool, pool_table, stage, stage_rows, (int32_t)layers, k_new.data(),
                          v_new.data(), total);
          for (int64_t l = 0; l < layers; ++l) {
            const Planes here = at_layer(pool, l);
            if (fused)
              attend_fused(b, qp + l * rows, here, at_layer(stage, l), op + l * rows);
            else
              attend(b, qp + l * rows, here, op + l * rows);
          }
          if (committed)
            check("spec_accept_commit",
                  api.spec_accept_commit(s.p, s.q, s.x, s.u, s.indptr, s.bs, s.vocab, s.max_k,
                                         s.len, s.tok, b.lens, committed, s.ws, s.ws_bytes,
                                         s.stream));
          else if (accepts)
            accept(s);
        },
        accepts ? wrap2 : yes, s.out);
  });
}

PyObject* py_draft_stage(PyObject*, PyObject* const* a, Py_ssize_t n) {
  // 0 k_pool 1 v_pool 2 q 3 k_new 4 v_new 5 probs 6 uniforms 7 table 8 lens [K][bs] 9 indptr
  // 10 max_len 11 k_stage 12 v_stage 13 stage_table (None: prepared already) 14 tokens 15 out
  // 16 workspace 17 scale 18 append tables 19 sample workspace
  return entry([&]() -> PyObject* {
    need(n == 20);
    const Tensor &k = bf16(a[0]), &q = bf16(a[2]), &kn = bf16(a[3]), &vn = bf16(a[4]);
    const Tensor &p = f32(a[5]), &u = f32(a[6]), &t = i32(a[7]), &l = i32(a[8]), &qi = i32(a[9]);
    const Tensor &tok = i32(a[14]), &out = bf16(a[15]);
    need(q.dim() == 4 && kn.dim() == 4 && l.dim() == 2 && k.dim() == 5);
    const int64_t steps = l.size(0);
    Batch b;
    b.bs = small(l.size(1));
    b.hq = small(q.size(2));
    b.d = small(q.size(3));
    b.hkv = small(k.size(1));
    const Planes pool = planes(k, bf16(a[1]), false, b.hkv, b.d);
    need(q.size(0) >= steps && q.size(1) == b.bs && out.sizes() == q.sizes() &&
         kn.size(0) >= steps && kn.size(1) == b.bs && kn.size(2) == b.hkv &&
         kn.size(3) == b.d && vn.sizes() == kn.sizes());
    need(t.dim() == 2 && t.size(0) == b.bs && qi.numel() == (int64_t)b.bs + 1);
    need(p.dim() == 3 && p.size(0) == b.bs && p.size(1) >= steps && u.dim() == 2 &&
         u.size(0) >= steps && u.size(1) == b.bs && tok.dim() == 2 && tok.size(0) == b.bs &&
         tok.size(1) == p.size(1));
    b.width = small(t.size(1));
    b.table = t.data_ptr<int32_t>();
    b.stage = nullptr;
    b.indptr = qi.data_ptr<int32_t>();
    b.max_q = 1;
    b.max_len = integer(a[10]);
    b.scale = scale_of(a[17], b.d);
    const Tensor &ws = tensor(a[16], at::kByte), &sws = tensor(a[19], at::kByte);
    need(ws.device() == q.device() && sws.device() == q.device() && p.device() == q.device() &&
         k.device() == q.device());
    b.ws = (char*)ws.data_ptr();
    b.ws_bytes = ws.numel();
    b.stream = stream_of(q);
    Planes stage{nullptr, nullptr, 0, 0};
    Held h;
    const int32_t *pool_table = nullptr, *stage_rows = nullptr;
    const bool fused = a[13] != Py_None;
    if (fused) {
      stage_table(b, a[13]);
      stage = planes(bf16(a[11]), bf16(a[12]), false, b.hkv, b.d);
      PyObject** tables = items_of(a[18], 2);
      const Tensor &pt = held(h, i32(tables[0])), &sr = held(h, i32(tables[1]));
      need(pt.dim() == 2 && pt.size(0) == b.bs && pt.size(1) == b.width &&
           sr.sizes() == pt.sizes());
      pool_table = pt.data_ptr<int32_t>();
      stage_rows = sr.data_ptr<int32_t>();
    }
    const char *qp = (const char*)q.data_ptr(), *kp = (const char*)kn.data_ptr(),
               *vp = (const char*)vn.data_ptr();
    char *op = (char*)out.data_ptr(), *swp = (char*)sws.data_ptr();
    const size_t swn = sws.numel();
    const float *pp = p.data_ptr<float>(), *up = u.data_ptr<float>();
    const int32_t* lp = l.data_ptr<int32_t>();
    int32_t* tp = tok.data_ptr<int32_t>();
    const int32_t vocab = small(p.size(2)), ostride = small(std::max<int64_t>(1, p.size(1)));
    const int64_t row = p.size(1) * vocab;
    // the draws of all steps in one launch, at the end, if a workspace holds
    // their sums (the attention's is free by then): for 64 requests x 4 steps at
    // vocab 151936 four launch pairs of 13.3 us -> one launch of 27.1 us
    const size_t need_ws = api.accept_ws(small(b.bs * steps), vocab);
    void* all_ws = swn >= need_ws ? (void*)swp : b.ws_bytes >= need_ws ? (void*)b.ws : nullptr;
    const size_t all_wn = swn >= need_ws ? swn : b.ws_bytes;
    // (a sample workspace that one step's draw refuses is still refused, there)
    if ((uintptr_t)all_ws % 8 || b.bs * steps > (1 << 20) || (uintptr_t)swp % 8 ||
        swn < api.accept_ws(b.bs, vocab))
      all_ws = nullptr;
    const int64_t qb = (int64_t)b.bs * b.hq * b.d * 2, nb = (int64_t)b.bs * b.hkv * b.d * 2;
    return unlocked(
        [&] {
          for (int64_t i = 0; i < steps; ++i) {
            b.lens = lp + i * b.bs;
            if (fused && i == 0) {
              const void *k0 = kp, *v0 = vp;
              append_layers(b, pool, pool_table, stage, stage_rows, 1, &k0, &v0, b.bs);
              attend_fused(b, qp, pool, stage, op);
            } else {
              append(pool, kp + i * nb, vp + i * nb, b.table, b.width, b.lens, b, b.bs);
              attend(b, qp + i * qb, pool, op + i * qb);
            }
            if (all_ws) continue;
            check("sample", api.sample(pp + i * vocab, b.bs > 1 ? row : vocab, up + i * b.bs, b.bs,
                                       vocab, tp + i, ostride, swp, swn, b.stream));
          }
          if (all_ws && steps > 0)
            check("sample", api.sample_steps(pp, row, up, b.bs, (int32_t)steps, vocab, tp, ostride,
                                             all_ws, all_wn, b.stream));
        },
        yes, nullptr);
  });
}

// bind(addresses): the library's entry points, in the order of Api.
PyObject* py_bind(PyObject*, PyObject* addresses) {
  void** to = (void**)&api;
  const Py_ssize_t n = sizeof(Api) / sizeof(void*);
  if (!PyTuple_CheckExact(addresses) || PyTuple_GET_SIZE(addresses) != n) {
    PyErr_SetString(PyExc_ValueError, "bind: one address per entry point");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    void* p = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (!p) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: NULL address");
      return nullptr;
    }
    to[i] = p;
  }
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(verify_attention),
                         FAST(gather_verify_attention),
                         FAST(spec_accept),
                         FAST(sample),
                         FAST(kv_gather),
                         FAST(kv_append),
                         FAST(commit_lengths),
                         FAST(verify_round),
                         FAST(draft_stage),
                         {"bind", py_bind, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
#undef FAST

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nsd_torch", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nsd_torch() { return PyModule_Create(&module); }
