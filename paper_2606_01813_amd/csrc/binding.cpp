// The Python binding's calls, natively: checks the tensors of a call against the plan, as the Python
// checks do, and calls the library.
//
// A call's checks look at up to thirteen tensors.  Through the tensors' Python attributes they cost more
// than the kernels of a small round: 16 of the 22 us of host time of a build, 30 of the 37 us of the three
// stage calls.  Here a call takes about 1 us besides the launches.
//
// A function returns the library's status, or None when it cannot vouch for every argument: then the
// caller takes the Python path, which decides (and raises) as it always did.  Nothing is kept from one
// call to the next.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <initializer_list>

#include "caddtree.h"

namespace {

// What the checks need of a plan, and the library's functions (ctypes has loaded them).
struct Spec {
  caddtree_plan_t plan;
  int device;            // GPU index; -1: host tensors (tests of the checks themselves)
  int64_t L, V, K, cap;  // cap at least 1, as the outputs are shaped
  c10::ScalarType dtype;
  int mask;              // caddtree_mask_t
  decltype(&caddtree_build) build;
  decltype(&caddtree_build_noalloc) build_noalloc;
  decltype(&caddtree_reduce_topk) reduce_topk;
  decltype(&caddtree_expand) expand;
  decltype(&caddtree_emit) emit;
  decltype(&caddtree_accept) accept;
};

// One call's view of its arguments: ok falls, and stays down, at the first one that is not as it should be.
struct Call {
  const Spec& s;
  bool ok = true;
  PyObject* held[16];    // attributes fetched from an outputs object, until the call returns
  int n_held = 0;

  explicit Call(const Spec& spec) : s(spec) {}
  ~Call() {
    for (int i = 0; i < n_held; ++i) Py_DECREF(held[i]);
  }
  Call(const Call&) = delete;
  Call& operator=(const Call&) = delete;

  PyObject* attr(PyObject* o, PyObject* name) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (v == nullptr) {
      PyErr_Clear();
      ok = false;
      return Py_None;
    }
    held[n_held++] = v;
    return v;
  }

  // the tensor behind o: exactly a torch.Tensor, strided, with storage, on the plan's device
  c10::TensorImpl* tensor(PyObject* o) {
    if (!ok || !THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    c10::TensorImpl* t = THPVariable_Unpack(o).unsafeGetTensorImpl();
    const c10::Device d = t->device();
    const bool here = s.device >= 0 ? d.is_cuda() && d.index() == s.device : d.is_cpu();
    if (!here || t->layout() != c10::kStrided || !t->has_storage() || t->has_symbolic_sizes_strides()) {
      ok = false;
      return nullptr;
    }
    return t;
  }

  // a contiguous tensor of `type`, shaped [>= B, dims...]; None gives nullptr unless it is required
  void* data(PyObject* o, c10::ScalarType type, std::initializer_list<int64_t> dims, int64_t B, bool required) {
    if (o == Py_None) {
      if (required) ok = false;
      return nullptr;
    }
    c10::TensorImpl* t = tensor(o);
    if (t == nullptr) return nullptr;
    const auto sz = t->sizes();
    bool good = c10::typeMetaToScalarType(t->dtype()) == type && sz.size() == 1 + dims.size() && sz[0] >= B &&
                t->is_contiguous();
    size_t i = 1;
    if (good)
      for (const int64_t d : dims) good = good && sz[i++] == d;
    if (!good || t->numel() == 0) {
      ok = false;
      return nullptr;
    }
    return t->mutable_data();
  }

  // rows (b, i) at element (b L + i) stride
  void* logits(PyObject* o, int64_t* B, int64_t* stride) {
    c10::TensorImpl* t = tensor(o);
    if (t == nullptr) return nullptr;
    const auto sz = t->sizes();
    if (c10::typeMetaToScalarType(t->dtype()) != s.dtype || sz.size() != 3 || sz[1] != s.L || sz[2] < s.V ||
        t->numel() == 0) {
      ok = false;
      return nullptr;
    }
    const auto st = t->strides();
    int64_t rs;
    bool good = true;
    if (s.L > 1) {
      rs = st[1];
      good = sz[0] == 1 || st[0] == rs * s.L;
    } else {
      rs = sz[0] > 1 ? st[0] : sz[2];
    }
    if (sz[2] > 1 && st[2] != 1) good = false;
    if (!good || rs < s.V) {
      ok = false;
      return nullptr;
    }
    *B = sz[0];
    *stride = rs;
    return const_cast<void*>(t->data());
  }

  int64_t rows(PyObject* o) {
    c10::TensorImpl* t = tensor(o);
    if (t == nullptr || t->sizes().empty()) {
      ok = false;
      return 0;
    }
    return t->sizes()[0];
  }

  const int64_t* ctx(PyObject* o, int64_t B) {
    if (o == Py_None) return nullptr;
    void* p = data(o, c10::kLong, {}, B, true);
    if (ok && rows(o) != B) ok = false;
    return static_cast<const int64_t*>(p);
  }

  void* mask(PyObject* o, int64_t B) {
    if (s.mask == CADDTREE_MASK_U8) return data(o, c10::kByte, {s.cap, s.cap}, B, false);
    if (o == Py_None) return nullptr;
    if (s.mask == CADDTREE_MASK_BITS32) {
      c10::TensorImpl* t = tensor(o);
      if (t == nullptr) return nullptr;
      const c10::ScalarType type = c10::typeMetaToScalarType(t->dtype());
      if (type != c10::kInt && type != c10::kUInt32) {
        ok = false;
        return nullptr;
      }
      return data(o, type, {s.cap, (s.cap + 31) / 32}, B, false);
    }
    ok = false;           // a mask for a plan without one: the Python path decides
    return nullptr;
  }

  int64_t integer(PyObject* o, int64_t lo, int64_t hi) {
    int over = 0;
    const long long v = PyLong_CheckExact(o) ? PyLong_AsLongLongAndOverflow(o, &over) : lo - 1;
    if (over != 0 || v < lo || v > hi) ok = false;
    return v;
  }
  int32_t offset(PyObject* o) { return (int32_t)integer(o, INT32_MIN, INT32_MAX); }
  hipStream_t stream(PyObject* o) {
    const unsigned long long v = PyLong_CheckExact(o) ? PyLong_AsUnsignedLongLong(o) : 0;
    if (!PyLong_CheckExact(o) || PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(v));
  }
};

// the attributes of an outputs object
enum Field { kTokenIds, kParent, kDepth, kPathProb, kNStar, kPhi, kTheta, kMask, kPosIds, kTopkIds, kTopkLogit,
             kTopkLq, kLse, kFields };
const char* const kNames[kFields] = {"token_ids", "parent", "depth", "path_prob", "n_star", "phi", "theta",
                                     "mask", "pos_ids", "topk_ids", "topk_logit", "topk_lq", "lse"};
PyObject* g_name[kFields];   // interned

template <typename T>
T* as(void* p) { return static_cast<T*>(p); }

const char* const kSpecName = "caddtree.spec";

// an exception came out of the library's call, whose work may be enqueued already: not to be called again
struct LibraryThrew {};

template <typename F>
PyObject* guarded(PyObject* const* args, Py_ssize_t nargs, Py_ssize_t want, F&& body) {
  if (nargs != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, nargs);
    return nullptr;
  }
  const Spec* s = static_cast<const Spec*>(PyCapsule_GetPointer(args[0], kSpecName));
  if (s == nullptr) return nullptr;
  int status = -1;
  try {
    status = body(*s);
  } catch (const LibraryThrew&) {
    PyErr_SetString(PyExc_RuntimeError, "the caddtree library threw an exception");
    return nullptr;
  } catch (...) {          // a tensor that cannot be looked at this way
    status = -1;
  }
  if (status < 0) Py_RETURN_NONE;
  return PyLong_FromLong(status);
}

// the library's call without the interpreter's lock, as ctypes makes it; the lock is back however the call ends
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F>
int unlocked(F&& f) {
  try {
    const Unlocked u;
    return (int)f();
  } catch (...) {
    throw LibraryThrew();
  }
}

void tree_fields(Call& c, PyObject* out, int64_t B, caddtree_outputs_t* o) {
  const int64_t cap = c.s.cap;
  o->parent = as<int32_t>(c.data(c.attr(out, g_name[kParent]), c10::kInt, {cap}, B, true));
  o->n_star = as<int32_t>(c.data(c.attr(out, g_name[kNStar]), c10::kInt, {}, B, true));
  o->depth = as<int32_t>(c.data(c.attr(out, g_name[kDepth]), c10::kInt, {cap}, B, true));
  o->token_ids = as<int32_t>(c.data(c.attr(out, g_name[kTokenIds]), c10::kInt, {cap}, B, true));
  o->path_prob = as<float>(c.data(c.attr(out, g_name[kPathProb]), c10::kFloat, {cap}, B, false));
  o->phi = as<float>(c.data(c.attr(out, g_name[kPhi]), c10::kFloat, {}, B, false));
  o->theta = as<float>(c.data(c.attr(out, g_name[kTheta]), c10::kFloat, {}, B, false));
}

void emit_fields(Call& c, PyObject* out, int64_t B, caddtree_outputs_t* o) {
  o->pos_ids = as<int32_t>(c.data(c.attr(out, g_name[kPosIds]), c10::kInt, {c.s.cap}, B, false));
  o->mask = c.mask(c.attr(out, g_name[kMask]), B);
}

void topk_fields(Call& c, PyObject* out, int64_t B, bool required, caddtree_outputs_t* o) {
  const int64_t L = c.s.L, K = c.s.K;
  o->topk_ids = as<int32_t>(c.data(c.attr(out, g_name[kTopkIds]), c10::kInt, {L, K}, B, required));
  o->topk_logit = as<float>(c.data(c.attr(out, g_name[kTopkLogit]), c10::kFloat, {L, K}, B, required));
  o->lse = as<double>(c.data(c.attr(out, g_name[kLse]), c10::kDouble, {L}, B, required));
}

// spec, logits, out, pos_offset, workspace (None for the no-allocation call), ctx_len, stream, noalloc
PyObject* py_build(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 8, [&](const Spec& s) -> int {
    Call c(s);
    int64_t B = 0, stride = 0;
    const void* x = c.logits(a[1], &B, &stride);
    if (!c.ok) return -1;
    caddtree_outputs_t o = {};
    tree_fields(c, a[2], B, &o);
    emit_fields(c, a[2], B, &o);
    topk_fields(c, a[2], B, false, &o);
    o.topk_lq = as<float>(c.data(c.attr(a[2], g_name[kTopkLq]), c10::kFloat, {s.L, s.K}, B, false));
    const int32_t pos = c.offset(a[3]);
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (c.ok && a[4] != Py_None) {
      c10::TensorImpl* t = c.tensor(a[4]);
      if (t == nullptr || !t->is_contiguous() || t->numel() == 0) return -1;
      ws = t->mutable_data();
      ws_bytes = (size_t)t->numel() * t->itemsize();
    }
    const int64_t* ctx = c.ctx(a[5], B);
    const hipStream_t st = c.stream(a[6]);
    if (!c.ok) return -1;
    if (a[7] == Py_True)
      return unlocked([&] { return s.build_noalloc(s.plan, x, B, stride, pos, ctx, &o, st); });
    return unlocked([&] { return s.build(s.plan, x, B, stride, pos, ctx, &o, ws, ws_bytes, st); });
  });
}

// spec, logits, topk_ids, topk_logit, lse, topk_lq, stream
PyObject* py_reduce_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 7, [&](const Spec& s) -> int {
    Call c(s);
    int64_t B = 0, stride = 0;
    const void* x = c.logits(a[1], &B, &stride);
    if (!c.ok) return -1;
    auto* ids = as<int32_t>(c.data(a[2], c10::kInt, {s.L, s.K}, B, true));
    auto* logit = as<float>(c.data(a[3], c10::kFloat, {s.L, s.K}, B, true));
    auto* lse = as<double>(c.data(a[4], c10::kDouble, {s.L}, B, true));
    auto* lq = as<float>(c.data(a[5], c10::kFloat, {s.L, s.K}, B, false));
    const hipStream_t st = c.stream(a[6]);
    if (!c.ok) return -1;
    return unlocked([&] { return s.reduce_topk(s.plan, x, B, stride, ids, logit, lq, lse, st); });
  });
}

// spec, topk_ids, topk_logit, lse, out, ctx_len, stream
PyObject* py_expand(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 7, [&](const Spec& s) -> int {
    Call c(s);
    const int64_t B = c.rows(a[1]);
    auto* ids = as<int32_t>(c.data(a[1], c10::kInt, {s.L, s.K}, B, true));
    auto* logit = as<float>(c.data(a[2], c10::kFloat, {s.L, s.K}, B, true));
    auto* lse = as<double>(c.data(a[3], c10::kDouble, {s.L}, B, true));
    if (!c.ok) return -1;
    caddtree_outputs_t o = {};
    tree_fields(c, a[4], B, &o);
    const int64_t* ctx = c.ctx(a[5], B);
    const hipStream_t st = c.stream(a[6]);
    if (!c.ok) return -1;
    return unlocked([&] {
      return s.expand(s.plan, ids, logit, lse, B, ctx, o.token_ids, o.parent, o.depth, o.path_prob, o.n_star, o.phi,
                      o.theta, st);
    });
  });
}

// spec, out, pos_offset, stream
PyObject* py_emit(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 4, [&](const Spec& s) -> int {
    Call c(s);
    PyObject* par = c.attr(a[1], g_name[kParent]);
    const int64_t B = c.rows(par);
    caddtree_outputs_t o = {};
    o.parent = as<int32_t>(c.data(par, c10::kInt, {s.cap}, B, true));
    o.n_star = as<int32_t>(c.data(c.attr(a[1], g_name[kNStar]), c10::kInt, {}, B, true));
    emit_fields(c, a[1], B, &o);
    o.depth = as<int32_t>(c.data(c.attr(a[1], g_name[kDepth]), c10::kInt, {s.cap}, B, o.pos_ids != nullptr));
    const int32_t pos = c.offset(a[2]);
    const hipStream_t st = c.stream(a[3]);
    if (!c.ok) return -1;
    return unlocked([&] { return s.emit(s.plan, o.parent, o.depth, o.n_star, B, pos, o.mask, o.pos_ids, st); });
  });
}

// spec, topk, tree, u, accept_len, round_cost, ctx_len, stream
PyObject* py_accept(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(a, n, 8, [&](const Spec& s) -> int {
    Call c(s);
    PyObject* tok = c.attr(a[2], g_name[kTokenIds]);
    c10::TensorImpl* t = c.tensor(tok);
    if (t == nullptr || t->sizes().size() != 2) return -1;
    const int64_t B = t->sizes()[0], stride = t->sizes()[1];
    if (stride > INT32_MAX) return -1;
    auto* ids = as<int32_t>(c.data(tok, c10::kInt, {stride}, B, true));
    auto* par = as<int32_t>(c.data(c.attr(a[2], g_name[kParent]), c10::kInt, {stride}, B, true));
    auto* ns = as<int32_t>(c.data(c.attr(a[2], g_name[kNStar]), c10::kInt, {}, B, true));
    caddtree_outputs_t o = {};
    topk_fields(c, a[1], B, true, &o);
    auto* u = as<double>(c.data(a[3], c10::kDouble, {s.L}, B, true));
    if (!c.ok || c.rows(a[3]) != B) return -1;
    auto* al = as<int32_t>(c.data(a[4], c10::kInt, {}, B, true));
    auto* rc = as<double>(c.data(a[5], c10::kDouble, {}, B, false));
    const int64_t* ctx = a[5] != Py_None ? c.ctx(a[6], B) : nullptr;
    const hipStream_t st = c.stream(a[7]);
    if (!c.ok) return -1;
    return unlocked([&] {
      return s.accept(s.plan, o.topk_ids, o.topk_logit, o.lse, B, ids, par, (int32_t)stride, ns, u, ctx, al, rc, st);
    });
  });
}

// handle, device, L, V, K, cap, bf16, mask, the addresses of build, build_noalloc, reduce_topk, expand, emit, accept
PyObject* py_spec(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 14) {
    PyErr_Format(PyExc_TypeError, "14 arguments expected, got %zd", n);
    return nullptr;
  }
  int64_t v[14];
  for (int i = 0; i < 14; ++i) {
    v[i] = (int64_t)PyLong_AsUnsignedLongLongMask(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  Spec* s = new Spec();
  s->plan = reinterpret_cast<caddtree_plan_t>(v[0]);
  s->device = (int)v[1];
  s->L = v[2];
  s->V = v[3];
  s->K = v[4];
  s->cap = v[5] > 1 ? v[5] : 1;
  s->dtype = v[6] ? c10::kBFloat16 : c10::kFloat;
  s->mask = (int)v[7];
  s->build = reinterpret_cast<decltype(s->build)>(v[8]);
  s->build_noalloc = reinterpret_cast<decltype(s->build_noalloc)>(v[9]);
  s->reduce_topk = reinterpret_cast<decltype(s->reduce_topk)>(v[10]);
  s->expand = reinterpret_cast<decltype(s->expand)>(v[11]);
  s->emit = reinterpret_cast<decltype(s->emit)>(v[12]);
  s->accept = reinterpret_cast<decltype(s->accept)>(v[13]);
  PyObject* cap = PyCapsule_New(s, kSpecName, [](PyObject* o) {
    delete static_cast<Spec*>(PyCapsule_GetPointer(o, kSpecName));
  });
  if (cap == nullptr) delete s;
  return cap;
}

#define CALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {CALL(spec), CALL(build), CALL(reduce_topk), CALL(expand), CALL(emit), CALL(accept),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  for (int i = 0; i < kFields; ++i)
    if ((g_name[i] = PyUnicode_InternFromString(kNames[i])) == nullptr) return nullptr;
  return PyModule_Create(&g_module);
}
