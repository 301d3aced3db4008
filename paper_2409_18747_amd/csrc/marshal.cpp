// The marshalling of binding.py in C++, for the calls as programs make them: plain contiguous tensors on one GPU,
// the current stream.  Checks and conversions of a call take the interpreter and ctypes 3 to 8 us, as long as the
// kernels of the smallest calls last; here a few tenths of one (figures in binding.py).
//
// Every function either does the whole call, or finds something it does not know or that does not match,
// has done nothing, and returns None: then binding.py goes through the call itself and says what is
// wrong.  What passes here is not looked at again, and the kernels index by it: every condition on an argument that
// binding.py has stands here too, and one that is added there is added here (tests/test_gpu_marshal_refusals.py holds
// the two together).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/cottn.h"

namespace {

// The library's functions, as the library that binding.py has loaded exports them.
struct Library {
  decltype(&cottn_workspace_bytes_dkdv) workspace_bytes_dkdv;
  decltype(&cottn_fwd_causal) fwd_causal;
  decltype(&cottn_fwd_causal_from_state) fwd_causal_from_state;
  decltype(&cottn_fwd_causal_varlen) fwd_causal_varlen;
  decltype(&cottn_fwd_causal_dkdv) fwd_causal_dkdv;
  decltype(&cottn_fwd_bidir) fwd_bidir;
  decltype(&cottn_fwd_bidir_varlen) fwd_bidir_varlen;
  decltype(&cottn_fwd_bidir_dkdv) fwd_bidir_dkdv;
  decltype(&cottn_bwd_causal) bwd_causal;
  decltype(&cottn_bwd_causal_from_state) bwd_causal_from_state;
  decltype(&cottn_bwd_causal_varlen) bwd_causal_varlen;
  decltype(&cottn_bwd_causal_dkdv) bwd_causal_dkdv;
  decltype(&cottn_bwd_bidir) bwd_bidir;
  decltype(&cottn_bwd_bidir_varlen) bwd_bidir_varlen;
  decltype(&cottn_bwd_bidir_dkdv) bwd_bidir_dkdv;
  decltype(&cottn_step_dkdv) step_dkdv;
  decltype(&cottn_scale_from_m_varlen) scale_from_m_varlen;
  decltype(&cottn_scale_backward_varlen) scale_backward_varlen;
} lib;
PyObject* error_type = nullptr;   // binding.CottnError

// binding.py's numbers for the variants of a forward or backward
enum Variant { CAUSAL = 0, CAUSAL_FROM_STATE = 1, CAUSAL_VARLEN = 2, CAUSAL_DKDV = 3, BIDIR = 4, BIDIR_VARLEN = 5, BIDIR_DKDV = 6 };
bool is_bidir(int v) { return v >= BIDIR; }
bool has_lengths(int v) { return v == CAUSAL_VARLEN || v == BIDIR_VARLEN; }
bool own_widths(int v) { return v == CAUSAL_DKDV || v == BIDIR_DKDV; }

PyObject* raise_status(int status, const char* where) {
  if (PyObject* e = PyObject_CallFunction(error_type, "is", status, where)) {
    PyErr_SetObject(error_type, e);
    Py_DECREF(e);
  }
  return nullptr;
}

// Tensors that somebody else has a say in (modes, transforms, lazily conjugated or negated views), or with named dimensions,
// which their results take over: binding.py's.
constexpr c10::DispatchKeySet kNotPlain({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
                                         c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                         c10::DispatchKey::Batched, c10::DispatchKey::Functionalize,
                                         c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                         c10::DispatchKey::ZeroTensor, c10::DispatchKey::Named});
bool modes_on() { return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set(); }

// A plain contiguous tensor on a GPU, or null.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.key_set().has_any(kNotPlain) ||
      t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || !t.is_contiguous())
    return nullptr;
  return &t;
}

bool like(const at::Tensor& t, const at::Tensor& ref) {
  return t.sizes() == ref.sizes() && t.scalar_type() == ref.scalar_type() && t.device() == ref.device();
}

int dtype_code(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return COTTN_F32;
    case at::kBFloat16: return COTTN_BF16;
    case at::kHalf: return COTTN_F16;
    default: return -1;
  }
}

// The arguments of a call one after the other.  Any that is not as it has to be clears `ok`.
struct Call {
  PyObject* const* next;
  bool ok = true;
  c10::Device device = c10::Device(c10::kCPU);

  const at::Tensor* tensor() {
    const at::Tensor* t = plain(*next++);
    ok = ok && t != nullptr;
    return t;
  }
  // Q and the like, whose place all others share
  const at::Tensor* first(int dims) {
    const at::Tensor* t = tensor();
    if (!ok || t->dim() != dims || dtype_code(*t) < 0) {
      ok = false;
      return nullptr;
    }
    device = t->device();
    return t;
  }
  const at::Tensor* rows_like(const at::Tensor* ref, bool optional = false) {
    if (optional && *next == Py_None) {
      ++next;
      return nullptr;
    }
    const at::Tensor* t = tensor();
    ok = ok && ref != nullptr && like(*t, *ref);
    return t;
  }
  void* floats(int64_t numel, bool optional = false) {
    if (optional && *next == Py_None) {
      ++next;
      return nullptr;
    }
    const at::Tensor* t = tensor();
    ok = ok && t->scalar_type() == at::kFloat && t->numel() == numel && t->device() == device;
    return ok ? t->data_ptr() : nullptr;
  }
  const int* lengths(int64_t B) {
    const at::Tensor* t = tensor();
    ok = ok && t->scalar_type() == at::kInt && t->numel() == B && t->device() == device;
    return ok ? static_cast<const int*>(t->data_ptr()) : nullptr;
  }
  // a workspace and its size
  void* bytes(size_t& size) {
    size = 0;
    if (*next == Py_None) {
      ++next;
      return nullptr;
    }
    const at::Tensor* t = tensor();
    ok = ok && t->device() == device;
    if (!ok) return nullptr;
    size = t->nbytes();
    return t->data_ptr();
  }
  int integer() {
    PyObject* o = *next++;
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    ok = ok && overflow == 0 && v >= INT_MIN && v <= INT_MAX;
    return int(v);
  }
  float real() {
    PyObject* o = *next++;
    ok = ok && PyFloat_CheckExact(o);
    return ok ? float(PyFloat_AS_DOUBLE(o)) : 0.f;
  }
};

// Other threads run Python meanwhile, as under ctypes: an allocation or a launch may wait for the GPU.
struct Unlocked {
  PyThreadState* const thread = PyEval_SaveThread();
  Unlocked() = default;
  Unlocked(const Unlocked&) = delete;
  ~Unlocked() { PyEval_RestoreThread(thread); }
};

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the given object, or a new tensor (of `made`), as a result
PyObject* result(PyObject* given, at::Tensor& made) {
  if (given == Py_None) return THPVariable_Wrap(std::move(made));
  Py_INCREF(given);
  return given;
}

bool sizes_fit(const at::Tensor& q) {
  for (int64_t n : q.sizes())
    if (n > INT_MAX) return false;
  return true;
}

// fwd(variant, Q, K, V, s, seq_len or None, state_in or None, O, state, workspace, chunk, eps)
PyObject* fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 12 || modes_on()) Py_RETURN_NONE;
  Call c{args};
  const int variant = c.integer();
  const at::Tensor *Q = c.first(4), *K = c.rows_like(Q), *V = nullptr;
  if (!c.ok || !sizes_fit(*Q)) Py_RETURN_NONE;
  const int B = int(Q->size(0)), H = int(Q->size(1)), N = int(Q->size(2)), dk = int(Q->size(3)), dt = dtype_code(*Q);
  int dv = dk;
  if (own_widths(variant)) {
    V = c.tensor();
    if (!c.ok || V->dim() != 4 || V->size(0) != B || V->size(1) != H || V->size(2) != N || V->size(3) > INT_MAX ||
        V->scalar_type() != Q->scalar_type() || V->device() != c.device)
      Py_RETURN_NONE;
    dv = int(V->size(3));
  } else {
    V = c.rows_like(Q);
  }
  const int64_t units = int64_t(B) * H;
  const float* s = static_cast<const float*>(c.floats(has_lengths(variant) ? units : H));
  const int* seq_len = has_lengths(variant) ? c.lengths(B) : (++c.next, nullptr);
  const float* state_in = variant == CAUSAL_FROM_STATE ? static_cast<const float*>(c.floats(units * dk * dv)) : (++c.next, nullptr);
  PyObject* given_O = *c.next;
  const at::Tensor* O = c.rows_like(V, true);
  float* state = static_cast<float*>(c.floats(units * dk * dv, true));
  const bool given_workspace = *c.next != Py_None;
  size_t have = 0;
  void* workspace = c.bytes(have);
  const int chunk = c.integer();
  const float eps = c.real();
  if (!c.ok) Py_RETURN_NONE;

  at::Tensor made, scratch;
  if (!given_workspace) {
    have = lib.workspace_bytes_dkdv(is_bidir(variant) ? COTTN_OP_FWD_BIDIR : COTTN_OP_FWD_CAUSAL, B, H, N, dk, dv, chunk, dt);
    if (have == size_t(-1)) Py_RETURN_NONE;
  }
  int st = COTTN_E_ARG;
  const char* where = "";
  {
    const Unlocked unlocked;
    if (O == nullptr) {
      made = at::empty(V->sizes(), V->options());
      O = &made;
    }
    if (!given_workspace && have > 0) {
      scratch = at::empty({int64_t(have)}, Q->options().dtype(at::kByte));
      workspace = scratch.data_ptr();
    }
    const void *q = Q->data_ptr(), *k = K->data_ptr(), *v = V->data_ptr();
    void *o = O->data_ptr(), *stream = current_stream();
    switch (variant) {
      case CAUSAL:
        where = "cottn_fwd_causal";
        st = lib.fwd_causal(q, k, v, s, o, state, workspace, have, B, H, N, dk, chunk, dt, eps, stream);
        break;
      case CAUSAL_FROM_STATE:
        where = "cottn_fwd_causal_from_state";
        st = lib.fwd_causal_from_state(q, k, v, s, state_in, o, state, workspace, have, B, H, N, dk, chunk, dt, eps, stream);
        break;
      case CAUSAL_VARLEN:
        where = "cottn_fwd_causal_varlen";
        st = lib.fwd_causal_varlen(q, k, v, s, seq_len, o, state, workspace, have, B, H, N, dk, chunk, dt, eps, stream);
        break;
      case CAUSAL_DKDV:
        where = "cottn_fwd_causal_dkdv";
        st = lib.fwd_causal_dkdv(q, k, v, s, o, state, workspace, have, B, H, N, dk, dv, chunk, dt, eps, stream);
        break;
      case BIDIR:
        where = "cottn_fwd_bidir";
        st = lib.fwd_bidir(q, k, v, s, o, state, workspace, have, B, H, N, dk, dt, eps, stream);
        break;
      case BIDIR_VARLEN:
        where = "cottn_fwd_bidir_varlen";
        st = lib.fwd_bidir_varlen(q, k, v, s, seq_len, o, state, workspace, have, B, H, N, dk, dt, eps, stream);
        break;
      case BIDIR_DKDV:
        where = "cottn_fwd_bidir_dkdv";
        st = lib.fwd_bidir_dkdv(q, k, v, s, o, state, workspace, have, B, H, N, dk, dv, dt, eps, stream);
        break;
    }
  }
  if (st != COTTN_OK) return raise_status(st, where);
  return result(given_O, made);
  END_HANDLE_TH_ERRORS
}

// bwd(variant, Q, K, V, s, seq_len or None, dO, state_in, rev_state_in, dQ, dK, dV, ds, rev_state_out,
//     fwd_workspace, workspace, chunk, eps)
PyObject* bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 18 || modes_on()) Py_RETURN_NONE;
  Call c{args};
  const int variant = c.integer();
  const at::Tensor *Q = c.first(4), *K = c.rows_like(Q), *V = nullptr;
  if (!c.ok || !sizes_fit(*Q)) Py_RETURN_NONE;
  const int B = int(Q->size(0)), H = int(Q->size(1)), N = int(Q->size(2)), dk = int(Q->size(3)), dt = dtype_code(*Q);
  int dv = dk;
  if (own_widths(variant)) {
    V = c.tensor();
    if (!c.ok || V->dim() != 4 || V->size(0) != B || V->size(1) != H || V->size(2) != N || V->size(3) > INT_MAX ||
        V->scalar_type() != Q->scalar_type() || V->device() != c.device)
      Py_RETURN_NONE;
    dv = int(V->size(3));
  } else {
    V = c.rows_like(Q);
  }
  const int64_t units = int64_t(B) * H, scales = has_lengths(variant) ? units : H, states = units * dk * dv;
  const float* s = static_cast<const float*>(c.floats(scales));
  const int* seq_len = has_lengths(variant) ? c.lengths(B) : (++c.next, nullptr);
  const at::Tensor* dO = c.rows_like(V);
  const float* state_in = static_cast<const float*>(c.floats(states, true));
  const float* rev_in = static_cast<const float*>(c.floats(states, true));
  PyObject* const* given = c.next;   // dQ, dK, dV, ds
  const at::Tensor* grads[3] = {c.rows_like(Q, true), nullptr, nullptr};
  grads[1] = c.rows_like(Q, true);
  grads[2] = c.rows_like(V, true);
  float* ds = static_cast<float*>(c.floats(scales, true));
  float* rev_out = static_cast<float*>(c.floats(states, true));
  size_t fwd_have = 0, have = 0;
  const void* fwd_workspace = c.bytes(fwd_have);
  const bool given_workspace = *c.next != Py_None;
  void* workspace = c.bytes(have);
  const int chunk = c.integer();
  const float eps = c.real();
  if (!c.ok) Py_RETURN_NONE;

  if (!given_workspace) {
    have = lib.workspace_bytes_dkdv(is_bidir(variant) ? COTTN_OP_BWD_BIDIR : COTTN_OP_BWD_CAUSAL, B, H, N, dk, dv, chunk, dt);
    if (have == size_t(-1)) Py_RETURN_NONE;
  }
  at::Tensor made[4], scratch;
  int st = COTTN_E_ARG;
  const char* where = "";
  {
    const Unlocked unlocked;
    for (int i = 0; i < 3; ++i)
      if (grads[i] == nullptr) {
        const at::Tensor* ref = i < 2 ? Q : V;
        made[i] = at::empty(ref->sizes(), ref->options());
        grads[i] = &made[i];
      }
    if (given[3] == Py_None) {
      made[3] = has_lengths(variant) ? at::empty({B, H}, Q->options().dtype(at::kFloat)) : at::empty({H}, Q->options().dtype(at::kFloat));
      ds = static_cast<float*>(made[3].data_ptr());
    }
    if (!given_workspace && have > 0) {
      scratch = at::empty({int64_t(have)}, Q->options().dtype(at::kByte));
      workspace = scratch.data_ptr();
    }
    const void *q = Q->data_ptr(), *k = K->data_ptr(), *v = V->data_ptr(), *go = dO->data_ptr();
    void *dq = grads[0]->data_ptr(), *dkey = grads[1]->data_ptr(), *dval = grads[2]->data_ptr(), *stream = current_stream();
    switch (variant) {
      case CAUSAL:
        where = "cottn_bwd_causal";
        st = lib.bwd_causal(q, k, v, s, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H, N, dk, chunk, dt,
                            eps, stream);
        break;
      case CAUSAL_FROM_STATE:
        where = "cottn_bwd_causal_from_state";
        st = lib.bwd_causal_from_state(q, k, v, s, go, state_in, rev_in, dq, dkey, dval, ds, rev_out, fwd_workspace, fwd_have,
                                       workspace, have, B, H, N, dk, chunk, dt, eps, stream);
        break;
      case CAUSAL_VARLEN:
        where = "cottn_bwd_causal_varlen";
        st = lib.bwd_causal_varlen(q, k, v, s, seq_len, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H,
                                   N, dk, chunk, dt, eps, stream);
        break;
      case CAUSAL_DKDV:
        where = "cottn_bwd_causal_dkdv";
        st = lib.bwd_causal_dkdv(q, k, v, s, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H, N, dk, dv,
                                 chunk, dt, eps, stream);
        break;
      case BIDIR:
        where = "cottn_bwd_bidir";
        st = lib.bwd_bidir(q, k, v, s, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H, N, dk, dt, eps,
                           stream);
        break;
      case BIDIR_VARLEN:
        where = "cottn_bwd_bidir_varlen";
        st = lib.bwd_bidir_varlen(q, k, v, s, seq_len, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H,
                                  N, dk, dt, eps, stream);
        break;
      case BIDIR_DKDV:
        where = "cottn_bwd_bidir_dkdv";
        st = lib.bwd_bidir_dkdv(q, k, v, s, go, dq, dkey, dval, ds, fwd_workspace, fwd_have, workspace, have, B, H, N, dk, dv,
                                dt, eps, stream);
        break;
    }
  }
  if (st != COTTN_OK) return raise_status(st, where);
  PyObject* all = PyTuple_New(4);
  if (all == nullptr) return nullptr;
  for (int i = 0; i < 4; ++i) {
    PyObject* o = result(given[i], made[i]);
    if (o == nullptr) {
      Py_DECREF(all);
      return nullptr;
    }
    PyTuple_SET_ITEM(all, i, o);
  }
  return all;
  END_HANDLE_TH_ERRORS
}

// step(own_widths, q, k, v, s, state, o, eps)
PyObject* step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8 || modes_on()) Py_RETURN_NONE;
  Call c{args};
  const bool widths = c.integer() != 0;
  const at::Tensor *q = c.first(3), *k = c.rows_like(q), *v = nullptr;
  if (!c.ok || !sizes_fit(*q)) Py_RETURN_NONE;
  const int B = int(q->size(0)), H = int(q->size(1)), dk = int(q->size(2)), dt = dtype_code(*q);
  int dv = dk;
  if (widths) {
    v = c.tensor();
    if (!c.ok || v->dim() != 3 || v->size(0) != B || v->size(1) != H || v->size(2) > INT_MAX ||
        v->scalar_type() != q->scalar_type() || v->device() != c.device)
      Py_RETURN_NONE;
    dv = int(v->size(2));
  } else {
    v = c.rows_like(q);
  }
  const float* s = static_cast<const float*>(c.floats(H));
  float* state = static_cast<float*>(c.floats(int64_t(B) * H * dk * dv));
  PyObject* given = *c.next;
  const at::Tensor* o = c.rows_like(v, true);
  const float eps = c.real();
  if (!c.ok) Py_RETURN_NONE;
  at::Tensor made;
  int st;
  {
    const Unlocked unlocked;
    if (o == nullptr) {
      made = at::empty(v->sizes(), v->options());
      o = &made;
    }
    st = lib.step_dkdv(q->data_ptr(), k->data_ptr(), v->data_ptr(), s, state, o->data_ptr(), B, H, dk, dv, dt, eps,
                       current_stream());
  }
  if (st != COTTN_OK) return raise_status(st, widths ? "cottn_step_dkdv" : "cottn_step");
  return result(given, made);
  END_HANDLE_TH_ERRORS
}

// scale_varlen(m, seq_len, ds or None, result): s from m, or with ds the gradient of m
PyObject* scale_varlen(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4 || modes_on()) Py_RETURN_NONE;
  Call c{args};
  const at::Tensor *m = c.tensor(), *seq_len = c.tensor();
  if (!c.ok || m->scalar_type() != at::kFloat || seq_len->scalar_type() != at::kInt || seq_len->device() != m->device() ||
      m->numel() > INT_MAX || seq_len->numel() > INT_MAX)
    Py_RETURN_NONE;
  c.device = m->device();
  const int B = int(seq_len->numel()), H = int(m->numel());
  const bool backward = *c.next != Py_None;
  const float* ds = static_cast<const float*>(c.floats(int64_t(B) * H, true));
  PyObject* given = *c.next;
  float* out = static_cast<float*>(c.floats(backward ? H : int64_t(B) * H, true));
  if (!c.ok) Py_RETURN_NONE;
  at::Tensor made;
  const float* mp = static_cast<const float*>(m->data_ptr());
  const int* lp = static_cast<const int*>(seq_len->data_ptr());
  int st;
  {
    const Unlocked unlocked;
    if (given == Py_None) {
      made = backward ? at::empty({H}, m->options()) : at::empty({B, H}, m->options());
      out = static_cast<float*>(made.data_ptr());
    }
    st = backward ? lib.scale_backward_varlen(mp, lp, ds, out, B, H, current_stream())
                  : lib.scale_from_m_varlen(mp, lp, out, B, H, current_stream());
  }
  if (st != COTTN_OK) return raise_status(st, backward ? "cottn_scale_backward_varlen" : "cottn_scale_from_m_varlen");
  return result(given, made);
  END_HANDLE_TH_ERRORS
}

// bind(path of the library, which is loaded already; class of the error to raise with a status)
PyObject* bind(PyObject*, PyObject* args) {
  const char* path = nullptr;
  PyObject* error = nullptr;
  if (!PyArg_ParseTuple(args, "sO", &path, &error)) return nullptr;
  void* handle = dlopen(path, RTLD_NOW);
  if (handle == nullptr) {
    PyErr_SetString(PyExc_ImportError, dlerror());
    return nullptr;
  }
  Library found{};
  bool all = true;
  const auto find = [&](auto& f, const char* name) {
    f = reinterpret_cast<std::decay_t<decltype(f)>>(dlsym(handle, name));
    all = all && f != nullptr;
  };
#define COTTN_FIND(name) find(found.name, "cottn_" #name)
  COTTN_FIND(workspace_bytes_dkdv);
  COTTN_FIND(fwd_causal);
  COTTN_FIND(fwd_causal_from_state);
  COTTN_FIND(fwd_causal_varlen);
  COTTN_FIND(fwd_causal_dkdv);
  COTTN_FIND(fwd_bidir);
  COTTN_FIND(fwd_bidir_varlen);
  COTTN_FIND(fwd_bidir_dkdv);
  COTTN_FIND(bwd_causal);
  COTTN_FIND(bwd_causal_from_state);
  COTTN_FIND(bwd_causal_varlen);
  COTTN_FIND(bwd_causal_dkdv);
  COTTN_FIND(bwd_bidir);
  COTTN_FIND(bwd_bidir_varlen);
  COTTN_FIND(bwd_bidir_dkdv);
  COTTN_FIND(step_dkdv);
  COTTN_FIND(scale_from_m_varlen);
  COTTN_FIND(scale_backward_varlen);
#undef COTTN_FIND
  if (!all) {
    PyErr_Format(PyExc_ImportError, "%s lacks a function of cottn.h", path);
    return nullptr;
  }
  lib = found;
  Py_INCREF(error);
  Py_XDECREF(error_type);
  error_type = error;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fwd)), METH_FASTCALL, nullptr},
    {"bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bwd)), METH_FASTCALL, nullptr},
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(step)), METH_FASTCALL, nullptr},
    {"scale_varlen", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(scale_varlen)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: binding.py compares it with what it runs under (build.py: marshal_target)
PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* made = PyModule_Create(&module);
  if (made != nullptr && PyModule_AddStringConstant(made, "built_for", COTTN_BUILT_FOR) < 0) Py_CLEAR(made);
  return made;
}
