// The calls of a decoding step without Python between the arguments and the library: verify_attn, draft_window_attn,
// accept, hsr_fc and draft_qkv_append for arguments as programs pass them.  Each function returns NotImplemented where
// an argument is anything else (a tensor subclass, another dtype, shape or stride than the library takes, a host
// array that is not an int32 numpy array, ...) or a torch function mode is active; binding.py's own code then takes the
// call, converts what can be converted and raises what has to be raised.  Nothing is kept between calls.
//
// Host time, us (ctypes and Python alone / here), three calls each: draft token (hsr_fc, draft_qkv_append,
// draft_window_attn) 30.5 / 14.8; step of the tiny configuration (draft_window_attn, verify_attn, accept: five launches)
// 40 / 21.6, of which the launches are 13.  The kernels take 26 us of the draft token, which no longer waits for the
// host, and 21 of the step, where the two are level.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstring>

#include "../../include/sparrow.h"

namespace {

PyObject *g_check, *g_stream_ptr, *g_ndarray;            // binding._check, binding._stream_ptr, numpy.ndarray

// The library's functions, in the copy of the library that binding.py has loaded: linked by name, the loader could map
// another one, and _check would read the wrong copy's error text.
#define SPARROW_FUNCTIONS(f) \
  f(verify_attn_workspace) f(verify_attn) f(draft_window_attn) f(accept_workspace) f(accept_trees) f(hsr_fc) f(draft_qkv_append)
struct Library {
#define SPARROW_MEMBER(n) decltype(&sparrow_##n) n;
  SPARROW_FUNCTIONS(SPARROW_MEMBER)
} lib;
#define SPARROW_STRING_OF(x) #x
#define SPARROW_STRING(x) SPARROW_STRING_OF(x)
#define SPARROW_NAME(n) "sparrow_" #n,
constexpr const char *kFunctions[] = {SPARROW_FUNCTIONS(SPARROW_NAME)};
// Code compiled against the headers of one torch and one Python reads another's objects wrongly, without an error:
// binding.py takes this part only where it runs under the same ones.
constexpr char kBuiltFor[] = "torch " TORCH_VERSION ", Python " SPARROW_STRING(PY_MAJOR_VERSION) "." SPARROW_STRING(PY_MINOR_VERSION);
constexpr int kNumFunctions = sizeof(kFunctions) / sizeof(kFunctions[0]);
static_assert(sizeof(Library) == kNumFunctions * sizeof(void *), "one address after the other");

PyObject *new_ref(PyObject *o) {
  Py_INCREF(o);
  return o;
}

struct NotHere {};                                       // the general code takes the call
void need(bool ok) {
  if (!ok) throw NotHere{};
}

const at::Tensor &tensor(PyObject *o) {
  need(THPVariable_CheckExact(o));
  return THPVariable_Unpack(o);
}
bool none(PyObject *o) { return o == Py_None; }
void *ptr(const at::Tensor &t) { return t.data_ptr(); }
void *opt_ptr(PyObject *o) { return none(o) ? nullptr : ptr(tensor(o)); }

int64_t integer(PyObject *o) {
  need(PyLong_CheckExact(o));
  const int64_t x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    need(false);
  }
  return x;
}
int32_t int_arg(PyObject *o) {
  const int64_t x = integer(o);
  need(x >= INT32_MIN && x <= INT32_MAX);
  return (int32_t)x;
}
float float_arg(PyObject *o) {
  need(PyFloat_CheckExact(o));
  return (float)PyFloat_AS_DOUBLE(o);
}
bool truth(PyObject *o) {
  need(PyBool_Check(o));
  return o == Py_True;
}
int32_t dtype_code(const at::Tensor &t) {
  if (t.scalar_type() == at::kBFloat16) return SPARROW_BF16;
  need(t.scalar_type() == at::kFloat);
  return SPARROW_F32;
}
bool of(const at::Tensor &t, at::ScalarType type) { return t.scalar_type() == type; }

// A one-dimensional contiguous int32 numpy array, held for the call.
class HostInts {
 public:
  explicit HostInts(PyObject *o) {
    need(Py_TYPE(o) == (PyTypeObject *)g_ndarray);
    if (PyObject_GetBuffer(o, &buf_, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
      PyErr_Clear();
      need(false);
    }
    held_ = true;
    const bool ok = buf_.ndim == 1 && buf_.itemsize == 4 && buf_.format != nullptr && buf_.format[0] == 'i' && buf_.format[1] == 0;
    if (!ok) {
      PyBuffer_Release(&buf_);
      held_ = false;
      need(false);
    }
  }
  ~HostInts() {
    if (held_) PyBuffer_Release(&buf_);
  }
  HostInts(const HostInts &) = delete;
  HostInts &operator=(const HostInts &) = delete;
  const int32_t *data() const { return (const int32_t *)buf_.buf; }
  int64_t size() const { return buf_.shape[0]; }

 private:
  Py_buffer buf_;
  bool held_ = false;
};

class Object {                                           // an owned reference
 public:
  explicit Object(PyObject *o) : o_(o) {}
  ~Object() { Py_XDECREF(o_); }
  Object(const Object &) = delete;
  Object &operator=(const Object &) = delete;
  PyObject *get() const { return o_; }
  PyObject *release() {
    PyObject *o = o_;
    o_ = nullptr;
    return o;
  }

 private:
  PyObject *o_;
};

struct Raised {};                                        // a Python exception is set

void *stream_arg(PyObject *o) {
  Object p(PyObject_CallOneArg(g_stream_ptr, o));
  if (p.get() == nullptr) throw Raised{};
  void *s = PyLong_AsVoidPtr(p.get());
  if (s == nullptr && PyErr_Occurred()) throw Raised{};
  return s;
}

template <class F> void call(F f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  if (rc == SPARROW_OK) return;
  Object code(PyLong_FromLong(rc));
  if (code.get() != nullptr) Object(PyObject_CallOneArg(g_check, code.get()));
  throw Raised{};                                        // (_check raises SparrowError for every other status)
}

// k and v: [T, Hkv, d] of equal shape and strides, contiguous in d
void check_kv(const at::Tensor &k, const at::Tensor &v) {
  need(k.dim() == 3 && k.stride(2) == 1 && v.strides() == k.strides() && v.sizes() == k.sizes());
}
sparrow_attn_desc desc_of(int32_t dtype, int64_t n_q_heads, const at::Tensor &k, int64_t d, float scale, int64_t parent_stride) {
  sparrow_attn_desc a;
  a.dtype = dtype;
  a.n_q_heads = (int32_t)n_q_heads;
  a.n_kv_heads = (int32_t)k.size(1);
  a.head_dim = (int32_t)d;
  a.scale = scale;
  a.kv_stride_token = k.stride(0);
  a.kv_stride_head = k.stride(1);
  a.parent_stride = (int32_t)parent_stride;
  return a;
}

const int32_t *parent_arg(PyObject *o, int64_t n_q, int64_t B, int64_t *stride) {
  *stride = 0;
  if (none(o)) return nullptr;
  const at::Tensor &p = tensor(o);
  need(of(p, at::kInt));
  if (!(p.dim() == 1 && p.numel() == n_q && p.is_contiguous())) {
    need(p.dim() == 2 && p.size(0) == B && p.size(1) == n_q && p.stride(1) == 1 && n_q > 0);
    *stride = B > 1 ? p.stride(0) : n_q;
  }
  return (const int32_t *)ptr(p);
}

// out / lse of the attention calls: the caller's, or new ones
PyObject *new_out(PyObject *o, const at::Tensor &q) {
  if (none(o)) return THPVariable_Wrap(at::empty_like(q));
  tensor(o);
  return new_ref(o);
}
PyObject *new_lse(PyObject *o, bool want, const at::Tensor &q) {
  if (none(o) && want) return THPVariable_Wrap(at::empty({q.size(0), q.size(1)}, q.options().dtype(at::kFloat)));
  if (!none(o)) tensor(o);
  return new_ref(o);
}
void made(const Object &o) {
  if (o.get() == nullptr) throw Raised{};
}
int64_t bytes_of(const at::Tensor &t) { return t.numel() * t.element_size(); }

// (q, k, v, cu_seqlens, parent, n_q, scale, out, lse, want_lse, workspace, stream)
PyObject *verify_attn(PyObject *const *a) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
  const HostInts cu(a[3]);
  const int64_t B = cu.size() - 1;
  const int32_t n_q = int_arg(a[5]);
  need(B > 0 && n_q > 0);
  check_kv(k, v);
  need(q.dim() == 3 && q.is_contiguous());
  int64_t parent_stride;
  const int32_t *parent = parent_arg(a[4], n_q, B, &parent_stride);
  const sparrow_attn_desc d = desc_of(dtype_code(q), q.size(1), k, q.size(2), float_arg(a[6]), parent_stride);
  Object out(new_out(a[7], q)), lse(new_lse(a[8], truth(a[9]), q));
  made(out);
  made(lse);
  at::Tensor ws;
  if (none(a[10])) {
    const size_t bytes = lib.verify_attn_workspace(&d, (int32_t)B, n_q, (int64_t)cu.data()[B] - cu.data()[0]);
    if (bytes > 0) ws = at::empty({(int64_t)bytes}, q.options().dtype(at::kByte));
  } else {
    ws = tensor(a[10]);
  }
  void *const st = stream_arg(a[11]);
  void *const pq = ptr(q), *const pk = ptr(k), *const pv = ptr(v), *const po = ptr(tensor(out.get())), *const pl = opt_ptr(lse.get());
  void *const pw = ws.defined() ? ptr(ws) : nullptr;
  const size_t ws_bytes = ws.defined() ? (size_t)bytes_of(ws) : 0;
  call([&] { return lib.verify_attn(&d, pq, pk, pv, cu.data(), parent, (int32_t)B, n_q, po, (float *)pl, pw, ws_bytes, st); });
  return PyTuple_Pack(2, out.get(), lse.get());
}

// (q, k, v, cu_seqlens, text_idx, cu_text, window, scale, out, lse, want_lse, stream)
PyObject *draft_window_attn(PyObject *const *a) {
  const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &idx = tensor(a[4]);
  const HostInts cu(a[3]), ct(a[5]);
  check_kv(k, v);
  need(q.dim() == 3 && q.is_contiguous());
  const int64_t B = q.size(0);
  need(B > 0 && B <= SPARROW_MAX_BATCH && cu.size() == B + 1 && ct.size() == B + 1);
  need(of(idx, at::kInt) && idx.is_contiguous());
  const sparrow_attn_desc d = desc_of(dtype_code(q), q.size(1), k, q.size(2), float_arg(a[7]), 0);
  const int32_t window = int_arg(a[6]);
  Object out(new_out(a[8], q)), lse(new_lse(a[9], truth(a[10]), q));
  made(out);
  made(lse);
  void *const st = stream_arg(a[11]);
  void *const pq = ptr(q), *const pk = ptr(k), *const pv = ptr(v), *const pi = ptr(idx), *const po = ptr(tensor(out.get()));
  void *const pl = opt_ptr(lse.get());
  call([&] {
    return lib.draft_window_attn(&d, pq, pk, pv, cu.data(), (const int32_t *)pi, ct.data(), (int32_t)B, window, po,
                                     (float *)pl, nullptr, 0, st);
  });
  return PyTuple_Pack(2, out.get(), lse.get());
}

// (hidden_rows, lm_head, draft_ids, parent, B, n_q, workspace, stream): outputs as binding.accept makes them
PyObject *accept(PyObject *const *a) {
  const at::Tensor &hid = tensor(a[0]), &W = tensor(a[1]);
  const int32_t B = int_arg(a[4]), n_q = int_arg(a[5]);
  need(B > 0 && B <= 512 && n_q > 0 && n_q <= SPARROW_MAX_NQ);
  need(hid.dim() == 2 && W.dim() == 2 && hid.is_contiguous() && W.is_contiguous() && hid.scalar_type() == W.scalar_type());
  const int64_t H = hid.size(1), V = W.size(0);
  need(hid.size(0) == (int64_t)B * (n_q + 1) && W.size(1) == H && H <= INT32_MAX && V <= INT32_MAX);
  const int32_t code = dtype_code(hid);
  int64_t parent_stride;
  const int32_t *parent = parent_arg(a[3], n_q, B, &parent_stride);
  void *const drafts = opt_ptr(a[2]);
  at::Tensor ws;
  if (none(a[6])) {
    const size_t bytes = lib.accept_workspace(code, B, n_q, (int32_t)H, (int32_t)V);
    if (bytes > 0) ws = at::empty({(int64_t)bytes}, hid.options().dtype(at::kByte));
  } else {
    ws = tensor(a[6]);
  }
  const at::TensorOptions ints = hid.options().dtype(at::kInt);
  const at::Tensor ids = at::empty({(int64_t)B * (n_q + 1)}, ints), len = at::empty({B}, ints), path = at::empty({B, n_q}, ints),
                   bonus = at::empty({B}, ints);
  void *const st = stream_arg(a[7]);
  void *const ph = ptr(hid), *const pw = ptr(W), *const ps = ws.defined() ? ptr(ws) : nullptr;
  const size_t ws_bytes = ws.defined() ? (size_t)bytes_of(ws) : 0;
  int32_t *const pi = (int32_t *)ptr(ids), *const pl = (int32_t *)ptr(len), *const pp = (int32_t *)ptr(path), *const pb = (int32_t *)ptr(bonus);
  call([&] {
    return lib.accept_trees(code, ph, pw, (const int32_t *)drafts, parent, (int32_t)parent_stride, B, n_q, (int32_t)H, (int32_t)V,
                                pi, pl, pp, pb, ps, ws_bytes, st);
  });
  Object r(PyDict_New());
  made(r);
  const std::pair<const char *, const at::Tensor *> items[] = {{"target_ids", &ids}, {"accept_len", &len}, {"accept_path", &path}, {"bonus_id", &bonus}};
  for (const auto &it : items) {
    Object t(THPVariable_Wrap(*it.second));
    made(t);
    if (PyDict_SetItemString(r.get(), it.first, t.get()) != 0) throw Raised{};
  }
  return r.release();
}

// (embed, token_ids, h_prev, w_fc, b_fc, out, stream)
PyObject *hsr_fc(PyObject *const *a) {
  const at::Tensor &embed = tensor(a[0]), &tok = tensor(a[1]), &h = tensor(a[2]), &w = tensor(a[3]);
  need(h.dim() == 2 && embed.dim() == 2 && w.dim() == 2);
  const int64_t M = h.size(0), H = h.size(1);
  need(M > 0 && M <= INT32_MAX && H <= INT32_MAX / 2 && embed.size(0) <= INT32_MAX);
  const int32_t code = dtype_code(h);
  need(h.is_contiguous() && embed.is_contiguous() && w.is_contiguous() && of(embed, h.scalar_type()) && of(w, h.scalar_type()));
  need(embed.size(1) == H && w.size(0) == H && w.size(1) == 2 * H);
  need(of(tok, at::kInt) && tok.dim() == 1 && tok.size(0) == M && tok.is_contiguous());
  void *bias = nullptr;
  if (!none(a[4])) {
    const at::Tensor &b = tensor(a[4]);
    need(b.is_contiguous() && of(b, h.scalar_type()));
    bias = ptr(b);
  }
  Object out(new_out(a[5], h));
  made(out);
  void *const st = stream_arg(a[6]);
  void *const pe = ptr(embed), *const pt = ptr(tok), *const ph = ptr(h), *const pw = ptr(w), *const po = ptr(tensor(out.get()));
  call([&] { return lib.hsr_fc(code, pe, (const int32_t *)pt, ph, pw, bias, (int32_t)M, (int32_t)H, (int32_t)embed.size(0), po, st); });
  return out.release();
}

// (z, norm_weight, eps, w_qkv, b_qkv, rope_cos, rope_sin, kv_rows, n_q_heads, k_cache, v_cache, q_out, stream)
PyObject *draft_qkv_append(PyObject *const *a) {
  const at::Tensor &z = tensor(a[0]), &norm = tensor(a[1]), &w = tensor(a[3]), &cs = tensor(a[5]), &sn = tensor(a[6]),
                   &k = tensor(a[9]), &v = tensor(a[10]);
  need(z.dim() == 2 && w.dim() == 2);
  const int64_t M = z.size(0), H = z.size(1);
  need(M > 0 && M <= INT32_MAX && H <= INT32_MAX);
  check_kv(k, v);
  const int64_t Hkv = k.size(1), d = k.size(2);
  const int32_t Hq = int_arg(a[8]);
  const int32_t code = dtype_code(z);
  need(z.is_contiguous() && norm.is_contiguous() && w.is_contiguous() && of(norm, z.scalar_type()) && of(w, z.scalar_type()));
  void *bias = nullptr;
  if (!none(a[4])) {
    const at::Tensor &b = tensor(a[4]);
    need(b.is_contiguous() && of(b, z.scalar_type()));
    bias = ptr(b);
  }
  need(Hq > 0 && w.size(0) == (Hq + 2 * Hkv) * d && w.size(1) == H);
  for (const at::Tensor *t : {&cs, &sn})
    need(of(*t, at::kFloat) && t->dim() == 2 && t->size(0) == M && t->size(1) == d / 2 && t->is_contiguous());
  const HostInts rows(a[7]);
  need(rows.size() == M);
  const sparrow_attn_desc desc = desc_of(code, Hq, k, d, 0.f, 0);
  const float eps = float_arg(a[2]);
  if (!none(a[11])) tensor(a[11]);
  Object out(none(a[11]) ? THPVariable_Wrap(at::empty({M, Hq, d}, z.options())) : new_ref(a[11]));
  made(out);
  void *const st = stream_arg(a[12]);
  void *const pz = ptr(z), *const pn = ptr(norm), *const pw = ptr(w), *const pc = ptr(cs), *const ps = ptr(sn), *const pk = ptr(k),
             *const pv = ptr(v), *const po = ptr(tensor(out.get()));
  call([&] {
    return lib.draft_qkv_append(&desc, pz, pn, eps, pw, bias, (const float *)pc, (const float *)ps, rows.data(), (int32_t)M,
                                    (int32_t)H, po, pk, pv, st);
  });
  return out.release();
}

template <PyObject *(*kCall)(PyObject *const *), int kArgs>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != kArgs) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  if (g_check == nullptr || at::impl::torch_function_mode_enabled()) return new_ref(Py_NotImplemented);
  try {
    return kCall(args);
  } catch (const NotHere &) {
    return new_ref(Py_NotImplemented);
  } catch (const Raised &) {
    return nullptr;
  } catch (const std::exception &) {                     // torch refused (no memory, no data pointer): let it say so in Python
    return new_ref(Py_NotImplemented);
  }
}

// setup(check, stream_ptr, ndarray, addresses of FUNCTIONS...)
PyObject *setup(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 3 + kNumFunctions) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  void *at[kNumFunctions];
  for (int i = 0; i < kNumFunctions; ++i) {
    at[i] = PyLong_AsVoidPtr(args[3 + i]);
    if (at[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "%s has no address", kFunctions[i]);
      return nullptr;
    }
  }
  std::memcpy(&lib, at, sizeof(lib));
  g_check = new_ref(args[0]);
  g_stream_ptr = new_ref(args[1]);
  g_ndarray = new_ref(args[2]);
  Py_RETURN_NONE;
}

#define SPARROW_ENTRY(f, n) {#f, (PyCFunction)(void (*)())entry<f, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SPARROW_ENTRY(verify_attn, 12),
                         SPARROW_ENTRY(draft_window_attn, 12),
                         SPARROW_ENTRY(accept, 8),
                         SPARROW_ENTRY(hsr_fc, 7),
                         SPARROW_ENTRY(draft_qkv_append, 13),
                         {"setup", (PyCFunction)(void (*)())setup, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  Object m(PyModule_Create(&module)), names(PyTuple_New(kNumFunctions));
  if (m.get() == nullptr || names.get() == nullptr) return nullptr;
  for (int i = 0; i < kNumFunctions; ++i) {
    PyObject *s = PyUnicode_FromString(kFunctions[i]);
    if (s == nullptr) return nullptr;
    PyTuple_SET_ITEM(names.get(), i, s);
  }
  if (PyObject_SetAttrString(m.get(), "FUNCTIONS", names.get()) != 0 ||
      PyModule_AddStringConstant(m.get(), "BUILT_FOR", kBuiltFor) != 0)
    return nullptr;
  return m.release();
}
