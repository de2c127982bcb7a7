// Native half of the binding: the calls a decode loop makes per token and per round (draft_entropy, draft_step,
// verify), argument marshalling only.  At one sequence the kernels of such a call take 5 to 20 us, and building
// the argument structs in Python took 5 to 12 us of host time per call, more than a drafting kernel runs.
// Here a drafting call takes 3.3 to 4 us of host time with its launch, a verification 9 us with its three.
//
// binding.py hands over the entry points of libadasd.so as it loaded it, and the Python objects that are needed
// to raise and to allocate; keyword arguments, defaults, checks and exceptions are those of its signatures.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/adasd.h"

namespace {

struct Abi {
  decltype(&adasd_draft_entropy) draft_entropy;
  decltype(&adasd_draft_step) draft_step;
  decltype(&adasd_verify) verify;
  decltype(&adasd_verify_noalloc) verify_noalloc;
} g_abi;
PyObject* g_error = nullptr;         // AdasdError(code, where)
PyObject* g_alloc_result = nullptr;  // alloc_verify_result(B, K, device)

struct Fail {};                      // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Fail{};
}
void check(int rc, const char* where) {
  if (rc == 0) return;
  PyObject* e = PyObject_CallFunction(g_error, "is", rc, where);
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw Fail{};
}

// Positional and keyword arguments into slots; the first `required` must be there.
template <int N>
void parse(const char* fn, PyObject* const (&names)[N], int required, PyObject* const* args, Py_ssize_t nargs, PyObject* kw,
           PyObject* (&slot)[N]) {
  if (nargs > N) {
    PyErr_Format(PyExc_TypeError, "%s() takes at most %d positional arguments (%zd given)", fn, N, nargs);
    throw Fail{};
  }
  for (int i = 0; i < N; ++i) slot[i] = i < nargs ? args[i] : nullptr;
  const Py_ssize_t nk = kw ? PyTuple_GET_SIZE(kw) : 0;
  for (Py_ssize_t k = 0; k < nk; ++k) {
    PyObject* name = PyTuple_GET_ITEM(kw, k);
    int at = -1;
    for (int i = 0; i < N && at < 0; ++i)
      if (names[i] == name) at = i;              // (both interned, as a rule)
    for (int i = 0; i < N && at < 0; ++i)
      if (PyUnicode_Compare(names[i], name) == 0) at = i;
    if (at < 0) {
      PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", fn, name);
      throw Fail{};
    }
    if (slot[at]) {
      PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", fn, name);
      throw Fail{};
    }
    slot[at] = args[nargs + k];
  }
  for (int i = 0; i < required; ++i)
    if (!slot[i]) {
      PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%U'", fn, names[i]);
      throw Fail{};
    }
}

uint64_t integer(PyObject* o, uint64_t fallback) {       // any Python integer, taken modulo 2^64
  if (!o) return fallback;
  const uint64_t v = PyLong_CheckExact(o) ? PyLong_AsUnsignedLongLongMask(o) : [&] {
    PyObject* i = PyNumber_Index(o);
    if (!i) throw Fail{};
    const uint64_t w = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return w;
  }();
  if (v == (uint64_t)-1 && PyErr_Occurred()) throw Fail{};
  return v;
}

struct Ref {                                              // attribute of an object, new reference
  PyObject* o;
  Ref(PyObject* from, PyObject* name) : o(PyObject_GetAttr(from, name)) {
    if (!o) throw Fail{};
  }
  ~Ref() { Py_DECREF(o); }
  Ref(const Ref&) = delete;
};
uint64_t int_attr(PyObject* from, PyObject* name) { return integer(Ref(from, name).o, 0); }

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a torch tensor", name);
    throw Fail{};
  }
  return THPVariable_Unpack(o);
}
const char* type_name(at::ScalarType t) {
  switch (t) {
    case at::kFloat: return "torch.float32";
    case at::kInt: return "torch.int32";
    case at::kByte: return "torch.uint8";
    default: return "torch.float64";
  }
}
void* need(PyObject* o, at::ScalarType type, const char* name) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) {
    PyErr_Format(PyExc_ValueError, "%s must be a contiguous CUDA tensor of %s", name, type_name(type));
    throw Fail{};
  }
  return t.data_ptr();
}
void* maybe(PyObject* o, at::ScalarType type, const char* name) { return o && o != Py_None ? need(o, type, name) : nullptr; }
void* raw(PyObject* from, PyObject* name) {               // data pointer of a tensor attribute (NULL for None)
  Ref r(from, name);
  return r.o == Py_None ? nullptr : tensor(r.o, "state and result fields").data_ptr();
}
adasd_dtype logits_type(PyObject* o) {
  const at::Tensor& t = THPVariable_Unpack(o);
  if (t.scalar_type() == at::kBFloat16) return ADASD_BF16;
  if (t.scalar_type() == at::kFloat) return ADASD_F32;
  PyObject* type = PyObject_GetAttrString(o, "dtype");
  if (type) {
    PyErr_Format(PyExc_TypeError, "logits must be bfloat16 or float32, got %S", type);
    Py_DECREF(type);
  }
  throw Fail{};
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

PyObject* intern(const char* s) { return PyUnicode_InternFromString(s); }

// An output: the caller's tensor, checked, or a new one.
struct Output {
  PyObject* o;
  void* ptr;
  Output(PyObject* given, int64_t n, at::ScalarType type, const at::Tensor& like, const char* name) {
    if (given && given != Py_None) {
      ptr = need(given, type, name);
      o = given;
      Py_INCREF(o);
    } else {
      at::Tensor t = at::empty({n}, like.options().dtype(type));
      ptr = t.data_ptr();
      o = THPVariable_Wrap(std::move(t));
      if (!o) throw Fail{};
    }
  }
  ~Output() { Py_XDECREF(o); }
  Output(const Output&) = delete;
  PyObject* give() {
    PyObject* r = o;
    o = nullptr;
    return r;
  }
};

struct Names {
  PyObject *ptr = intern("ptr"), *bytes = intern("bytes"), *B = intern("B"), *cap = intern("cap"), *T_G = intern("T_G"),
           *ent_sum = intern("ent_sum"), *ent_cnt = intern("ent_cnt"), *LA = intern("LA"), *LR = intern("LR"),
           *nA = intern("nA"), *nR = intern("nR"), *mom = intern("mom"), *n_accept = intern("n_accept"),
           *next_token = intern("next_token"), *H_p = intern("H_p"), *H_q = intern("H_q"), *d_js = intern("d_js"),
           *p_accept = intern("p_accept"), *accept_mask = intern("accept_mask"), *status = intern("status"),
           *base_test = intern("base_test"), *reject_rule = intern("reject_rule"), *kde_min_n = intern("kde_min_n"),
           *bw_rule = intern("bw_rule"), *relaxed_off = intern("relaxed_off"), *d_eps = intern("d_eps"),
           *stats_path = intern("stats_path"), *apply_update = intern("apply_update"), *list_update = intern("list_update"),
           *wait_polls = intern("wait_polls");
};
Names* N = nullptr;

const at::Tensor& draft_rows(PyObject* o) {
  const at::Tensor& x = tensor(o, "draft_logits");
  if (x.dim() != 2 || !x.is_cuda() || x.stride(1) != 1)
    fail(PyExc_ValueError, "draft_logits must be a CUDA tensor [B, V] with contiguous vocabulary");
  return x;
}

template <class F> PyObject* guarded(F f) {
  try {
    return f();
  } catch (const Fail&) {
    return nullptr;
  } catch (...) {                      // out of memory, a failed stream look-up, ...: the classes that torch's own calls raise
    torch::translate_exception_to_python(std::current_exception());
    return nullptr;
  }
}

PyObject* py_draft_entropy(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
  return guarded([&]() -> PyObject* {
    static PyObject* const names[] = {intern("draft_logits"), intern("workspace"), intern("T_G"), intern("active"),
                                      intern("step"), intern("k_max"), intern("H_out"), intern("stop_out")};
    PyObject* a[8];
    parse("draft_entropy", names, 2, args, nargs, kw, a);
    const at::Tensor& x = draft_rows(a[0]);
    const int B = (int)x.size(0), V = (int)x.size(1);
    Output H(a[6], B, at::kFloat, x, "H_out"), stop(a[7], B, at::kByte, x, "stop_out");
    const float* tg = (const float*)maybe(a[2], at::kFloat, "T_G");
    const uint8_t* active = (const uint8_t*)maybe(a[3], at::kByte, "active");
    const adasd_dtype dt = logits_type(a[0]);
    const int step = (int)integer(a[4], 0), k_max = (int)integer(a[5], 1 << 30);
    const int64_t stride = B > 1 ? x.stride(0) : V;
    void *ws = (void*)int_attr(a[1], N->ptr), *st = stream(), *rows = x.data_ptr();
    const size_t ws_bytes = int_attr(a[1], N->bytes);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_abi.draft_entropy(rows, dt, B, V, stride, tg, active, step, k_max, (float*)H.ptr, (uint8_t*)stop.ptr, ws, ws_bytes, st);
    Py_END_ALLOW_THREADS
    check(rc, "adasd_draft_entropy");
    PyObject* r = PyTuple_New(2);
    if (!r) throw Fail{};
    PyTuple_SET_ITEM(r, 0, H.give());
    PyTuple_SET_ITEM(r, 1, stop.give());
    return r;
  });
}

PyObject* py_draft_step(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
  return guarded([&]() -> PyObject* {
    static PyObject* const names[] = {intern("draft_logits"), intern("workspace"), intern("T_G"), intern("active"),
                                      intern("step"), intern("k_max"), intern("seed"), intern("seq_id"), intern("rounds"),
                                      intern("round0"), intern("H_out"), intern("stop_out"), intern("token_out"),
                                      intern("status_out")};
    PyObject* a[14];
    parse("draft_step", names, 2, args, nargs, kw, a);
    const at::Tensor& x = draft_rows(a[0]);
    const int B = (int)x.size(0), V = (int)x.size(1);
    const float* tg = (const float*)maybe(a[2], at::kFloat, "T_G");
    const uint8_t* active = (const uint8_t*)maybe(a[3], at::kByte, "active");
    const uint32_t* seq = (const uint32_t*)maybe(a[7], at::kInt, "seq_id");
    const uint32_t* rounds = (const uint32_t*)maybe(a[8], at::kInt, "rounds");
    Output H(a[10], B, at::kFloat, x, "H_out"), stop(a[11], B, at::kByte, x, "stop_out"),
        token(a[12], B, at::kInt, x, "token_out"), status(a[13], B, at::kInt, x, "status_out");
    const adasd_dtype dt = logits_type(a[0]);
    const int step = (int)integer(a[4], 0), k_max = (int)integer(a[5], 1 << 30);
    const uint64_t seed = integer(a[6], 0);
    const uint32_t round0 = (uint32_t)integer(a[9], 0);
    const int64_t stride = B > 1 ? x.stride(0) : V;
    void *ws = (void*)int_attr(a[1], N->ptr), *st = stream(), *rows = x.data_ptr();
    const size_t ws_bytes = int_attr(a[1], N->bytes);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_abi.draft_step(rows, dt, B, V, stride, tg, active, step, k_max, seed, seq, rounds, round0, (float*)H.ptr,
                          (uint8_t*)stop.ptr, (int32_t*)token.ptr, (uint32_t*)status.ptr, ws, ws_bytes, st);
    Py_END_ALLOW_THREADS
    check(rc, "adasd_draft_step");
    PyObject* r = PyTuple_New(4);
    if (!r) throw Fail{};
    PyTuple_SET_ITEM(r, 0, H.give());
    PyTuple_SET_ITEM(r, 1, stop.give());
    PyTuple_SET_ITEM(r, 2, token.give());
    PyTuple_SET_ITEM(r, 3, status.give());
    return r;
  });
}

PyObject* py_verify(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
  return guarded([&]() -> PyObject* {
    static PyObject* const names[] = {intern("target_logits"), intern("draft_logits"), intern("draft_tokens"),
                                      intern("workspace"), intern("state"), intern("draft_len"), intern("seed"),
                                      intern("seq_id"), intern("rounds"), intern("round0"), intern("options"), intern("out")};
    PyObject* a[12];
    parse("verify", names, 4, args, nargs, kw, a);
    const at::Tensor &p = tensor(a[0], "target_logits"), &q = tensor(a[1], "draft_logits");
    if (p.dim() != 3 || q.dim() != 3) fail(PyExc_ValueError, "logits must be [B, k(+1), V]");
    const int64_t B = p.size(0), K = p.size(1) - 1, V = p.size(2);
    if (q.size(0) != B || q.size(1) != K || q.size(2) != V) {
      PyErr_Format(PyExc_ValueError, "draft_logits must be [%lld, %lld, %lld]", (long long)B, (long long)K, (long long)V);
      throw Fail{};
    }
    if (p.stride(2) != 1 || (K > 0 && q.stride(2) != 1)) fail(PyExc_ValueError, "vocabulary dimension must be contiguous");
    if (p.scalar_type() != q.scalar_type()) fail(PyExc_TypeError, "target and draft logits must share a dtype");
    adasd_verify_args v{};
    v.draft_tokens = (const int32_t*)need(a[2], at::kInt, "draft_tokens");
    v.draft_len = (const int32_t*)maybe(a[5], at::kInt, "draft_len");
    v.seq_id = (const uint32_t*)maybe(a[7], at::kInt, "seq_id");
    v.round = (const uint32_t*)maybe(a[8], at::kInt, "rounds");
    v.target_logits = p.data_ptr();
    v.draft_logits = q.data_ptr();
    v.dt = logits_type(a[0]);
    v.B = (int32_t)B;
    v.k_max = (int32_t)K;
    v.V = (int32_t)V;
    v.t_seq_stride = p.stride(0);
    v.t_pos_stride = p.stride(1);
    v.d_seq_stride = K > 0 ? q.stride(0) : V;
    v.d_pos_stride = K > 0 ? q.stride(1) : V;
    v.seed = integer(a[6], 0);
    v.round0 = (uint32_t)integer(a[9], 0);
    adasd_state s{};
    if (a[4] && a[4] != Py_None) {
      PyObject* o = a[4];
      s.B = (int32_t)int_attr(o, N->B);
      s.cap = (int32_t)int_attr(o, N->cap);
      s.T_G = (float*)raw(o, N->T_G);
      s.ent_sum = (double*)raw(o, N->ent_sum);
      s.ent_cnt = (int32_t*)raw(o, N->ent_cnt);
      s.LA = (float*)raw(o, N->LA);
      s.LR = (float*)raw(o, N->LR);
      s.nA = (int32_t*)raw(o, N->nA);
      s.nR = (int32_t*)raw(o, N->nR);
      s.mom = (double*)raw(o, N->mom);
      v.state = &s;
    }
    adasd_options opt{};
    const bool has_opt = a[10] && a[10] != Py_None;
    if (has_opt) {
      PyObject* o = a[10];
      opt.base_test = (int32_t)int_attr(o, N->base_test);
      opt.reject_rule = (int32_t)int_attr(o, N->reject_rule);
      opt.kde_min_n = (int32_t)int_attr(o, N->kde_min_n);
      opt.bw_rule = (int32_t)int_attr(o, N->bw_rule);
      opt.relaxed_off = (int32_t)int_attr(o, N->relaxed_off);
      const double eps = PyFloat_AsDouble(Ref(o, N->d_eps).o);
      if (eps == -1.0 && PyErr_Occurred()) throw Fail{};
      opt.d_eps = (float)eps;
      opt.stats_path = (int32_t)int_attr(o, N->stats_path);
      opt.apply_update = (int32_t)int_attr(o, N->apply_update);
      opt.list_update = (int32_t)int_attr(o, N->list_update);
      opt.wait_polls = (int32_t)int_attr(o, N->wait_polls);
    }
    PyObject* out = a[11];
    if (out && out != Py_None) {
      Py_INCREF(out);
    } else {
      PyObject* dev = PyObject_GetAttrString(a[0], "device");
      if (!dev) throw Fail{};
      out = PyObject_CallFunction(g_alloc_result, "LLN", (long long)B, (long long)K, dev);
      if (!out) throw Fail{};
    }
    struct Drop {
      PyObject* o;
      ~Drop() { Py_XDECREF(o); }
    } drop{out};
    v.n_accept = (int32_t*)raw(out, N->n_accept);
    v.next_token = (int32_t*)raw(out, N->next_token);
    v.H_p = (float*)raw(out, N->H_p);
    v.H_q = (float*)raw(out, N->H_q);
    v.d_js = (float*)raw(out, N->d_js);
    v.p_accept = (float*)raw(out, N->p_accept);
    v.accept_mask = (uint8_t*)raw(out, N->accept_mask);
    v.status = (uint32_t*)raw(out, N->status);
    const bool noalloc = a[3] == Py_None;
    if (!noalloc) {
      v.workspace = (void*)int_attr(a[3], N->ptr);
      v.ws_bytes = int_attr(a[3], N->bytes);
    }
    void* st = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = (noalloc ? g_abi.verify_noalloc : g_abi.verify)(&v, has_opt ? &opt : nullptr, st);
    Py_END_ALLOW_THREADS
    check(rc, noalloc ? "adasd_verify_noalloc" : "adasd_verify");
    drop.o = nullptr;
    return out;
  });
}

// connect(error class, result allocator, addresses of draft_entropy, draft_step, verify, verify_noalloc)
PyObject* py_connect(PyObject*, PyObject* args) {
  PyObject *err, *alloc;
  unsigned long long f[4];
  if (!PyArg_ParseTuple(args, "OOKKKK", &err, &alloc, &f[0], &f[1], &f[2], &f[3])) return nullptr;
  Py_INCREF(err);
  Py_INCREF(alloc);
  Py_XSETREF(g_error, err);
  Py_XSETREF(g_alloc_result, alloc);
  g_abi.draft_entropy = (decltype(g_abi.draft_entropy))f[0];
  g_abi.draft_step = (decltype(g_abi.draft_step))f[1];
  g_abi.verify = (decltype(g_abi.verify))f[2];
  g_abi.verify_noalloc = (decltype(g_abi.verify_noalloc))f[3];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"draft_entropy", (PyCFunction)(void (*)(void))py_draft_entropy, METH_FASTCALL | METH_KEYWORDS, nullptr},
    {"draft_step", (PyCFunction)(void (*)(void))py_draft_step, METH_FASTCALL | METH_KEYWORDS, nullptr},
    {"verify", (PyCFunction)(void (*)(void))py_verify, METH_FASTCALL | METH_KEYWORDS, nullptr},
    {"connect", py_connect, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  N = new Names;
  return PyModule_Create(&module);
}
