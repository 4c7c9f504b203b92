// The two calls a serving program makes per layer and generated token, decode attention and the decode step, from Python
// without ctypes: arguments are read from the tensors and the cache object, outputs allocated, the C ABI called.  Nothing
// is kept from one call for the next.  Through ctypes a step over a short context took longer on the host than on the GPU
// (a descriptor of 14 fields, two allocations at 1.4 us, 18 converted arguments); one sequence of 640 tokens, 32 heads:
// 11.1 -> 6.8 us a step, which is its time on the GPU.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/akvq.h"

namespace {

constexpr int64_t kHeadDim = 128;

// Attribute names of the cache object, made once.
struct Names {
  PyObject *B, *Hkv, *G, *T_cap, *S_cap, *T_len, *k_codes, *v_codes, *k_meta, *v_meta, *k_sal, *v_sal, *sal_idx, *sal_cnt,
      *fine_mask, *W, *k_win, *v_win, *workspace, *decode, *struct_, *window_struct;
} names;
// What the package's own cache class describes itself with, and the types of the descriptions (plain_cache).
struct Plain {
  PyObject *struct_ = nullptr, *window_struct = nullptr, *cache_type = nullptr, *window_type = nullptr;
} plain;

struct Held {  // an owned reference
  PyObject *p = nullptr;
  Held() = default;
  explicit Held(PyObject *q) : p(q) {}
  Held(const Held &) = delete;
  Held &operator=(const Held &) = delete;
  ~Held() { Py_XDECREF(p); }
};
struct Failed {};  // a Python error is set

[[noreturn]] void refuse(const char *why) {
  PyErr_SetString(PyExc_AssertionError, why);
  throw Failed();
}
#define REQUIRE(cond) do { if (!(cond)) refuse(#cond); } while (0)

int64_t int_attr(PyObject *o, PyObject *name) {
  Held v(PyObject_GetAttr(o, name));
  if (!v.p) throw Failed();
  const long long x = PyLong_AsLongLong(v.p);
  if (x == -1 && PyErr_Occurred()) throw Failed();
  return x;
}
const at::Tensor &tensor(PyObject *o) {
  if (!THPVariable_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "a tensor is expected");
    throw Failed();
  }
  return THPVariable_Unpack(o);
}
// device pointer of a tensor attribute (null for None where that is allowed); the object keeps the tensor
void *ptr_attr(PyObject *o, PyObject *name, bool optional = false) {
  Held v(PyObject_GetAttr(o, name));
  if (!v.p) throw Failed();
  if (optional && v.p == Py_None) return nullptr;
  return tensor(v.p).data_ptr();
}
// A cache whose method `name` is not the package's own (a derived class, a method put on the object) is asked by that method;
// true: its description is in `out`, which `held` keeps, or it has none.  Otherwise the attributes are read, which say what the
// own method would say without making the description in Python (3 us).
template <typename T>
bool described(PyObject *cache, PyObject *name, PyObject *own, PyObject *type, Held &held, T &out) {
  Held method(PyObject_GetAttr(cache, name));
  if (!method.p) {  // nothing to ask
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Failed();
    PyErr_Clear();
    return false;
  }
  if (PyMethod_Check(method.p) && PyMethod_GET_FUNCTION(method.p) == own) return false;
  held.p = PyObject_CallNoArgs(method.p);
  if (!held.p) throw Failed();
  if (held.p == Py_None) return true;
  const int is = type ? PyObject_IsInstance(held.p, type) : 0;
  if (is < 0) throw Failed();
  Py_buffer view;
  if (is == 0 || PyObject_GetBuffer(held.p, &view, PyBUF_SIMPLE) != 0) {
    PyErr_Format(PyExc_TypeError, "%U() of the cache did not return a descriptor", name);
    throw Failed();
  }
  const bool fits = view.len == (Py_ssize_t)sizeof(T);
  if (fits) std::memcpy(&out, view.buf, sizeof(T));
  PyBuffer_Release(&view);
  if (!fits) {
    PyErr_Format(PyExc_TypeError, "%U() of the cache returned a descriptor of another size", name);
    throw Failed();
  }
  return true;
}
double number(PyObject *o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw Failed();
  return x;
}
long integer(PyObject *o) {
  const long x = PyLong_AsLong(o);
  if (x == -1 && PyErr_Occurred()) throw Failed();
  return x;
}

struct Call {
  akvq_cache cache;
  akvq_window win;
  akvq_rope rope;
  const akvq_window *win_p = nullptr;
  const akvq_rope *rope_p = nullptr;
  Held rope_pair, cache_held, win_held;  // keep what the pointers come from
  uint32_t *fine_mask = nullptr;
  int Hq = 0, n_split = 0;
  uint32_t flags = 0;
  float sm_scale = 0.0f;
  const void *q = nullptr;
  at::Tensor out, lse, ws_tensor;
  void *ws = nullptr;
  size_t ws_bytes = 0;
  void *stream = nullptr;
};

// What both calls share.  more_rows: rows the call itself adds to the cache; check_out: out is looked at.
void gather(Call &c, PyObject *cache, PyObject *q_obj, PyObject *scale, PyObject *n_split, PyObject *flags, PyObject *out,
            PyObject *lse, PyObject *rope, int64_t more_rows, bool check_out) {
  akvq_cache &k = c.cache;
  const int32_t cache_B = (int32_t)int_attr(cache, names.B), Hkv = (int32_t)int_attr(cache, names.Hkv);
  const int32_t T_len = (int32_t)int_attr(cache, names.T_len);
  if (!described(cache, names.struct_, plain.struct_, plain.cache_type, c.cache_held, k)) {
    k.B = cache_B;
    k.Hkv = Hkv;
    k.G = (int32_t)int_attr(cache, names.G);
    k.T_cap = (int32_t)int_attr(cache, names.T_cap);
    k.S_cap = (int32_t)int_attr(cache, names.S_cap);
    k.T_len = T_len;
    k.k_codes = static_cast<uint32_t *>(ptr_attr(cache, names.k_codes));
    k.v_codes = static_cast<uint32_t *>(ptr_attr(cache, names.v_codes));
    k.k_meta = static_cast<uint32_t *>(ptr_attr(cache, names.k_meta));
    k.v_meta = static_cast<uint32_t *>(ptr_attr(cache, names.v_meta));
    k.k_sal = static_cast<uint16_t *>(ptr_attr(cache, names.k_sal));
    k.v_sal = static_cast<uint16_t *>(ptr_attr(cache, names.v_sal));
    k.sal_idx = static_cast<int32_t *>(ptr_attr(cache, names.sal_idx));
    k.sal_cnt = static_cast<int32_t *>(ptr_attr(cache, names.sal_cnt));
  } else if (c.cache_held.p == Py_None) {
    PyErr_SetString(PyExc_TypeError, "struct() of the cache returned None");
    throw Failed();
  }
  c.fine_mask = static_cast<uint32_t *>(ptr_attr(cache, names.fine_mask, true));
  const int64_t W = int_attr(cache, names.W);
  if (more_rows != 0 || W != 0 || c.fine_mask != nullptr || rope != Py_None) {
    if (described(cache, names.window_struct, plain.window_struct, plain.window_type, c.win_held, c.win)) {
      if (c.win_held.p != Py_None) c.win_p = &c.win;
    } else if (W != 0) {
      c.win = akvq_window{static_cast<uint16_t *>(ptr_attr(cache, names.k_win)),
                          static_cast<uint16_t *>(ptr_attr(cache, names.v_win)), (int32_t)W};
      c.win_p = &c.win;
    }
  }
  const at::Tensor &q = tensor(q_obj);
  REQUIRE(q.scalar_type() == at::kHalf && q.is_contiguous());
  if (q.dim() != 3) {
    PyErr_SetString(PyExc_ValueError, "q has to be [B, Hq, 128]");
    throw Failed();
  }
  const int64_t B = q.size(0);
  c.Hq = (int)q.size(1);
  c.q = q.data_ptr();
  c.sm_scale = (float)number(scale);
  c.flags = (uint32_t)integer(flags);
  const long n = integer(n_split);
  c.n_split = n > 0 ? (int)n : 0;
  const int most = n > 0 ? (int)n : akvq_decode_default_splits(cache_B, Hkv, (int)(T_len + more_rows));
  Held bytes(PyLong_FromSize_t(akvq_decode_workspace_bytes((int)B, c.Hq, most)));
  PyObject *args[3] = {cache, names.decode, bytes.p};
  Held ws(PyObject_VectorcallMethod(names.workspace, args, 3 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr));
  if (!ws.p) throw Failed();
  c.ws_tensor = tensor(ws.p);
  c.ws = c.ws_tensor.data_ptr();
  c.ws_bytes = (size_t)c.ws_tensor.numel();
  const at::ScalarType dtype = (c.flags & AKVQ_OUT_FP16) ? at::kHalf : at::kFloat;
  if (out == Py_None) c.out = at::empty({B, c.Hq, kHeadDim}, q.options().dtype(check_out ? dtype : at::kFloat).requires_grad(false));
  else c.out = tensor(out);
  if (check_out) REQUIRE(c.out.scalar_type() == dtype && c.out.is_contiguous());
  if (lse == Py_None) c.lse = at::empty({B, c.Hq}, q.options().dtype(at::kFloat).requires_grad(false));
  else c.lse = tensor(lse);
  if (rope != Py_None) {  // (a pair of two tensors: None inside it is an error)
    c.rope_pair.p = PySequence_Tuple(rope);
    if (!c.rope_pair.p) throw Failed();
    if (PyTuple_GET_SIZE(c.rope_pair.p) != 2) {
      PyErr_SetString(PyExc_ValueError, "rope has to be a pair (cos, sin)");
      throw Failed();
    }
    const at::Tensor &cos = tensor(PyTuple_GET_ITEM(c.rope_pair.p, 0)), &sin = tensor(PyTuple_GET_ITEM(c.rope_pair.p, 1));
    REQUIRE(cos.scalar_type() == at::kHalf && sin.scalar_type() == at::kHalf && cos.is_contiguous() && sin.is_contiguous());
    REQUIRE(cos.sizes() == sin.sizes() && cos.dim() >= 2 && cos.size(-2) == 1 && cos.size(-1) == 64);
    REQUIRE(cos.dim() == 2 || (cos.dim() == 3 && cos.size(0) == cache_B));
    c.rope = akvq_rope{static_cast<const uint16_t *>(cos.data_ptr()), static_cast<const uint16_t *>(sin.data_ptr()),
                       cos.dim() == 3 ? 64 : 0};
    c.rope_p = &c.rope;
  }
  c.stream = c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream();
}

PyObject *result(int status, Call &c) {
  Held out(THPVariable_Wrap(c.out)), lse(THPVariable_Wrap(c.lse));
  if (!out.p || !lse.p) return nullptr;
  return Py_BuildValue("iOO", status, out.p, lse.p);
}

// decode_attention(cache, q, sm_scale, n_split, flags, out, lse, rope) -> (status, out, lse)
PyObject *decode_attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8) {
    PyErr_SetString(PyExc_TypeError, "decode_attention takes 8 arguments");
    return nullptr;
  }
  try {
    Call c;
    gather(c, a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], 0, true);
    void *const out = c.out.data_ptr();
    float *const lse = static_cast<float *>(c.lse.data_ptr());
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = akvq_decode_attention_rope(&c.cache, c.fine_mask, c.win_p, c.q, c.rope_p, c.Hq, c.sm_scale, out, lse, c.n_split,
                                        c.ws, c.ws_bytes, c.flags, c.stream);
    Py_END_ALLOW_THREADS
    return result(status, c);
  } catch (const Failed &) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// decode_step(cache, k_new, v_new, q, clip, sm_scale, n_split, flags, out, lse, rope) -> (status, out, lse)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 11) {
    PyErr_SetString(PyExc_TypeError, "decode_step takes 11 arguments");
    return nullptr;
  }
  try {
    const at::Tensor &k = tensor(a[1]), &v = tensor(a[2]);
    REQUIRE(k.scalar_type() == at::kHalf && v.scalar_type() == at::kHalf);
    REQUIRE(k.is_contiguous() && v.is_contiguous());
    const int64_t shape[4] = {int_attr(a[0], names.B), int_attr(a[0], names.Hkv), 1, kHeadDim};
    REQUIRE(k.sizes() == at::IntArrayRef(shape, 4) && k.sizes() == v.sizes());
    const float clip = (float)number(a[4]);
    Call c;
    gather(c, a[0], a[3], a[5], a[6], a[7], a[8], a[9], a[10], 1, false);
    const void *const k_new = k.data_ptr(), *const v_new = v.data_ptr();
    void *const out = c.out.data_ptr();
    float *const lse = static_cast<float *>(c.lse.data_ptr());
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = akvq_decode_step(&c.cache, c.fine_mask, c.win_p, k_new, v_new, c.q, c.rope_p, c.Hq, clip, c.sm_scale, out, lse,
                              c.n_split, c.ws, c.ws_bytes, c.flags, c.stream);
    Py_END_ALLOW_THREADS
    return result(status, c);
  } catch (const Failed &) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// plain_cache(struct, window_struct, cache_type, window_type): the functions of the package's own cache class, and the types
// they return
PyObject *plain_cache(PyObject *, PyObject *args) {
  Plain p;
  if (!PyArg_ParseTuple(args, "OOOO", &p.struct_, &p.window_struct, &p.cache_type, &p.window_type)) return nullptr;
  for (PyObject *o : {p.struct_, p.window_struct, p.cache_type, p.window_type}) Py_INCREF(o);
  plain = p;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"plain_cache", plain_cache, METH_VARARGS, nullptr},
    {"decode_attention", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_attention)), METH_FASTCALL, nullptr},
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_akvq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__akvq_torch(void) {
  struct { PyObject **slot; const char *text; } table[] = {
      {&names.B, "B"}, {&names.Hkv, "Hkv"}, {&names.G, "G"}, {&names.T_cap, "T_cap"}, {&names.S_cap, "S_cap"},
      {&names.T_len, "T_len"}, {&names.k_codes, "k_codes"}, {&names.v_codes, "v_codes"}, {&names.k_meta, "k_meta"},
      {&names.v_meta, "v_meta"}, {&names.k_sal, "k_sal"}, {&names.v_sal, "v_sal"}, {&names.sal_idx, "sal_idx"},
      {&names.sal_cnt, "sal_cnt"}, {&names.fine_mask, "fine_mask"}, {&names.W, "W"}, {&names.k_win, "k_win"},
      {&names.v_win, "v_win"}, {&names.workspace, "workspace"}, {&names.decode, "decode"},
      {&names.struct_, "struct"}, {&names.window_struct, "window_struct"}};
  for (auto &t : table)
    if ((*t.slot = PyUnicode_InternFromString(t.text)) == nullptr) return nullptr;
  return PyModule_Create(&module);
}
