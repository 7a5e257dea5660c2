// Argument marshalling of binding.py in native code: the calls of a training or serving loop, with every tensor given
// by the caller.  A call through ctypes spends about 11 us in Python on its checks and conversions (each tensor's shape,
// type, layout and pointer; the parameter block; the stream), which is more than the GPU needs for a few short rows.
//
// Each function checks its arguments as binding.py does and calls the C ABI; it returns the error code, or None where an
// argument is missing or not as expected, and binding.py then takes its own path, which allocates or raises.
// Nothing is kept between calls.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/blossom.h"

namespace {

PyObject *g_fields[13];  // interned names of the parameter block's fields, in its order
PyObject *g_cuda_stream;
const char *kFields[13] = {"B", "H", "L", "d", "block", "topk", "window", "dtype", "softmax_scale", "stis_mode", "save_for_bwd", "stis_block",
                           "last_block_only"};

// One call's arguments, read in order; `ok` falls at the first that is not as expected.
struct Call {
  PyObject *const *arg;
  bool ok = true;
  blossom_params p{};
  at::ScalarType T{};
  int64_t NB = 0;
  void *stream = nullptr;

  explicit Call(PyObject *const *a) : arg(a) {}

  bool params()
  {
    PyObject *obj = *arg++;
    long v[13];
    for (int i = 0; i < 13 && ok; ++i) {
      PyObject *x = PyObject_GetAttr(obj, g_fields[i]);
      if (!x) return ok = false;
      if (i == 8) p.softmax_scale = (float)PyFloat_AsDouble(x);
      else v[i] = PyLong_AsLong(x);
      Py_DECREF(x);
      ok = !PyErr_Occurred() && (i == 8 || v[i] == (int32_t)v[i]);
    }
    if (!ok) return false;
    p.B = (int32_t)v[0]; p.H = (int32_t)v[1]; p.L = (int32_t)v[2]; p.d = (int32_t)v[3]; p.block = (int32_t)v[4];
    p.topk = (int32_t)v[5]; p.window = (int32_t)v[6]; p.dtype = (int32_t)v[7]; p.stis_mode = (int32_t)v[9];
    p.save_for_bwd = (int32_t)v[10]; p.stis_block = (int32_t)v[11]; p.last_block_only = (int32_t)v[12];
    if (p.block < 1) return ok = false;
    NB = ((int64_t)p.L + p.block - 1) / p.block;
    T = p.dtype == 0 ? at::kFloat : at::kBFloat16;
    return true;
  }
  int32_t whole()
  {
    const long v = PyLong_AsLong(*arg++);
    ok = ok && !PyErr_Occurred() && v == (int32_t)v;
    return (int32_t)v;
  }
  float real()
  {
    const double v = PyFloat_AsDouble(*arg++);
    ok = ok && !PyErr_Occurred();
    return (float)v;
  }
  // contiguous device tensor of this shape and type (or, if `optional`, None)
  template <typename P = void>
  P *tensor(at::IntArrayRef shape, at::ScalarType type, bool optional = false)
  {
    PyObject *obj = *arg++;
    if (obj == Py_None) {
      ok = ok && optional;
      return nullptr;
    }
    if (!ok || !THPVariable_Check(obj)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor &t = THPVariable_Unpack(obj);
    ok = t.is_cuda() && t.scalar_type() == type && t.sizes() == shape && t.is_contiguous();
    return ok ? static_cast<P *>(t.data_ptr()) : nullptr;
  }
  // any tensor; None only where `need` is 0
  void *workspace(size_t need, size_t *bytes)
  {
    PyObject *obj = *arg++;
    *bytes = 0;
    if (obj == Py_None) {
      ok = ok && need == 0;
      return nullptr;
    }
    if (!ok || !THPVariable_Check(obj)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor &t = THPVariable_Unpack(obj);
    *bytes = t.nbytes();
    return t.data_ptr();
  }
  // None: torch's current stream
  void on_stream()
  {
    PyObject *obj = *arg++;
    if (!ok) return;
    if (obj == Py_None) {
      stream = (void *)c10::hip::getCurrentHIPStream().stream();
      return;
    }
    PyObject *x = PyObject_GetAttr(obj, g_cuda_stream);
    if (x) {
      stream = PyLong_AsVoidPtr(x);
      Py_DECREF(x);
    }
    ok = !PyErr_Occurred();
  }
  template <typename F>
  PyObject *run(F &&f)
  {
    if (!ok) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  }
};

#define FASTCALL(name, count)                                                     \
  PyObject *name##_body(Call &c);                                                 \
  PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n)                 \
  {                                                                               \
    if (n != (count)) {                                                           \
      PyErr_SetString(PyExc_TypeError, #name " takes " #count " arguments");      \
      return nullptr;                                                             \
    }                                                                             \
    try {                                                                         \
      Call c(args);                                                               \
      if (!c.params()) {                                                          \
        PyErr_Clear();                                                            \
        Py_RETURN_NONE;                                                           \
      }                                                                           \
      return name##_body(c);                                                      \
    } catch (...) { /* a tensor without storage and the like: binding.py says what is wrong */ \
      PyErr_Clear();                                                              \
      Py_RETURN_NONE;                                                             \
    }                                                                             \
  }                                                                               \
  PyObject *name##_body(Call &c)

// select_blocks(p, Q, K, valid_len, sel, ws, stream)
FASTCALL(select_blocks, 7)
{
  const blossom_params &p = c.p;
  const int64_t x[4] = {p.B, p.H, p.L, p.d}, s[4] = {p.B, p.H, c.NB, p.topk}, b[1] = {p.B};
  void *Q = c.tensor(x, c.T), *K = c.tensor(x, c.T);
  int32_t *vl = c.tensor<int32_t>(b, at::kInt), *sel = c.tensor<int32_t>(s, at::kInt);
  size_t bytes;
  void *ws = c.workspace(1, &bytes);
  c.on_stream();
  return c.run([&] { return blossom_select_blocks(&p, Q, K, vl, sel, ws, bytes, c.stream); });
}

// rope_select_blocks(p, Q, K, rope_cos, rope_sin, valid_len, Q_rot, K_rot, sel, ws, stream)
FASTCALL(rope_select_blocks, 11)
{
  const blossom_params &p = c.p;
  const int64_t x[4] = {p.B, p.H, p.L, p.d}, s[4] = {p.B, p.H, c.NB, p.topk}, r[2] = {p.L, p.d / 2}, b[1] = {p.B};
  void *Q = c.tensor(x, c.T), *K = c.tensor(x, c.T);
  float *cos = c.tensor<float>(r, at::kFloat), *sin = c.tensor<float>(r, at::kFloat);
  int32_t *vl = c.tensor<int32_t>(b, at::kInt);
  void *Qr = c.tensor(x, c.T), *Kr = c.tensor(x, c.T);
  int32_t *sel = c.tensor<int32_t>(s, at::kInt);
  size_t bytes;
  void *ws = c.workspace(1, &bytes);
  c.on_stream();
  return c.run([&] { return blossom_rope_select_blocks(&p, Q, K, cos, sin, vl, Qr, Kr, sel, ws, bytes, c.stream); });
}

// select_positions(p, kv_groups, cmp_block, cmp_stride, Q, K, valid_len, score_scale, sel_pos, ws, stream)
FASTCALL(select_positions, 11)
{
  const blossom_params &p = c.p;
  const int32_t G = c.whole(), l = c.whole(), st = c.whole();
  const int64_t q[4] = {p.B, p.H, p.L, p.d}, k[4] = {p.B, G, p.L, p.d}, s[4] = {p.B, G, p.L, p.topk}, b[1] = {p.B};
  void *Q = c.tensor(q, c.T), *K = c.tensor(k, c.T);
  int32_t *vl = c.tensor<int32_t>(b, at::kInt);
  const float scale = c.real();
  int32_t *sel = c.tensor<int32_t>(s, at::kInt);
  size_t bytes;
  void *ws = c.workspace(1, &bytes);
  c.on_stream();
  return c.run([&] { return blossom_select_positions(&p, G, l, st, scale, Q, K, vl, sel, ws, bytes, c.stream); });
}

// The forward's arguments from Q on: G key/value groups, selection rows of shape `s`.
struct FwdTensors {
  void *Q, *K, *V;
  int32_t *vl, *sel;
  float *gw, *gb;
  void *O;
  float *o_lt, *o_st, *lse_lt, *lse_st;
  FwdTensors(Call &c, int64_t G, at::IntArrayRef s)
  {
    const blossom_params &p = c.p;
    const int64_t x[4] = {p.B, p.H, p.L, p.d}, k[4] = {p.B, G, p.L, p.d}, b[1] = {p.B}, w[2] = {p.H, 2 * (int64_t)p.d}, h[1] = {p.H};
    const at::IntArrayRef row(x, 3);
    Q = c.tensor(x, c.T);
    K = c.tensor(k, c.T);
    V = c.tensor(k, c.T);
    vl = c.tensor<int32_t>(b, at::kInt);
    sel = c.tensor<int32_t>(s, at::kInt);
    gw = c.tensor<float>(w, at::kFloat);
    gb = c.tensor<float>(h, at::kFloat, true);
    O = c.tensor(x, c.T);
    o_lt = c.tensor<float>(x, at::kFloat, true);
    o_st = c.tensor<float>(x, at::kFloat, true);
    lse_lt = c.tensor<float>(row, at::kFloat, true);
    lse_st = c.tensor<float>(row, at::kFloat, true);
  }
};

// attn_fwd(p, Q, K, V, valid_len, sel, gate_w, gate_b, O, o_lt, o_st, lse_lt, lse_st, ws, stream)
FASTCALL(attn_fwd, 15)
{
  const blossom_params &p = c.p;
  const int64_t s[4] = {p.B, p.H, c.NB, p.topk};
  const FwdTensors t(c, p.H, s);
  size_t bytes;
  void *ws = c.workspace(blossom_workspace_bytes(&p, BLOSSOM_WS_FWD), &bytes);
  c.on_stream();
  return c.run([&] {
    return blossom_attn_fwd(&p, t.Q, t.K, t.V, t.vl, t.sel, t.gw, t.gb, t.O, t.o_lt, t.o_st, t.lse_lt, t.lse_st, ws, bytes, c.stream);
  });
}

// attn_fwd_positions(p, kv_groups, Q, K, V, valid_len, sel_pos, gate_w, gate_b, O, o_lt, o_st, lse_lt, lse_st, stream)
FASTCALL(attn_fwd_positions, 15)
{
  const blossom_params &p = c.p;
  const int32_t G = c.whole();
  const int64_t s[4] = {p.B, G, p.L, p.topk};
  const FwdTensors t(c, G, s);
  c.on_stream();
  return c.run([&] {
    return blossom_attn_fwd_positions(&p, G, t.Q, t.K, t.V, t.vl, t.sel, t.gw, t.gb, t.O, t.o_lt, t.o_st, t.lse_lt, t.lse_st, c.stream);
  });
}

// The backward's arguments from Q on.
struct BwdTensors {
  void *Q, *K, *V;
  int32_t *vl, *sel;
  float *gw, *gb, *o_lt, *o_st, *lse_lt, *lse_st;
  void *dO, *dQ, *dK, *dV;
  float *dgw, *dgb;
  void *ws;
  size_t bytes;
  BwdTensors(Call &c, int64_t G, at::IntArrayRef s)
  {
    const blossom_params &p = c.p;
    const int64_t x[4] = {p.B, p.H, p.L, p.d}, k[4] = {p.B, G, p.L, p.d}, b[1] = {p.B}, w[2] = {p.H, 2 * (int64_t)p.d}, h[1] = {p.H};
    const at::IntArrayRef row(x, 3);
    Q = c.tensor(x, c.T);
    K = c.tensor(k, c.T);
    V = c.tensor(k, c.T);
    vl = c.tensor<int32_t>(b, at::kInt);
    sel = c.tensor<int32_t>(s, at::kInt);
    gw = c.tensor<float>(w, at::kFloat);
    gb = c.tensor<float>(h, at::kFloat, true);
    o_lt = c.tensor<float>(x, at::kFloat);
    o_st = c.tensor<float>(x, at::kFloat);
    lse_lt = c.tensor<float>(row, at::kFloat);
    lse_st = c.tensor<float>(row, at::kFloat);
    dO = c.tensor(x, c.T);
    dQ = c.tensor(x, c.T);
    dK = c.tensor(k, c.T);
    dV = c.tensor(k, c.T);
    dgw = c.tensor<float>(w, at::kFloat);
    dgb = c.tensor<float>(h, at::kFloat);
    ws = c.workspace(1, &bytes);
  }
};

// attn_bwd(p, Q, K, V, valid_len, sel, gate_w, gate_b, o_lt, o_st, lse_lt, lse_st, dO, dQ, dK, dV, d_gate_w, d_gate_b, ws,
//          rope_cos, rope_sin, stream); both tables None: blossom_attn_bwd, else blossom_attn_bwd_rope
FASTCALL(attn_bwd, 22)
{
  const blossom_params &p = c.p;
  const int64_t s[4] = {p.B, p.H, c.NB, p.topk}, r[2] = {p.L, p.d / 2};
  const BwdTensors t(c, p.H, s);
  float *cos = c.tensor<float>(r, at::kFloat, true), *sin = c.tensor<float>(r, at::kFloat, true);
  c.ok = c.ok && !cos == !sin;
  c.on_stream();
  return c.run([&] {
    if (cos)
      return blossom_attn_bwd_rope(&p, t.Q, t.K, t.V, t.vl, t.sel, t.gw, t.gb, t.o_lt, t.o_st, t.lse_lt, t.lse_st, t.dO, cos, sin,
                                   t.dQ, t.dK, t.dV, t.dgw, t.dgb, t.ws, t.bytes, c.stream);
    return blossom_attn_bwd(&p, t.Q, t.K, t.V, t.vl, t.sel, t.gw, t.gb, t.o_lt, t.o_st, t.lse_lt, t.lse_st, t.dO, t.dQ, t.dK, t.dV,
                            t.dgw, t.dgb, t.ws, t.bytes, c.stream);
  });
}

// attn_bwd_positions(p, kv_groups, Q, K, V, valid_len, sel_pos, gate_w, gate_b, o_lt, o_st, lse_lt, lse_st, dO, dQ, dK, dV,
//                    d_gate_w, d_gate_b, ws, stream)
FASTCALL(attn_bwd_positions, 21)
{
  const blossom_params &p = c.p;
  const int32_t G = c.whole();
  const int64_t s[4] = {p.B, G, p.L, p.topk};
  const BwdTensors t(c, G, s);
  c.on_stream();
  return c.run([&] {
    return blossom_attn_bwd_positions(&p, G, t.Q, t.K, t.V, t.vl, t.sel, t.gw, t.gb, t.o_lt, t.o_st, t.lse_lt, t.lse_st, t.dO, t.dQ,
                                      t.dK, t.dV, t.dgw, t.dgb, t.ws, t.bytes, c.stream);
  });
}

// out_proj_ln(p, d_model, O, W_O_t, bias, H_prev, ln_gamma, ln_beta, ln_eps, S, mean, rstd, stream)
FASTCALL(out_proj_ln, 13)
{
  const blossom_params &p = c.p;
  const int32_t dm = c.whole();
  const int64_t x[4] = {p.B, p.H, p.L, p.d}, w[2] = {dm, (int64_t)p.H * p.d}, h[3] = {p.B, p.L, dm}, g[1] = {dm};
  const at::IntArrayRef row(h, 2);
  void *O = c.tensor(x, c.T), *W = c.tensor(w, c.T);
  float *bias = c.tensor<float>(g, at::kFloat, true);
  void *prev = c.tensor(h, c.T);
  float *gamma = c.tensor<float>(g, at::kFloat), *beta = c.tensor<float>(g, at::kFloat);
  const float eps = c.real();
  void *S = c.tensor(h, c.T);
  float *mean = c.tensor<float>(row, at::kFloat, true), *rstd = c.tensor<float>(row, at::kFloat, true);
  c.on_stream();
  return c.run([&] { return blossom_out_proj_ln(&p, dm, O, W, bias, prev, gamma, beta, eps, S, mean, rstd, c.stream); });
}

#define ENTRY(name) {#name, (PyCFunction)(void *)name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {ENTRY(select_blocks), ENTRY(rope_select_blocks), ENTRY(select_positions), ENTRY(attn_fwd),
                          ENTRY(attn_fwd_positions), ENTRY(attn_bwd), ENTRY(attn_bwd_positions), ENTRY(out_proj_ln),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
  for (int i = 0; i < 13; ++i)
    if (!(g_fields[i] = PyUnicode_InternFromString(kFields[i]))) return nullptr;
  if (!(g_cuda_stream = PyUnicode_InternFromString("cuda_stream"))) return nullptr;
  return PyModule_Create(&kModule);
}
