// Native argument marshalling of the Python binding (ssdi8.py): checks the tensors, allocates the
// outputs with PyTorch and calls the C ABI, for the calls a program makes per layer or per token.
// A small layer's kernels take 20 to 40 us; the same checks through Python objects and ctypes cost
// 12 us per quantize_act, 22 us per ssd_chunk_scan.
//
// Each entry returns None when an argument is not of the plain form it takes (wrong type, device,
// dtype, shape, layout; a tensor subclass; memory that cannot be allocated), before anything is
// launched: the caller then takes the Python path, which raises the error that belongs to it (or
// accepts what is allowed there).  The GIL is released during the library call.
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ssdi8.h"

namespace {

decltype(&ssdi8_quantize_act) g_quantize = nullptr;
decltype(&ssdi8_ssd_workspace_size) g_workspace_size = nullptr;
decltype(&ssdi8_ssd_chunk_scan) g_scan = nullptr;
decltype(&ssdi8_decode_step) g_decode = nullptr;
c10::DeviceType g_device = c10::DeviceType::CUDA;   // where its tensors live

// Thrown (and caught at the entry) for arguments that belong to the Python path.
struct NotPlain {};

struct Shape {
  int64_t v[5];
  int n;
  Shape(std::initializer_list<int64_t> l) : n((int)l.size()) { std::copy(l.begin(), l.end(), v); }
};

const at::Tensor& any_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain();
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || t.device().type() != g_device ||
      !t.is_contiguous())
    throw NotPlain();
  return t;
}
const at::Tensor& tensor(PyObject* o, at::ScalarType dtype) {
  const at::Tensor& t = any_tensor(o);
  if (t.scalar_type() != dtype) throw NotPlain();
  return t;
}
bool has_shape(const at::Tensor& t, const Shape& s) {
  return t.dim() == s.n && std::equal(s.v, s.v + s.n, t.sizes().begin());
}
void* shaped(PyObject* o, at::ScalarType dtype, const Shape& s) {
  const at::Tensor& t = tensor(o, dtype);
  if (!has_shape(t, s)) throw NotPlain();
  return t.data_ptr();
}
float* floats(PyObject* o, const Shape& s) {
  return static_cast<float*>(shaped(o, at::kFloat, s));
}
float* floats_or_null(PyObject* o, const Shape& s) { return o == Py_None ? nullptr : floats(o, s); }
int float_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kHalf) return SSDI8_F16;
  if (t.scalar_type() == at::kFloat) return SSDI8_F32;
  throw NotPlain();
}
int64_t integer(PyObject* o) {
  if (!PyLong_Check(o)) throw NotPlain();   // bool is a PyLong
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw NotPlain();
  return v;
}
// No GIL while this lives; it is back also where an exception leaves.
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};
// An allocation may wait for the device, and the device for a host callback that takes the GIL.
at::Tensor empty(const at::Tensor& like, at::ScalarType dtype, std::initializer_list<int64_t> s) {
  NoGil no_gil;
  return at::empty(s, like.options().dtype(dtype).requires_grad(false));
}
// The library call.  Tensors are looked at before: data_ptr() throws for one without storage (a
// functorch wrapper).
template <typename F> ssdi8_status released(F&& f) {
  NoGil no_gil;
  return f();
}
template <typename F> PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (...) {   // NotPlain, c10 errors (allocation): the Python path decides
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}
void* stream_of(PyObject* o) { return reinterpret_cast<void*>((uintptr_t)integer(o)); }

// bind(quantize, workspace_size, scan, decode, device): the library's addresses and the type of the
// device its tensors live on
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  const char* device = n == 5 ? PyUnicode_AsUTF8(a[4]) : nullptr;
  if (!device) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "bind takes 4 addresses and a device");
    return nullptr;
  }
  void* p[4];
  for (int i = 0; i < 4; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  g_quantize = reinterpret_cast<decltype(g_quantize)>(p[0]);
  g_workspace_size = reinterpret_cast<decltype(g_workspace_size)>(p[1]);
  g_scan = reinterpret_cast<decltype(g_scan)>(p[2]);
  g_decode = reinterpret_cast<decltype(g_decode)>(p[3]);
  try {
    g_device = c10::Device(device).type();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_ValueError, e.what());
    return nullptr;
  }
  Py_RETURN_NONE;
}

// quantize(src, gran, scale or None, out or None, stream) -> (status, out, scale)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 5 || !g_quantize) throw NotPlain();
    const at::Tensor& src = any_tensor(a[0]);
    const int code = float_code(src);
    if (src.dim() != 4) throw NotPlain();
    const int64_t b = src.size(0), l = src.size(1), k = src.size(2), m = src.size(3);
    const int gran = (int)integer(a[1]);
    int64_t ns;
    switch (gran) {
      case SSDI8_GRAN_TENSOR: ns = 1; break;
      case SSDI8_GRAN_GROUP: ns = k; break;
      case SSDI8_GRAN_CHANNEL: ns = k * m; break;
      case SSDI8_GRAN_TOKEN: ns = b * l * k; break;
      default: throw NotPlain();
    }
    const bool dynamic = a[2] == Py_None;
    at::Tensor scale = dynamic ? empty(src, at::kFloat, {ns}) : tensor(a[2], at::kFloat);
    if (scale.numel() != ns) throw NotPlain();
    at::Tensor out = a[3] == Py_None ? empty(src, at::kChar, {b, l, k, m}) : tensor(a[3], at::kChar);
    if (!has_shape(out, {b, l, k, m})) throw NotPlain();
    void* st = stream_of(a[4]);
    const void* from = src.data_ptr();
    float* steps = static_cast<float*>(scale.data_ptr());
    int8_t* to = static_cast<int8_t*>(out.data_ptr());
    const ssdi8_status s = released([&] {
      return g_quantize(from, code, b, l, k, m, gran, steps, dynamic ? 1 : 0, to, st);
    });
    return Py_BuildValue("(iNN)", (int)s, THPVariable_Wrap(out), THPVariable_Wrap(scale));
  });
}

// scan(x, dt, A, Bq, Cq, B, C, B_scale, C_scale, xs_scale, state_scale, cb_scale, D, corr, init,
//      y or None, y_dtype (-1: that of x), workspace or None, timeouts or None, dt_softplus,
//      chunk, decay_shift, shift_round, final_state, path, stream)
//   -> (status, y, final_state_q or None, final_state or None)
PyObject* scan(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 26 || !g_scan) throw NotPlain();
    ssdi8_scan_args a = {};
    const at::Tensor& x = any_tensor(o[0]);
    if (x.dim() != 4) throw NotPlain();
    const int64_t B = x.size(0), L = x.size(1), H = x.size(2), P = x.size(3);
    a.x = x.data_ptr();
    a.x_dtype = float_code(x);
    const bool quantized = o[3] != Py_None;
    if (quantized ? (o[4] == Py_None || o[6] != Py_None) : (o[5] == Py_None || o[6] == Py_None))
      throw NotPlain();
    const at::Tensor& b = any_tensor(o[quantized ? 3 : 5]);
    const at::Tensor& c = any_tensor(o[quantized ? 4 : 6]);
    if (b.dim() != 4 || c.scalar_type() != b.scalar_type()) throw NotPlain();
    const int64_t G = b.size(2), N = b.size(3);
    if (!has_shape(b, {B, L, G, N}) || !has_shape(c, {B, L, G, N})) throw NotPlain();
    if (quantized) {
      if (b.scalar_type() != at::kChar) throw NotPlain();
      a.Bq = static_cast<const int8_t*>(b.data_ptr());
      a.Cq = static_cast<const int8_t*>(c.data_ptr());
    } else {
      a.bc_dtype = float_code(b);
      a.B = b.data_ptr();
      a.C = c.data_ptr();
    }
    a.dt = floats(o[1], {B, L, H});
    a.A = floats(o[2], {H});
    a.B_scale = floats(o[7], {G});
    a.c_per_token = tensor(o[8], at::kFloat).dim() == 3;
    a.C_scale = a.c_per_token ? floats(o[8], {B, L, G}) : floats(o[8], {G});
    a.xs_per_head = tensor(o[9], at::kFloat).dim() == 1;
    a.xs_scale = a.xs_per_head ? floats(o[9], {H}) : floats(o[9], {H, P});
    a.state_scale = floats(o[10], {H, P});
    a.cb_scale = floats(o[11], {G});
    a.D = floats_or_null(o[12], {H});
    a.corr = floats_or_null(o[13], {H, P});
    if (o[14] != Py_None)
      a.init_state_q = static_cast<const int8_t*>(shaped(o[14], at::kChar, {B, H, P, N}));
    if (o[18] != Py_None) a.hand_off_timeouts = static_cast<int*>(shaped(o[18], at::kInt, {1}));
    a.dt_softplus = (int)integer(o[19]);
    const ssdi8_dims d = {B, L, H, P, G, N, integer(o[20])};
    a.decay_shift = (int)integer(o[21]);
    a.shift_round = (int)integer(o[22]);
    a.path = (int)integer(o[24]);
    void* st = stream_of(o[25]);
    // allocations last
    const int64_t yd = integer(o[16]);
    a.y_dtype = yd < 0 ? a.x_dtype : (int)yd;
    const at::ScalarType ydt = a.y_dtype == SSDI8_F16 ? at::kHalf : at::kFloat;
    at::Tensor y = o[15] == Py_None ? empty(x, ydt, {B, L, H, P}) : tensor(o[15], ydt);
    if (!has_shape(y, {B, L, H, P})) throw NotPlain();
    a.y = y.data_ptr();
    const int64_t need = (int64_t)g_workspace_size(&d);
    at::Tensor ws = o[17] == Py_None ? empty(x, at::kByte, {need > 1 ? need : 1})
                                     : tensor(o[17], at::kByte);
    a.workspace = ws.data_ptr();
    a.workspace_bytes = (size_t)ws.numel();
    at::Tensor fq, fs;
    if (integer(o[23])) {
      fq = empty(x, at::kChar, {B, H, P, N});
      fs = empty(x, at::kFloat, {B, H, P, N});
      a.final_state_q = static_cast<int8_t*>(fq.data_ptr());
      a.final_state = static_cast<float*>(fs.data_ptr());
    }
    const ssdi8_status s = released([&] { return g_scan(&d, &a, st); });
    auto wrap = [](const at::Tensor& t) {
      if (t.defined()) return THPVariable_Wrap(t);
      Py_INCREF(Py_None);
      return Py_None;
    };
    return Py_BuildValue("(iNNN)", (int)s, wrap(y), wrap(fq), wrap(fs));
  });
}

// decode(x, dt, A, Bq, Cq, B_scale, C_scale, xs_scale, state_scale, cb_scale, state_q, D, corr,
//        dt_softplus, decay_shift, shift_round, y or None, y_dtype (-1: that of x), stream)
//   -> (status, y)
PyObject* decode(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 19 || !g_decode) throw NotPlain();
    ssdi8_decode_args a = {};
    const at::Tensor& x = any_tensor(o[0]);
    if (x.dim() != 3) throw NotPlain();
    const int64_t B = x.size(0), H = x.size(1), P = x.size(2);
    a.x = x.data_ptr();
    a.x_dtype = float_code(x);
    const at::Tensor& b = tensor(o[3], at::kChar);
    if (b.dim() != 3) throw NotPlain();
    const int64_t G = b.size(1), N = b.size(2);
    a.Bq = static_cast<const int8_t*>(shaped(o[3], at::kChar, {B, G, N}));
    a.Cq = static_cast<const int8_t*>(shaped(o[4], at::kChar, {B, G, N}));
    a.dt = floats(o[1], {B, H});
    a.A = floats(o[2], {H});
    a.B_scale = floats(o[5], {G});
    a.c_per_token = tensor(o[6], at::kFloat).dim() == 2;
    a.C_scale = a.c_per_token ? floats(o[6], {B, G}) : floats(o[6], {G});
    a.xs_per_head = tensor(o[7], at::kFloat).dim() == 1;
    a.xs_scale = a.xs_per_head ? floats(o[7], {H}) : floats(o[7], {H, P});
    a.state_scale = floats(o[8], {H, P});
    a.cb_scale = floats(o[9], {G});
    a.state_q = static_cast<int8_t*>(shaped(o[10], at::kChar, {B, H, P, N}));
    a.D = floats_or_null(o[11], {H});
    a.corr = floats_or_null(o[12], {H, P});
    a.dt_softplus = (int)integer(o[13]);
    a.decay_shift = (int)integer(o[14]);
    a.shift_round = (int)integer(o[15]);
    void* st = stream_of(o[18]);
    const int64_t yd = integer(o[17]);
    a.y_dtype = yd < 0 ? a.x_dtype : (int)yd;
    const at::ScalarType ydt = a.y_dtype == SSDI8_F16 ? at::kHalf : at::kFloat;
    at::Tensor y = o[16] == Py_None ? empty(x, ydt, {B, H, P}) : tensor(o[16], ydt);
    if (!has_shape(y, {B, H, P})) throw NotPlain();
    a.y = y.data_ptr();
    const ssdi8_status s = released([&] { return g_decode(B, H, P, G, N, &a, st); });
    return Py_BuildValue("(iN)", (int)s, THPVariable_Wrap(y));
  });
}

#define SSDI8_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", SSDI8_FAST(bind), "bind(quantize_act, ssd_workspace_size, ssd_chunk_scan, decode_step, device)"},
    {"quantize", SSDI8_FAST(quantize), "ssdi8_quantize_act"},
    {"scan", SSDI8_FAST(scan), "ssdi8_ssd_chunk_scan"},
    {"decode", SSDI8_FAST(decode), "ssdi8_decode_step"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
