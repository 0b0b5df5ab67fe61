// Python's way into the C ABI: checks and unpacks torch tensors in native code.  A call takes up to 12
// of them, and looking at one through the interpreter costs 0.45 us, as much as a launch costs for
// five; here it is 0.01 us.  Nothing is computed here and nothing is kept between calls.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/stc.h"

namespace {

PyObject* g_error;       // StcError(status, where)
PyObject* g_shape;       // stc_shape_t
PyObject* g_device;      // torch._C._cuda_getDevice
PyObject* g_raw_stream;  // torch._C._cuda_getCurrentRawStream, which takes the device
PyObject* g_any_stream;  // the package's own way, for builds of torch without these two

struct PythonError {};  // the interpreter's error is set

constexpr at::ScalarType kBf16 = at::kBFloat16, kF32 = at::kFloat, kU8 = at::kByte;

// The arguments of one call, in order.
class Args {
 public:
  Args(const char* where, PyObject* const* args, Py_ssize_t n, Py_ssize_t want)
      : where_(where), args_(args) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, not %zd", where, want, n);
      throw PythonError();
    }
  }

  const stc_shape_t* shape() {
    PyObject* o = next();
    const int is = PyObject_IsInstance(o, g_shape);
    if (is == 0) PyErr_Format(PyExc_TypeError, "%s: shape must be a stc_shape_t", where_);
    Py_buffer b;
    if (is != 1 || PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw PythonError();
    memcpy(&shape_, b.buf, sizeof shape_);  // a subclass can only be larger
    PyBuffer_Release(&b);
    return &shape_;
  }

  // Device pointer of a contiguous tensor (None: nullptr) of one of the given types.
  template <class... T>
  void* tensor(const char* name, T... types) {
    PyObject* o = next();
    bytes_ = 0;
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda()) {
      PyErr_Format(PyExc_TypeError, "%s must be a CUDA tensor", name);
      throw PythonError();
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_contiguous()) {
      PyErr_Format(PyExc_ValueError, "%s must be contiguous", name);
      throw PythonError();
    }
    if (sizeof...(T) > 0 && !((t.scalar_type() == types) || ...)) {
      PyObject* dtype = PyObject_GetAttrString(o, "dtype");
      if (dtype) PyErr_Format(PyExc_TypeError, "%s has dtype %S", name, dtype);
      Py_XDECREF(dtype);
      throw PythonError();
    }
    bytes_ = (size_t)t.numel() * t.element_size();
    return t.data_ptr();
  }
  void* bf16(const char* name) { return tensor(name, kBf16); }
  float* f32(const char* name) { return (float*)tensor(name, kF32); }
  uint8_t* u8(const char* name) { return (uint8_t*)tensor(name, kU8); }
  uint16_t* u16(const char* name) { return (uint16_t*)tensor(name, at::kShort, at::kUInt16); }
  uint32_t* u32(const char* name) { return (uint32_t*)tensor(name, at::kInt, at::kUInt32); }
  int32_t* i32(const char* name) { return (int32_t*)tensor(name, at::kInt); }
  void* ws() { return tensor("ws"); }
  size_t bytes() const { return bytes_; }  // of the tensor taken last

  // What int() takes; index(): whole numbers only.
  int integer() { return number(PyNumber_Long); }
  int index() { return number(PyNumber_Index); }

  // The current stream of the current device.
  void* stream() {
    PyObject* s = nullptr;
    if (g_device && g_raw_stream) {
      PyObject* dev = PyObject_CallNoArgs(g_device);
      if (dev) s = PyObject_CallOneArg(g_raw_stream, dev);
      Py_XDECREF(dev);
    } else {
      s = PyObject_CallNoArgs(g_any_stream);
    }
    if (!s) throw PythonError();
    void* p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw PythonError();
    return p;
  }

 private:
  PyObject* next() { return args_[at_++]; }
  int number(PyObject* (*convert)(PyObject*)) {
    PyObject* o = next();
    PyObject* i = PyLong_CheckExact(o) ? Py_NewRef(o) : convert(o);
    if (!i) throw PythonError();
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    if (v == ~0ull && PyErr_Occurred()) throw PythonError();
    return (int)v;
  }
  const char* where_;
  PyObject* const* args_;
  Py_ssize_t at_ = 0;
  stc_shape_t shape_;
  size_t bytes_ = 0;
};

// Runs `body`, which takes the arguments in order and returns the call to make; the call runs without
// the interpreter's lock.  A status other than STC_OK raises StcError.
template <class Body>
PyObject* run(const char* where, PyObject* const* args, Py_ssize_t n, Py_ssize_t want, Body body) {
  try {
    Args a(where, args, n, want);
    auto call = body(a);
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    if (status != STC_OK) {
      PyObject* e = PyObject_CallFunction(g_error, "is", status, where);
      if (e) PyErr_SetObject(g_error, e);
      Py_XDECREF(e);
      return nullptr;
    }
    Py_RETURN_NONE;
  } catch (const PythonError&) {
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

#define STC_PY(name, want, ...)                                                           \
  PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t n) {                        \
    return run("stc_" #name, args, n, want, [](Args& a) { __VA_ARGS__ });                 \
  }

STC_PY(build_page_bounds, 3,
  auto s = *a.shape(); auto K = a.bf16("K"); auto bounds = a.bf16("bounds"); auto st = a.stream();
  return [=] { return stc_build_page_bounds(&s, K, bounds, st); };)

STC_PY(route_and_pack_values, 12,
  auto s = *a.shape(); auto mode = a.index(); auto V = a.bf16("V"); auto logits = a.f32("logits");
  auto kcount = a.u8("kcount"); auto fixed_k = a.integer(); auto mask_in = a.u16("mask_in");
  auto mask = a.u16("mask"); auto off = a.u32("tok_off"); auto vpacked = a.bf16("vpacked");
  auto status = a.i32("dev_status"); auto ws = a.ws(); auto nws = a.bytes(); auto st = a.stream();
  return [=] { return stc_route_and_pack_values(&s, mode, V, logits, kcount, fixed_k, mask_in, mask, off, vpacked, status, ws, nws, st); };)

#define STC_PY_SELECT(name)                                                                        \
  STC_PY(name, 7,                                                                                  \
    auto s = *a.shape(); auto q = a.bf16("q"); auto bounds = a.bf16("bounds"); auto k = a.integer(); \
    auto idx = a.i32("page_idx"); auto score = a.f32("page_score"); auto ws = a.ws();              \
    auto nws = a.bytes(); auto st = a.stream();                                                    \
    return [=] { return stc_##name(&s, q, bounds, k, idx, score, ws, nws, st); };)
STC_PY_SELECT(select_pages)
STC_PY_SELECT(select_pages_per_head)

STC_PY(score_pages, 4,
  auto s = *a.shape(); auto q = a.bf16("q"); auto bounds = a.bf16("bounds");
  auto score = a.f32("page_score"); auto st = a.stream();
  return [=] { return stc_score_pages(&s, q, bounds, score, st); };)

#define STC_PY_ATTENTION(name)                                                                     \
  STC_PY(name, 10,                                                                                 \
    auto s = *a.shape(); auto q = a.bf16("q"); auto K = a.bf16("K"); auto v = a.bf16("vpacked");   \
    auto mask = a.u16("mask"); auto off = a.u32("tok_off"); auto idx = a.i32("page_idx");          \
    auto k = a.integer(); auto out = a.f32("out"); auto ws = a.ws(); auto nws = a.bytes();         \
    auto st = a.stream();                                                                          \
    return [=] { return stc_##name(&s, q, K, v, mask, off, idx, k, out, ws, nws, st); };)
STC_PY_ATTENTION(decode_attention)
STC_PY_ATTENTION(decode_attention_per_head)

STC_PY(decode_attention_tail, 14,
  auto s = *a.shape(); auto q = a.bf16("q"); auto K = a.bf16("K"); auto v = a.bf16("vpacked");
  auto mask = a.u16("mask"); auto off = a.u32("tok_off"); auto idx = a.i32("page_idx");
  auto k = a.integer(); auto Kt = a.bf16("K_tail"); auto Vt = a.bf16("V_tail");
  auto n_tail = a.integer(); auto cap = a.integer(); auto out = a.f32("out"); auto ws = a.ws();
  auto nws = a.bytes(); auto st = a.stream();
  return [=] { return stc_decode_attention_tail(&s, q, K, v, mask, off, idx, k, Kt, Vt, n_tail, cap, out, ws, nws, st); };)

STC_PY(decode_attention_union, 11,
  auto s = *a.shape(); auto q = a.bf16("q"); auto K = a.bf16("K"); auto v = a.bf16("vpacked");
  auto mask = a.u16("mask"); auto off = a.u32("tok_off"); auto idx = a.i32("union_idx");
  auto heads = a.u16("union_heads"); auto cap = a.integer(); auto out = a.f32("out");
  auto ws = a.ws(); auto nws = a.bytes(); auto st = a.stream();
  return [=] { return stc_decode_attention_union(&s, q, K, v, mask, off, idx, heads, cap, out, ws, nws, st); };)

STC_PY(union_pages, 6,
  auto s = *a.shape(); auto lists = a.i32("page_idx_per_head"); auto k = a.integer();
  auto idx = a.i32("union_idx"); auto heads = a.u16("union_heads"); auto cap = a.integer();
  auto st = a.stream();
  return [=] { return stc_union_pages(&s, lists, k, idx, heads, cap, st); };)

STC_PY(decode_step, 11,
  auto s = *a.shape(); auto q = a.bf16("q"); auto bounds = a.bf16("bounds"); auto K = a.bf16("K");
  auto v = a.bf16("vpacked"); auto mask = a.u16("mask"); auto off = a.u32("tok_off");
  auto k = a.integer(); auto idx = a.i32("page_idx"); auto out = a.f32("out"); auto ws = a.ws();
  auto nws = a.bytes(); auto st = a.stream();
  return [=] { return stc_decode_step(&s, q, bounds, K, v, mask, off, k, idx, out, ws, nws, st); };)

STC_PY(decode_step_static, 10,
  auto s = *a.shape(); auto q = a.bf16("q"); auto bounds = a.bf16("bounds"); auto K = a.bf16("K");
  auto v = a.bf16("vpacked"); auto mask = a.u16("mask"); auto off = a.u32("tok_off");
  auto k = a.integer(); auto idx = a.i32("page_idx"); auto out = a.f32("out"); auto st = a.stream();
  return [=] { return stc_decode_step_static(&s, q, bounds, K, v, mask, off, k, idx, out, st); };)

STC_PY(decode_step_tail, 15,
  auto s = *a.shape(); auto q = a.bf16("q"); auto bounds = a.bf16("bounds"); auto K = a.bf16("K");
  auto v = a.bf16("vpacked"); auto mask = a.u16("mask"); auto off = a.u32("tok_off");
  auto k = a.integer(); auto Kt = a.bf16("K_tail"); auto Vt = a.bf16("V_tail");
  auto n_tail = a.integer(); auto cap = a.integer(); auto idx = a.i32("page_idx");
  auto out = a.f32("out"); auto ws = a.ws(); auto nws = a.bytes(); auto st = a.stream();
  return [=] { return stc_decode_step_tail(&s, q, bounds, K, v, mask, off, k, Kt, Vt, n_tail, cap, idx, out, ws, nws, st); };)

STC_PY(flush_tail, 17,
  auto s = *a.shape(); auto Kt = a.bf16("K_tail"); auto Vt = a.bf16("V_tail"); auto nf = a.integer();
  auto n_tail = a.integer(); auto cap = a.integer(); auto mode = a.integer();
  auto logits = a.f32("logits"); auto kcount = a.u8("kcount"); auto fixed_k = a.integer();
  auto mask_in = a.u16("mask_in"); auto K = a.bf16("K"); auto bounds = a.bf16("bounds");
  auto mask = a.u16("mask"); auto off = a.u32("tok_off"); auto v = a.bf16("vpacked");
  auto status = a.i32("dev_status"); auto st = a.stream();
  return [=] { return stc_flush_tail(&s, Kt, Vt, nf, n_tail, cap, mode, logits, kcount, fixed_k, mask_in, K, bounds, mask, off, v, status, st); };)

STC_PY(append_tail, 7,
  auto s = *a.shape(); auto k = a.bf16("k_new"); auto v = a.bf16("v_new"); auto Kt = a.bf16("K_tail");
  auto Vt = a.bf16("V_tail"); auto n_tail = a.integer(); auto cap = a.integer(); auto st = a.stream();
  return [=] { return stc_append_tail(&s, k, v, Kt, Vt, n_tail, cap, st); };)

STC_PY(router_logits, 10,
  auto B = a.index(); auto Hkv = a.index(); auto N = a.index(); auto dm = a.index();
  auto G = a.index(); auto h = a.bf16("h"); auto W = a.bf16("W"); auto bias = a.f32("bias");
  auto per = a.integer(); auto logits = a.f32("logits"); auto st = a.stream();
  return [=] { return stc_router_logits(B, Hkv, N, dm, G, h, W, bias, per, logits, st); };)

STC_PY(compact_tokens, 9,
  auto src = a.bf16("src"); auto idx = a.i32("token_idx"); auto dst = a.bf16("dst");
  auto B = a.index(); auto Hkv = a.index(); auto N = a.index(); auto keep = a.index();
  auto D = a.index(); auto status = a.i32("dev_status"); auto st = a.stream();
  return [=] { return stc_compact_tokens(src, idx, dst, B, Hkv, N, keep, D, status, st); };)

PyMethodDef methods[] = {
#define STC_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
    STC_METHOD(build_page_bounds), STC_METHOD(route_and_pack_values), STC_METHOD(select_pages),
    STC_METHOD(select_pages_per_head), STC_METHOD(score_pages), STC_METHOD(decode_attention),
    STC_METHOD(decode_attention_per_head), STC_METHOD(decode_attention_tail),
    STC_METHOD(decode_attention_union), STC_METHOD(union_pages), STC_METHOD(decode_step),
    STC_METHOD(decode_step_static), STC_METHOD(decode_step_tail), STC_METHOD(flush_tail),
    STC_METHOD(append_tail), STC_METHOD(router_logits), STC_METHOD(compact_tokens),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The module takes what it needs of Python from its package when it is loaded.
PyMODINIT_FUNC PyInit__binding() {
  PyObject* torch_c = PyImport_ImportModule("torch._C");
  PyObject* pkg = PyImport_ImportModule("paper_2604_21335_amd");
  if (torch_c && pkg) {
    g_error = PyObject_GetAttrString(pkg, "StcError");
    g_shape = PyObject_GetAttrString(pkg, "stc_shape_t");
    g_any_stream = PyObject_GetAttrString(pkg, "_current_stream");
    if (g_error && g_shape && g_any_stream) {
      g_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
      if (g_device) g_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
      PyErr_Clear();
    }
  }
  Py_XDECREF(torch_c);
  Py_XDECREF(pkg);
  return g_error && g_shape && g_any_stream ? PyModule_Create(&module_def) : nullptr;
}
