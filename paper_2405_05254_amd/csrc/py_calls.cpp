// The binding's calls in native code: the checks and the marshalling of binding.py's functions, and the call itself.
// A decode step of a layer is a launch of 8 to 40 us; checked and marshalled in Python (attribute by attribute, then
// through ctypes) a call took 10 to 12 us of host time, so that steps over small caches and states were bound by it.
// Here it takes about 1 us and the launch.
//
// Arguments are positional and fixed (binding.py holds the names, defaults and documentation); a cache is passed as the
// address of its descriptor. The library is the one binding.py has loaded, found by path.
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <stdarg.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "yoco.h"

namespace {

PyObject* g_error = nullptr;             // YocoError

#define YOCO_CALLS(X)                                                                                                       \
  X(yoco_last_error_string) X(yoco_swa_prefill) X(yoco_global_kv_write_scaled) X(yoco_cross_attn_prefill) X(yoco_cross_attn_prefill_workspace) X(yoco_cross_attn_decode) \
  X(yoco_cross_attn_decode_noalloc) X(yoco_swa_cache_write) X(yoco_kv_cache_append) X(yoco_swa_decode) X(yoco_gret_prefill) X(yoco_gret_decode)
#define X(name) decltype(&::name) p_##name = nullptr;
YOCO_CALLS(X)
#undef X

struct Failed {};                        // a Python error is set
[[noreturn]] void fail(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  PyErr_FormatV(g_error, fmt, ap);
  va_end(ap);
  throw Failed();
}

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
    throw Failed();
  }
  return THPVariable_Unpack(o);
}
bool none(PyObject* o) { return o == Py_None; }

void* dev(const at::Tensor& t, const char* name) {
  if (!t.is_cuda()) fail("%s must be a device tensor", name);
  if (!t.is_contiguous()) fail("%s must be contiguous", name);
  return t.data_ptr();
}
void* dev_or_null(PyObject* o, const char* name) { return none(o) ? nullptr : dev(tensor(o, name), name); }

int dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return YOCO_F32;
  if (t.scalar_type() == at::kBFloat16) return YOCO_BF16;
  fail("unsupported tensor dtype %s", c10::toString(t.scalar_type()));
}
at::ScalarType torch_dtype(int code) { return code == YOCO_F32 ? at::kFloat : at::kBFloat16; }
at::ScalarType io_dtype(const yoco_kv_cache& c) { return torch_dtype(c.dtype); }     // of queries and outputs; 8-bit caches take bf16

// The output: a fresh tensor shaped like `like`, or the caller's, which must be exactly that (the C ABI sees a pointer only).
at::Tensor output(PyObject* o, const at::Tensor& like) {
  if (none(o)) return at::empty_like(like, like.options().memory_format(at::MemoryFormat::Contiguous));
  const at::Tensor& t = tensor(o, "out");
  if (t.sizes() != like.sizes() || t.scalar_type() != like.scalar_type() || t.device() != like.device())
    fail("out must have the shape, dtype and device of the result (%s on %s)", c10::toString(like.scalar_type()), like.device().str().c_str());
  return t;
}
struct Workspace {
  void* p = nullptr;
  size_t bytes = 0;
};
Workspace workspace(PyObject* o) {
  Workspace w;
  if (none(o)) return w;
  const at::Tensor& t = tensor(o, "workspace");
  w.p = dev(t, "workspace");
  if (t.get_device() != c10::hip::current_device()) fail("workspace must live on the current device");
  w.bytes = t.nbytes();
  return w;
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

int64_t integer(PyObject* o) {
  const int64_t x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) throw Failed();
  return x;
}
float real(PyObject* o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw Failed();
  return (float)x;
}
bool truth(PyObject* o) {
  const int x = PyObject_IsTrue(o);
  if (x < 0) throw Failed();
  return x != 0;
}
yoco_kv_cache cache(PyObject* o) {        // a copy: the call runs without the interpreter lock
  void* p = PyLong_AsVoidPtr(o);
  if (!p) {
    if (!PyErr_Occurred()) PyErr_SetString(g_error, "null cache");
    throw Failed();
  }
  return *(const yoco_kv_cache*)p;
}

// The interpreter lock is given up for the lifetime; taken back also where an exception passes (a device that is not there).
struct Unlocked {
  PyThreadState* s = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(s); }
};
// Runs the call without the interpreter lock (a full launch queue blocks) and raises what it reports.
template <typename F>
void call(F f) {
  int rc;
  {
    Unlocked u;
    rc = f();
  }
  if (rc) fail("libyoco error %d: %s", rc, p_yoco_last_error_string());
}

template <PyObject* (*F)(PyObject* const*)>
struct Entry {
  template <int N>
  static PyObject* run(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != N) return PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
    HANDLE_TH_ERRORS                     // torch's exceptions arrive as the types that torch raises (OutOfMemoryError)
    try {
      return F(a);
    } catch (const Failed&) {
      return nullptr;
    }
    END_HANDLE_TH_ERRORS
  }
};
PyObject* wrap(const at::Tensor& t, PyObject* given) {
  if (given && !none(given)) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(t);
}
PyObject* nothing() { Py_RETURN_NONE; }

void check_lens(const yoco_kv_cache& c, const at::Tensor& t, const char* name) {
  if (t.scalar_type() != at::kLong || t.dim() != 1 || t.size(0) != c.B) fail("%s must be int64 [B]", name);
}
void check_query(const yoco_kv_cache& c, const at::Tensor& q) {
  if (q.dim() != 3 || q.size(0) != c.B || q.size(2) != c.d || q.scalar_type() != io_dtype(c)) fail("q does not match the cache");
}
bool same_rows(const at::Tensor& t, int64_t n, const yoco_kv_cache& c) { return t.dim() == 3 && t.size(0) == n && t.size(1) == c.Hkv && t.size(2) == c.d; }

int64_t rows(const at::Tensor& k) {
  if (!k.dim()) fail("k/v rows do not match the cache");
  return k.size(0);
}

// q, k, v, window, scale, out
PyObject* swa_prefill(PyObject* const* a) {
  const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k"), &v = tensor(a[2], "v");
  if (q.dim() != 4 || k.dim() != 4 || k.size(0) != q.size(0) || k.size(1) != q.size(1) || k.size(3) != q.size(3) || v.sizes() != k.sizes() ||
      k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type())
    fail("q/k/v shapes or dtypes disagree");
  const int64_t window = integer(a[3]);
  const float scale = real(a[4]);
  const at::Tensor o = output(a[5], q);
  void *qp = dev(q, "q"), *kp = dev(k, "k"), *vp = dev(v, "v"), *op = dev(o, "o");
  const int dt = dtype_of(q);
  call([&] { return p_yoco_swa_prefill(qp, kp, vp, op, (int)q.size(0), q.size(1), (int)q.size(2), (int)k.size(2), (int)q.size(3), window, scale, dt, stream()); });
  return wrap(o, a[5]);
}

// cache, k, v, row_scale or None, b, pos0
PyObject* global_kv_write(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &k = tensor(a[1], "k"), &v = tensor(a[2], "v");
  const int64_t n = rows(k);
  if (n && (!same_rows(k, n, c) || v.sizes() != k.sizes() || v.scalar_type() != k.scalar_type())) fail("k/v rows do not match the cache");
  const void* rs = nullptr;
  if (!none(a[3])) {
    const at::Tensor& r = tensor(a[3], "row_scale");
    if (r.scalar_type() != at::kFloat || r.dim() != 1 || r.size(0) != n) fail("row_scale must be float32 [n]");
    if (n) rs = dev(r, "row_scale");
  }
  const int64_t b = integer(a[4]), pos0 = integer(a[5]);
  void *kp = n ? dev(k, "k") : nullptr, *vp = n ? dev(v, "v") : nullptr;
  const int dt = dtype_of(k);
  call([&] { return p_yoco_global_kv_write_scaled(&c, kp, vp, (const float*)rs, (int)b, pos0, n, dt, stream()); });
  return nothing();
}

// ring, k, v, b, pos0
PyObject* swa_cache_write(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &k = tensor(a[1], "k"), &v = tensor(a[2], "v");
  const int64_t n = rows(k);
  if (n && (!same_rows(k, n, c) || v.sizes() != k.sizes() || v.scalar_type() != k.scalar_type())) fail("k/v rows do not match the cache");
  const int64_t b = integer(a[3]), pos0 = integer(a[4]);
  void *kp = n ? dev(k, "k") : nullptr, *vp = n ? dev(v, "v") : nullptr;
  const int dt = dtype_of(k);
  call([&] { return p_yoco_swa_cache_write(&c, kp, vp, (int)b, pos0, n, dt, stream()); });
  return nothing();
}

// cache, k, v, pos, ring
PyObject* kv_cache_append(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &k = tensor(a[1], "k"), &v = tensor(a[2], "v"), &pos = tensor(a[3], "pos");
  if (!same_rows(k, c.B, c) || v.sizes() != k.sizes() || v.scalar_type() != k.scalar_type()) fail("k/v rows do not match the cache");
  check_lens(c, pos, "pos");
  const bool ring = truth(a[4]);
  void *kp = dev(k, "k"), *vp = dev(v, "v"), *pp = dev(pos, "pos");
  const int dt = dtype_of(k);
  call([&] { return p_yoco_kv_cache_append(&c, kp, vp, (const int64_t*)pp, ring, dt, stream()); });
  return nothing();
}

// Scratch from torch's pool of the current stream, to which it goes back when the call has been enqueued; undefined where it
// could cost the program more than the call gains. A request that the device cannot serve makes torch's allocator wait for
// the device and give its cached blocks back, so memory has to be there with room to spare (asking takes 3 us). Under
// capture the pool's blocks would be in use by the graph long after they went back. A capture of another thread or stream
// is not touched: in relaxed mode this thread may ask the driver.
at::Tensor spare_scratch(size_t bytes, const at::TensorOptions& on) {
  if (c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None) return {};
  const c10::DeviceIndex device = c10::hip::current_device();
  const double wanted = 2. * (double)bytes + (64 << 20);                  // the pool rounds up and takes whole segments
  try {
    c10::hip::HIPStreamCaptureModeGuard relaxed(hipStreamCaptureModeRelaxed);
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) != hipSuccess) {
      (void)hipGetLastError();
      return {};
    }
    if ((double)free < wanted) return {};
    const double share = c10::hip::HIPCachingAllocator::getMemoryFraction(device);       // what the program has allowed itself
    if (share < 1. && (double)c10::hip::HIPCachingAllocator::getDeviceStats(device).reserved_bytes[0].current + wanted > share * (double)total)
      return {};
    return at::empty({(int64_t)bytes}, on.dtype(at::kByte));
  } catch (const c10::Error&) {                                           // another allocator, without these questions or this memory
    return {};
  }
}

// cache, q, b, q_pos0, scale, out, workspace
PyObject* cross_attn_prefill(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor& q = tensor(a[1], "q");
  if (q.dim() != 3 || q.size(2) != c.d || q.scalar_type() != io_dtype(c)) fail("q does not match the cache");
  const int64_t b = integer(a[2]), q_pos0 = integer(a[3]);
  const float scale = real(a[4]);
  const at::Tensor o = output(a[5], q);
  Workspace w = workspace(a[6]);
  void *qp = dev(q, "q"), *op = dev(o, "o");
  // Without a workspace a call that takes its output from torch's allocator takes scratch there, too, where that is to be had
  // and the queries live where the launches go. One that is given its output allocates nothing.
  at::Tensor scratch;
  size_t useful = 0;
  if (!w.p && none(a[5]) && q.get_device() == c10::hip::current_device() &&
      p_yoco_cross_attn_prefill_workspace(&c, q_pos0, q.size(0), (int)q.size(1), scale, &useful) == 0 && useful) {
    scratch = spare_scratch(useful, q.options());
    if (scratch.defined()) {
      w.p = scratch.data_ptr();
      w.bytes = useful;
    }
  }
  call([&] { return p_yoco_cross_attn_prefill(&c, qp, op, (int)b, q_pos0, q.size(0), (int)q.size(1), scale, w.p, w.bytes, stream()); });
  return wrap(o, a[5]);
}

// cache, q, lens, scale, workspace, out
PyObject* cross_attn_decode(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &q = tensor(a[1], "q"), &lens = tensor(a[2], "lens");
  check_query(c, q);
  check_lens(c, lens, "lens");
  const float scale = real(a[3]);
  const at::Tensor o = output(a[5], q);
  const Workspace w = workspace(a[4]);
  void *qp = dev(q, "q"), *op = dev(o, "o"), *lp = dev(lens, "lens");
  call([&] { return p_yoco_cross_attn_decode(&c, qp, op, (const int64_t*)lp, (int)q.size(1), scale, w.p, w.bytes, stream()); });
  return wrap(o, a[5]);
}

// cache, q, lens, scale, out
PyObject* cross_attn_decode_noalloc(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &q = tensor(a[1], "q"), &lens = tensor(a[2], "lens");
  check_query(c, q);
  check_lens(c, lens, "lens");
  if (none(a[4])) fail("out is required");
  const float scale = real(a[3]);
  const at::Tensor o = output(a[4], q);
  void *qp = dev(q, "q"), *op = dev(o, "o"), *lp = dev(lens, "lens");
  call([&] { return p_yoco_cross_attn_decode_noalloc(&c, qp, op, (const int64_t*)lp, (int)q.size(1), scale, stream()); });
  return wrap(o, a[4]);
}

// ring, q, lens, scale, workspace, out, k_new, v_new
PyObject* swa_decode(PyObject* const* a) {
  const yoco_kv_cache c = cache(a[0]);
  const at::Tensor &q = tensor(a[1], "q"), &lens = tensor(a[2], "lens");
  check_query(c, q);
  if (c.dtype == YOCO_INT8) fail("q does not match the cache");
  check_lens(c, lens, "lens");
  if (none(a[6]) != none(a[7])) fail("k_new and v_new go together");
  if (!none(a[6])) {
    const at::Tensor &k = tensor(a[6], "k_new"), &v = tensor(a[7], "v_new");
    if (!same_rows(k, c.B, c) || v.sizes() != k.sizes() || k.scalar_type() != io_dtype(c) || v.scalar_type() != io_dtype(c))
      fail("k_new/v_new do not match the cache");
  }
  const float scale = real(a[3]);
  const at::Tensor o = output(a[5], q);
  const Workspace w = workspace(a[4]);
  void *qp = dev(q, "q"), *kp = dev_or_null(a[6], "k_new"), *vp = dev_or_null(a[7], "v_new"), *op = dev(o, "o"), *lp = dev(lens, "lens");
  call([&] { return p_yoco_swa_decode(&c, qp, kp, vp, op, (const int64_t*)lp, (int)q.size(1), scale, w.p, w.bytes, stream()); });
  return wrap(o, a[5]);
}

float* state(PyObject* o, const char* name, int64_t B, int64_t H, int64_t dk, int64_t dv) {
  if (none(o)) return nullptr;
  const at::Tensor& t = tensor(o, name);
  if (t.scalar_type() != at::kFloat || t.dim() != 4 || t.size(0) != B || t.size(1) != H || t.size(2) != dv || t.size(3) != dk)
    fail("%s must be float32 [B,H,dv,dk]", name);
  return (float*)dev(t, name);
}

// q, k, v, log_gamma, scale, chunk, group_norm, eps, state_in, state_out, workspace, out, gate
PyObject* gret_prefill(PyObject* const* a) {
  const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k"), &v = tensor(a[2], "v"), &lg = tensor(a[3], "log_gamma");
  if (q.dim() != 4 || v.dim() != 4 || k.sizes() != q.sizes() || v.sizes().slice(0, 3) != q.sizes().slice(0, 3) || k.scalar_type() != q.scalar_type() ||
      v.scalar_type() != q.scalar_type())
    fail("q/k/v shapes or dtypes disagree");
  const int64_t B = q.size(0), T = q.size(1), H = q.size(2), dk = q.size(3), dv = v.size(3);
  if (lg.scalar_type() != at::kFloat || lg.sizes() != q.sizes().slice(0, 3)) fail("log_gamma must be float32 [B,T,H]");
  if (!none(a[12])) {
    const at::Tensor& g = tensor(a[12], "gate");
    if (g.sizes() != v.sizes() || g.scalar_type() != v.scalar_type()) fail("gate must match v");
  }
  const float scale = real(a[4]), eps = real(a[7]);
  const int64_t chunk = integer(a[5]);
  const bool gn = truth(a[6]);
  const at::Tensor o = output(a[11], v);
  const Workspace w = workspace(a[10]);
  void *qp = nullptr, *kp = nullptr, *vp = nullptr, *gp = nullptr, *op = nullptr, *lp = nullptr;
  if (T) {
    qp = dev(q, "q");
    kp = dev(k, "k");
    vp = dev(v, "v");
    lp = dev(lg, "log_gamma");
    gp = dev_or_null(a[12], "gate");
    op = dev(o, "o");
  }
  float *si = state(a[8], "state_in", B, H, dk, dv), *so = state(a[9], "state_out", B, H, dk, dv);
  const int dt = dtype_of(q);
  call([&] {
    return p_yoco_gret_prefill(qp, kp, vp, (const float*)lp, gp, op, si, so, (int)B, T, (int)H, (int)dk, (int)dv, (int)chunk, scale, gn, eps, dt, w.p, w.bytes, stream());
  });
  return wrap(o, a[11]);
}

// q, k, v, log_gamma, state, scale, group_norm, eps, out, gate
PyObject* gret_decode(PyObject* const* a) {
  const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k"), &v = tensor(a[2], "v"), &lg = tensor(a[3], "log_gamma");
  if (q.dim() != 3 || v.dim() != 3 || k.sizes() != q.sizes() || v.size(0) != q.size(0) || v.size(1) != q.size(1) || k.scalar_type() != q.scalar_type() ||
      v.scalar_type() != q.scalar_type())
    fail("q/k/v shapes or dtypes disagree");
  const int64_t B = q.size(0), H = q.size(1), dk = q.size(2), dv = v.size(2);
  if (lg.scalar_type() != at::kFloat || lg.dim() != 2 || lg.size(0) != B || lg.size(1) != H) fail("log_gamma must be float32 [B,H]");
  if (!none(a[9])) {
    const at::Tensor& g = tensor(a[9], "gate");
    if (g.sizes() != v.sizes() || g.scalar_type() != v.scalar_type()) fail("gate must match v");
  }
  const float scale = real(a[5]), eps = real(a[7]);
  const bool gn = truth(a[6]);
  const at::Tensor o = output(a[8], v);
  void *qp = dev(q, "q"), *kp = dev(k, "k"), *vp = dev(v, "v"), *lp = dev(lg, "log_gamma"), *gp = dev_or_null(a[9], "gate"), *op = dev(o, "o");
  float* st = state(a[4], "state", B, H, dk, dv);
  const int dt = dtype_of(q);
  call([&] { return p_yoco_gret_decode(qp, kp, vp, (const float*)lp, gp, op, st, (int)B, (int)H, (int)dk, (int)dv, scale, gn, eps, dt, stream()); });
  return wrap(o, a[8]);
}

// path of libyoco, the exception type
PyObject* init(PyObject*, PyObject* args) {
  const char* path = nullptr;
  PyObject* error = nullptr;
  if (!PyArg_ParseTuple(args, "sO", &path, &error)) return nullptr;
  void* h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
  if (!h) return PyErr_Format(PyExc_OSError, "%s", dlerror());
#define X(name)                                                       \
  p_##name = (decltype(p_##name))dlsym(h, #name);                     \
  if (!p_##name) return PyErr_Format(PyExc_OSError, "%s has no %s", path, #name);
  YOCO_CALLS(X)
#undef X
  Py_INCREF(error);
  Py_XSETREF(g_error, error);
  Py_RETURN_NONE;
}

#define ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))Entry<name>::run<n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         ENTRY(swa_prefill, 6),
                         ENTRY(global_kv_write, 6),
                         ENTRY(swa_cache_write, 5),
                         ENTRY(kv_cache_append, 5),
                         ENTRY(cross_attn_prefill, 7),
                         ENTRY(cross_attn_decode, 6),
                         ENTRY(cross_attn_decode_noalloc, 5),
                         ENTRY(swa_decode, 8),
                         ENTRY(gret_prefill, 13),
                         ENTRY(gret_decode, 10),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }
