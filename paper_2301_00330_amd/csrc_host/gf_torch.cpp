// Host side of torch_api: descriptor and tensor checks, output allocation, workspace lookup and the call
// into libgf, in one native call per entry point.
//
// What bounds it: a filtered backward of one layer is two or three kernel launches, 6 - 10 us of host time; the
// same steps written in Python (six ctypes calls, three torch.empty, the stream and shape look-ups) took
// 30 - 38 us per layer and were the whole time of every case whose kernels take less than that.  Nothing is
// kept between calls but the default workspaces: a descriptor's shapes are recomputed each time
// (integer arithmetic, well below a microsecond).
//
// Arguments are positional here (METH_FASTCALL); torch_api.py owns names, defaults and documentation.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <vector>

#include "gf.h"

namespace {

typedef std::array<int64_t, 4> Shape;

PyObject* g_check = nullptr;       // torch_api._check: raises the ValueError that names what is wrong
PyObject* g_gferror = nullptr;     // binding.GfError
PyObject* g_workspace = nullptr;   // torch_api.Workspace
PyObject* g_int8 = nullptr;        // torch.int8
PyObject* g_oom = nullptr;         // torch.OutOfMemoryError
constexpr int kFields = 13;
const char* const kFieldNames[kFields] = {"N", "C_in", "C_out", "H_in", "W_in", "K_h", "K_w", "stride", "pad",
                                          "dilation", "groups", "r", "dtype"};
PyObject* g_fields[kFields];
PyObject *g_buf, *g_get;           // interned "buf", "get"

struct DefaultWs { int device; hipStream_t stream; PyObject* ws; };
std::vector<DefaultWs> g_default_ws;   // one per (device, stream): torch hands out a fixed pool of streams

// A Python exception is set; unwinds to the entry point.
struct Raised {};

void status(gf_status rc, const char* where) {
  if (rc == GF_OK) return;
  if (PyObject* e = PyObject_CallFunction(g_gferror, "is", (int)rc, where)) {
    PyErr_SetObject(g_gferror, e);
    Py_DECREF(e);
  }
  throw Raised();
}

struct Layer {
  PyObject* py;
  gf_conv_desc d;
  Shape x, gy, w, xu, gyu;
  at::ScalarType dt;

  explicit Layer(PyObject* o, bool exact = false) : py(o) {
    int32_t v[kFields];
    for (int i = 0; i < kFields; ++i) {
      PyObject* f = PyObject_GetAttr(o, g_fields[i]);
      if (!f) throw Raised();
      const long n = PyLong_AsLong(f);
      Py_DECREF(f);
      if (n == -1 && PyErr_Occurred()) throw Raised();
      v[i] = (int32_t)n;
    }
    d = gf_conv_desc{(uint32_t)sizeof(gf_conv_desc), v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9],
                     v[10], exact ? 1 : v[11], v[12]};   // vanilla BP has the shapes of r = 1
    int32_t Hy, Wy, Hp, Wp;
    status(gf_out_shape(&d, &Hy, &Wy, &Hp, &Wp), "gf_out_shape");
    d.r = v[11];
    x = {d.N, d.C_in, d.H_in, d.W_in};
    gy = {d.N, d.C_out, Hy, Wy};
    w = {d.C_out, d.C_in / d.groups, d.K_h, d.K_w};
    xu = exact || d.r == 1 ? x : Shape{d.N, d.C_in, Hp, Wp};
    gyu = {d.N, d.C_out, Hp, Wp};
    dt = d.dtype == GF_BF16 ? at::kBFloat16 : at::kFloat;
  }
};

// The tensor behind `o`, after torch_api._check's conditions; where one does not hold, _check says which.
const at::Tensor& tensor(PyObject* o, const Layer& l, const Shape& s, const char* what, bool codes = false) {
  if (THPVariable_Check(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.is_cuda() && t.scalar_type() == (codes ? at::kChar : l.dt) && t.dim() == 4 &&
        t.sizes() == at::IntArrayRef(s.data(), 4) && t.is_contiguous())
      return t;
  }
  PyObject* r = PyObject_CallFunction(g_check, "OO(LLLL)sO", o, l.py, (long long)s[0], (long long)s[1],
                                      (long long)s[2], (long long)s[3], what, codes ? g_int8 : Py_None);
  if (r) {
    Py_DECREF(r);
    PyErr_Format(PyExc_ValueError, "%s must be a contiguous device tensor", what);
  }
  throw Raised();
}

const at::Tensor& any_tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "out must be a tensor");
    throw Raised();
  }
  return THPVariable_Unpack(o);
}

at::Tensor make(const at::Tensor& like, at::IntArrayRef s, at::ScalarType dt) {
  return at::empty(s, at::TensorOptions().device(like.device()).dtype(dt));
}
at::Tensor make(const at::Tensor& like, const Shape& s, at::ScalarType dt) {
  return make(like, at::IntArrayRef(s.data(), 4), dt);
}

// Scratch of a call: the caller's workspace, else a default one per (device, current stream) -- calls on
// different streams may overlap in time and must not share scratch memory.  A workspace is any object whose
// get(bytes) returns (address, size); of torch_api.Workspace itself the buffer is read directly and `hold` keeps it
// alive while the interpreter lock is released around the launch.
struct Scratch {
  void* p = nullptr;
  size_t n = 0;
  at::Tensor hold;

  Scratch(const Layer& l, int op, PyObject* ws, const at::Tensor& on) {
    size_t need = 0;
    status(gf_workspace_bytes(&l.d, op, &need), "gf_workspace_bytes");
    if (ws == Py_None) ws = default_for(on);
    if ((PyObject*)Py_TYPE(ws) != g_workspace) {
      PyObject* r = PyObject_CallMethod(ws, "get", "n", (Py_ssize_t)need);
      PyObject* pair = r ? PySequence_Tuple(r) : nullptr;
      Py_XDECREF(r);
      unsigned long long addr = 0, size = 0;
      const bool ok = pair && PyArg_ParseTuple(pair, "KK", &addr, &size);
      Py_XDECREF(pair);
      if (!ok) throw Raised();
      p = reinterpret_cast<void*>((uintptr_t)addr);
      n = (size_t)size;
      return;
    }
    if (need == 0) return;
    PyObject* b = PyObject_GetAttr(ws, g_buf);
    if (!b) throw Raised();
    if (!THPVariable_Check(b) || (size_t)THPVariable_Unpack(b).numel() < need) {   // Workspace.get grows it
      Py_DECREF(b);
      PyObject* n_ = PyLong_FromSize_t(need);
      PyObject* r = n_ ? PyObject_CallMethodObjArgs(ws, g_get, n_, nullptr) : nullptr;
      Py_XDECREF(n_);
      if (!r) throw Raised();
      Py_DECREF(r);
      b = PyObject_GetAttr(ws, g_buf);
      if (!b) throw Raised();
    }
    hold = THPVariable_Unpack(b);
    Py_DECREF(b);
    p = hold.data_ptr();
    n = (size_t)hold.numel();
  }

  static PyObject* default_for(const at::Tensor& on) {
    const int dev = on.device().index();
    const hipStream_t st = c10::hip::getCurrentHIPStream((c10::DeviceIndex)dev).stream();
    for (const DefaultWs& e : g_default_ws)
      if (e.device == dev && e.stream == st) return e.ws;
    PyObject* pd = THPVariable_Wrap(on);
    PyObject* device = pd ? PyObject_GetAttrString(pd, "device") : nullptr;
    Py_XDECREF(pd);
    PyObject* ws = device ? PyObject_CallFunctionObjArgs(g_workspace, device, nullptr) : nullptr;
    Py_XDECREF(device);
    if (!ws) throw Raised();
    g_default_ws.push_back({dev, st, ws});
    return ws;
  }
};

void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

// The call itself, with the interpreter lock released (as a ctypes call would).
template <class F> void call(const char* where, F&& f) {
  void* const st = c10::hip::getCurrentHIPStream().stream();   // may throw: with the lock still held
  gf_status rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(st);
  Py_END_ALLOW_THREADS
  status(rc, where);
}

PyObject* wrap(const at::Tensor& t) {
  if (!t.defined()) Py_RETURN_NONE;
  PyObject* o = THPVariable_Wrap(t);
  if (!o) throw Raised();
  return o;
}
PyObject* tuple(std::initializer_list<at::Tensor> ts) {
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) throw Raised();
  Py_ssize_t i = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = nullptr;
    try { o = wrap(t); } catch (const Raised&) { Py_DECREF(r); throw; }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

float number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised();
  return (float)v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised();
  return v != 0;
}

// ---- entry points: positional arguments as torch_api passes them ----

PyObject* pool_activation(PyObject* const* a) {   // d, x, out
  const Layer l(a[0]);
  const at::Tensor& x = tensor(a[1], l, l.x, "x");
  at::Tensor out = a[2] == Py_None ? make(x, l.xu, x.scalar_type()) : any_tensor(a[2]);
  call("gf_pool_activation", [&](void* st) { return gf_pool_activation(&l.d, ptr(x), ptr(out), st); });
  return wrap(out);
}

// descs, xs, inv_deltas (sequences); without codes: storage-type sums, no third argument
template <bool CODES>
PyObject* pool_batch(PyObject* const* a) {
  struct Seq {
    PyObject* s;
    explicit Seq(PyObject* o) : s(PySequence_Fast(o, "a sequence is expected")) { if (!s) throw Raised(); }
    ~Seq() { Py_DECREF(s); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(s); }
    PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(s, i); }
  };
  const Seq ds(a[0]), xs(a[1]);
  const Seq v(a[CODES ? 2 : 1]);
  const Py_ssize_t m = std::min(ds.size(), xs.size());
  std::vector<gf_conv_desc> d;
  std::vector<const void*> in;
  std::vector<void*> out;
  std::vector<at::Tensor> made;
  std::vector<float> inv;
  for (Py_ssize_t i = 0; i < m; ++i) {
    const Layer l(ds[i]);
    const at::Tensor& x = tensor(xs[i], l, l.x, "x");
    made.push_back(make(x, l.xu, CODES ? at::kChar : x.scalar_type()));
    d.push_back(l.d);
    in.push_back(ptr(x));
    out.push_back(ptr(made.back()));
  }
  bool same = ds.size() == m && xs.size() == m;
  if constexpr (CODES) {
    same = same && v.size() == m;
    for (Py_ssize_t i = 0; same && i < m; ++i) inv.push_back(number(v[i]));
  }
  if (!same) {
    PyErr_SetString(PyExc_AssertionError, "one descriptor, one tensor (and one step size) per layer");
    throw Raised();
  }
  gf_conv_desc none{};
  const void* no_in = nullptr;
  void* no_out = nullptr;
  const gf_conv_desc* dp = m ? d.data() : &none;   // an empty call is the library's to refuse
  const void* const* ip = m ? in.data() : &no_in;
  void* const* op = m ? out.data() : &no_out;
  if constexpr (CODES)
    call("gf_pool_activation_batch_q8", [&](void* st) {
      return gf_pool_activation_batch_q8((int32_t)m, dp, ip, inv.data(), reinterpret_cast<int8_t* const*>(op), st);
    });
  else
    call("gf_pool_activation_batch", [&](void* st) { return gf_pool_activation_batch((int32_t)m, dp, ip, op, st); });
  PyObject* r = PyList_New(m);
  if (!r) throw Raised();
  for (Py_ssize_t i = 0; i < m; ++i) {
    PyObject* o = nullptr;
    try { o = wrap(made[i]); } catch (const Raised&) { Py_DECREF(r); throw; }
    PyList_SET_ITEM(r, i, o);
  }
  return r;
}

PyObject* pool_activation_batch(PyObject* const* a) { return pool_batch<false>(a); }
PyObject* pool_activation_batch_q8(PyObject* const* a) { return pool_batch<true>(a); }

PyObject* pool_activation_mask(PyObject* const* a) {   // d, x, hi
  const Layer l(a[0]);
  const at::Tensor& x = tensor(a[1], l, l.x, "x");
  const float hi = number(a[2]);
  at::Tensor xu = make(x, l.xu, x.scalar_type()), mu = make(x, l.xu, x.scalar_type());
  call("gf_pool_activation_mask", [&](void* st) { return gf_pool_activation_mask(&l.d, ptr(x), hi, ptr(xu), ptr(mu), st); });
  return tuple({xu, mu});
}

PyObject* filter_grad(PyObject* const* a) {   // d, g_y, out
  const Layer l(a[0]);
  const at::Tensor& gy = tensor(a[1], l, l.gy, "g_y");
  at::Tensor out = a[2] == Py_None ? make(gy, l.gyu, gy.scalar_type()) : any_tensor(a[2]);
  call("gf_filter_grad", [&](void* st) { return gf_filter_grad(&l.d, ptr(gy), ptr(out), st); });
  return wrap(out);
}

constexpr int64_t kTwo[1] = {2};

PyObject* filter_grad_snr(PyObject* const* a) {   // d, g_y, ws
  const Layer l(a[0]);
  const at::Tensor& gy = tensor(a[1], l, l.gy, "g_y");
  at::Tensor gyu = make(gy, l.gyu, gy.scalar_type()), stats = make(gy, at::IntArrayRef(kTwo), at::kDouble);
  const Scratch s(l, GF_OP_FILTER_SNR, a[2], gy);
  call("gf_filter_grad_snr", [&](void* st) {
    return gf_filter_grad_snr(&l.d, ptr(gy), ptr(gyu), static_cast<double*>(ptr(stats)), s.p, s.n, st);
  });
  return tuple({gyu, stats});
}

PyObject* conv_bwd_weight(PyObject* const* a) {   // d, x_u, gy_u, out, ws
  const Layer l(a[0]);
  const at::Tensor &xu = tensor(a[1], l, l.xu, "x_u"), &gyu = tensor(a[2], l, l.gyu, "gy_u");
  at::Tensor out = a[3] == Py_None ? make(xu, l.w, at::kFloat) : any_tensor(a[3]);
  const Scratch s(l, GF_OP_BWD_WEIGHT, a[4], xu);
  call("gf_conv_bwd_weight", [&](void* st) {
    return gf_conv_bwd_weight(&l.d, ptr(xu), ptr(gyu), static_cast<float*>(ptr(out)), s.p, s.n, st);
  });
  return wrap(out);
}

PyObject* conv_bwd_input(PyObject* const* a) {   // d, gy_u, w, reduced_out, out, ws
  const Layer l(a[0]);
  const at::Tensor &gyu = tensor(a[1], l, l.gyu, "gy_u"), &w = tensor(a[2], l, l.w, "w");
  const bool reduced = truth(a[3]);
  at::Tensor out = a[4] == Py_None ? make(gyu, reduced ? l.xu : l.x, gyu.scalar_type()) : any_tensor(a[4]);
  const Scratch s(l, GF_OP_BWD_INPUT, a[5], gyu);
  call("gf_conv_bwd_input", [&](void* st) {
    return gf_conv_bwd_input(&l.d, ptr(gyu), ptr(w), ptr(out), reduced, s.p, s.n, st);
  });
  return wrap(out);
}

PyObject* conv_bwd_filtered(PyObject* const* a) {   // d, g_y, x_u, w, want_gyu, ws
  const Layer l(a[0]);
  const at::Tensor &gy = tensor(a[1], l, l.gy, "g_y"), &xu = tensor(a[2], l, l.xu, "x_u"), &w = tensor(a[3], l, l.w, "w");
  at::Tensor gw = make(gy, l.w, at::kFloat), gx = make(gy, l.x, gy.scalar_type()), gyu;
  if (truth(a[4])) gyu = make(gy, l.gyu, gy.scalar_type());
  const Scratch s(l, GF_OP_BWD_FILTERED, a[5], gy);
  call("gf_conv_bwd_filtered", [&](void* st) {
    return gf_conv_bwd_filtered(&l.d, ptr(gy), ptr(xu), ptr(w), ptr(gyu), static_cast<float*>(ptr(gw)), ptr(gx), s.p,
                                s.n, st);
  });
  return tuple({gw, gx, gyu});
}

PyObject* conv_bwd_chained(PyObject* const* a) {   // d, gy_u, x_u, w, reduced_out, mask_u, ws
  const Layer l(a[0]);
  const at::Tensor &gyu = tensor(a[1], l, l.gyu, "gy_u"), &xu = tensor(a[2], l, l.xu, "x_u"), &w = tensor(a[3], l, l.w, "w");
  const bool reduced = truth(a[4]);
  const Shape& so = reduced ? l.xu : l.x;
  at::Tensor mask, gw = make(gyu, l.w, at::kFloat), gx = make(gyu, so, gyu.scalar_type());
  if (a[5] != Py_None) mask = tensor(a[5], l, so, "mask_u");
  const Scratch s(l, GF_OP_BWD_CHAINED, a[6], gyu);
  call("gf_conv_bwd_chained", [&](void* st) {
    return gf_conv_bwd_chained(&l.d, ptr(gyu), ptr(xu), ptr(w), static_cast<float*>(ptr(gw)), ptr(gx), reduced, ptr(mask),
                               s.p, s.n, st);
  });
  return tuple({gw, gx});
}

PyObject* conv_bwd_exact(PyObject* const* a) {   // d, x, w, g_y, want_gw, want_gx, ws
  const Layer l(a[0], true);
  const at::Tensor& gy = tensor(a[3], l, l.gy, "g_y");
  const bool want_gw = truth(a[4]), want_gx = truth(a[5]);
  at::Tensor x, w, gw, gx;
  if (want_gw) {
    x = tensor(a[1], l, l.x, "x");
    gw = make(gy, l.w, at::kFloat);
  }
  if (want_gx) {
    w = tensor(a[2], l, l.w, "w");
    gx = make(gy, l.x, gy.scalar_type());
  }
  const Scratch s(l, GF_OP_BWD_EXACT, a[6], gy);
  call("gf_conv_bwd_exact", [&](void* st) {
    return gf_conv_bwd_exact(&l.d, ptr(x), ptr(w), ptr(gy), static_cast<float*>(ptr(gw)), ptr(gx), s.p, s.n, st);
  });
  return tuple({gw, gx});
}

PyObject* conv_bwd_unique(PyObject* const* a) {   // d, gy_u, x_u, w, reduced_out, ws
  const Layer l(a[0]);
  const at::Tensor &gyu = tensor(a[1], l, l.gyu, "gy_u"), &xu = tensor(a[2], l, l.xu, "x_u"), &w = tensor(a[3], l, l.w, "w");
  const bool reduced = truth(a[4]);
  at::Tensor gw = make(gyu, l.w, at::kFloat), gx = make(gyu, reduced ? l.xu : l.x, l.dt);
  const Scratch s(l, GF_OP_BWD_UNIQUE, a[5], gyu);
  call("gf_conv_bwd_unique", [&](void* st) {
    return gf_conv_bwd_unique(&l.d, ptr(gyu), ptr(xu), ptr(w), static_cast<float*>(ptr(gw)), ptr(gx), reduced, s.p, s.n,
                              st);
  });
  return tuple({gw, gx});
}

int8_t* ptr8(const at::Tensor& t) { return static_cast<int8_t*>(ptr(t)); }

PyObject* filter_grad_q8(PyObject* const* a) {   // d, g_y, inv_delta
  const Layer l(a[0]);
  const at::Tensor& gy = tensor(a[1], l, l.gy, "g_y");
  const float inv = number(a[2]);
  at::Tensor out = make(gy, l.gyu, at::kChar);
  call("gf_filter_grad_q8", [&](void* st) { return gf_filter_grad_q8(&l.d, ptr(gy), inv, ptr8(out), st); });
  return wrap(out);
}

PyObject* pool_activation_q8(PyObject* const* a) {   // d, x, inv_delta
  const Layer l(a[0]);
  const at::Tensor& x = tensor(a[1], l, l.x, "x");
  const float inv = number(a[2]);
  at::Tensor out = make(x, l.xu, at::kChar);
  call("gf_pool_activation_q8", [&](void* st) { return gf_pool_activation_q8(&l.d, ptr(x), inv, ptr8(out), st); });
  return wrap(out);
}

PyObject* kernel_sum_q8(PyObject* const* a) {   // d, w, inv_delta
  const Layer l(a[0]);
  const at::Tensor& w = tensor(a[1], l, l.w, "w");
  const float inv = number(a[2]);
  at::Tensor out = make(w, at::IntArrayRef(l.w.data(), 2), at::kChar);
  call("gf_kernel_sum_q8", [&](void* st) { return gf_kernel_sum_q8(&l.d, ptr(w), inv, ptr8(out), st); });
  return wrap(out);
}

PyObject* conv_bwd_weight_q8(PyObject* const* a) {   // d, x_q, gy_q, scale, ws
  const Layer l(a[0]);
  const at::Tensor &xq = tensor(a[1], l, l.xu, "x_q", true), &gyq = tensor(a[2], l, l.gyu, "gy_q", true);
  const float scale = number(a[3]);
  at::Tensor gw = make(xq, l.w, at::kFloat);
  const Scratch s(l, GF_OP_BWD_WEIGHT_Q8, a[4], xq);
  call("gf_conv_bwd_weight_q8", [&](void* st) {
    return gf_conv_bwd_weight_q8(&l.d, ptr8(xq), ptr8(gyq), scale, static_cast<float*>(ptr(gw)), s.p, s.n, st);
  });
  return wrap(gw);
}

// gy_q and w_q are [N, C_out, H_p, W_p] and [C_out, C_in / groups]
PyObject* conv_bwd_input_q8(PyObject* const* a) {   // d, gy_q, w_q, scale, reduced_out, ws
  const Layer l(a[0]);
  const at::Tensor& gyq = tensor(a[1], l, l.gyu, "gy_q", true);
  if (!THPVariable_Check(a[2])) { PyErr_SetString(PyExc_TypeError, "w_q must be a tensor"); throw Raised(); }
  const at::Tensor& wq = THPVariable_Unpack(a[2]);
  if (!wq.is_cuda() || wq.scalar_type() != at::kChar || wq.sizes() != at::IntArrayRef(l.w.data(), 2) || !wq.is_contiguous()) {
    PyObject* r = PyObject_CallFunction(g_check, "OO(LL)sO", a[2], l.py, (long long)l.w[0], (long long)l.w[1], "w_q", g_int8);
    if (r) { Py_DECREF(r); PyErr_SetString(PyExc_ValueError, "w_q must be a contiguous device tensor"); }
    throw Raised();
  }
  const float scale = number(a[3]);
  const bool reduced = truth(a[4]);
  at::Tensor gx = make(gyq, reduced ? l.xu : l.x, l.dt);
  const Scratch s(l, GF_OP_BWD_INPUT_Q8, a[5], gyq);
  call("gf_conv_bwd_input_q8", [&](void* st) {
    return gf_conv_bwd_input_q8(&l.d, ptr8(gyq), ptr8(wq), scale, ptr(gx), reduced, s.p, s.n, st);
  });
  return wrap(gx);
}

PyObject* conv_bwd_filtered_q8(PyObject* const* a) {   // d, g_y, inv_gy, x_q, w, inv_w, scale_w, scale_x, want_gyq, ws
  const Layer l(a[0]);
  const at::Tensor &gy = tensor(a[1], l, l.gy, "g_y"), &xq = tensor(a[3], l, l.xu, "x_q", true), &w = tensor(a[4], l, l.w, "w");
  const float inv_gy = number(a[2]), inv_w = number(a[5]), scale_w = number(a[6]), scale_x = number(a[7]);
  const bool want = truth(a[8]);
  at::Tensor gw = make(gy, l.w, at::kFloat), gx = make(gy, l.x, l.dt), gyq;
  if (want) gyq = make(gy, l.gyu, at::kChar);
  const Scratch s(l, GF_OP_BWD_FILTERED_Q8, a[9], gy);
  call("gf_conv_bwd_filtered_q8", [&](void* st) {
    return gf_conv_bwd_filtered_q8(&l.d, ptr(gy), inv_gy, ptr8(xq), ptr(w), inv_w, scale_w, scale_x, ptr8(gyq),
                                   static_cast<float*>(ptr(gw)), ptr(gx), s.p, s.n, st);
  });
  return want ? tuple({gw, gx, gyq}) : tuple({gw, gx});
}

// METH_FASTCALL shell: argument count, and C++ exceptions (torch's among them) as Python ones
template <PyObject* (*F)(PyObject* const*), int NARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != NARGS) {
    PyErr_Format(PyExc_TypeError, "%d arguments expected, got %zd", NARGS, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Raised&) {
    return nullptr;
  } catch (const c10::OutOfMemoryError& e) {
    PyErr_SetString(g_oom, e.what_without_backtrace());
    return nullptr;
  } catch (const c10::Error& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// setup(check, gf_error, workspace_class, int8, out_of_memory_error): what this module calls back
PyObject* setup(PyObject* const* a) {
  PyObject** const to[5] = {&g_check, &g_gferror, &g_workspace, &g_int8, &g_oom};
  for (int i = 0; i < 5; ++i) {
    Py_INCREF(a[i]);
    Py_XDECREF(*to[i]);
    *to[i] = a[i];
  }
  Py_RETURN_NONE;
}

#define GF_ENTRY(name, nargs) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, nargs>)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    GF_ENTRY(setup, 5), GF_ENTRY(pool_activation, 3), GF_ENTRY(pool_activation_batch, 2),
    GF_ENTRY(pool_activation_batch_q8, 3),
    GF_ENTRY(pool_activation_mask, 3), GF_ENTRY(filter_grad, 3), GF_ENTRY(filter_grad_snr, 3),
    GF_ENTRY(conv_bwd_weight, 5), GF_ENTRY(conv_bwd_input, 6), GF_ENTRY(conv_bwd_filtered, 6),
    GF_ENTRY(conv_bwd_chained, 7), GF_ENTRY(conv_bwd_exact, 7), GF_ENTRY(conv_bwd_unique, 6),
    GF_ENTRY(filter_grad_q8, 3), GF_ENTRY(pool_activation_q8, 3), GF_ENTRY(kernel_sum_q8, 3),
    GF_ENTRY(conv_bwd_weight_q8, 5), GF_ENTRY(conv_bwd_input_q8, 6), GF_ENTRY(conv_bwd_filtered_q8, 10),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gf_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__gf_torch() {
  for (int i = 0; i < kFields; ++i)
    if (!(g_fields[i] = PyUnicode_InternFromString(kFieldNames[i]))) return nullptr;
  g_buf = PyUnicode_InternFromString("buf");
  g_get = PyUnicode_InternFromString("get");
  if (!g_buf || !g_get) return nullptr;
  return PyModule_Create(&module);
}
