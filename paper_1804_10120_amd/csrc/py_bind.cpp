// CPython extension of the torch binding: the calls a program makes most, from
// the tensors to the C ABI without passing through Python.
//
// What bounds a small call is the host.  Marshalling seven tensors, allocating
// the output and entering the library through ctypes took 19 us where the
// kernel takes 4; from here it takes 4.4.  The adjoint with its six outputs:
// 31 and 8 us; a batch of 48 subgrids given as dicts: 460 and 29.  The autograd
// node is native too, because the engine runs it on a thread of its own: as a
// Python function it waited for the interpreter there, and a forward and
// backward pass over 20^3 points took 190 us, now 80 (41 of them the engine's
// own, for a node that does nothing).
//
// Every function here serves the plain case and answers None to all others --
// another type, shape, device or layout, a tensor subclass, an active mode or
// transform, zero points -- which the Python code of ops.py and autograd.py
// then handles as if this module were not there, its error messages included.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/functions/basic_ops.h>
#include <torch/csrc/autograd/grad_mode.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <utility>
#include <vector>

#include "../../include/tl.h"

namespace {

// The entry points, by the addresses init() was given (the library that
// _abi.lib() loaded).
enum Entry { kInverse, kChristoffel, kCovDeriv, kDtg, kChain, kBwd, kFwdBwd, kEntries };
void* g_entry[kEntries] = {};
decltype(&tl_expr) g_expr = nullptr;
decltype(&tl_batch_run_noalloc) g_noalloc = nullptr;
decltype(&tl_batch_plan_launch) g_plan_launch = nullptr;
PyObject* g_check = nullptr;  // _abi.check: raises TLError for a status

struct Spec {
  int nin, nout;
  int in[7], out[7];
  int alpha;  // input whose shape ([n] or [1, n]) a one-component output takes
};
const Spec kSpec[kEntries] = {
    {1, 1, {6}, {6}, 0},
    {2, 1, {6, 18}, {18}, 0},
    {3, 1, {18, 3, 9}, {9}, 0},
    {3, 1, {1, 6, 9}, {6}, 0},
    {6, 1, {6, 18, 3, 9, 6, 1}, {6}, 5},
    {6, 6, {6, 18, 3, 6, 1, 6}, {6, 18, 3, 9, 6, 1}, 4},
    {7, 7, {6, 18, 3, 9, 6, 1, 6}, {6, 6, 18, 3, 9, 6, 1}, 5},
};

template <class F>
F entry(Entry e) {
  return reinterpret_cast<F>(g_entry[e]);
}

tl_status call(Entry e, int64_t n, const tl_cfield* i, const tl_field* o, void* s) {
  switch (e) {
    case kInverse: return entry<decltype(&tl_sym_inverse)>(e)(n, i[0], o[0], s, nullptr);
    case kChristoffel:
      return entry<decltype(&tl_christoffel)>(e)(n, i[0], i[1], o[0], s, nullptr);
    case kCovDeriv:
      return entry<decltype(&tl_cov_deriv)>(e)(n, i[0], i[1], i[2], o[0], s, nullptr);
    case kDtg: return entry<decltype(&tl_dtg)>(e)(n, i[0], i[1], i[2], o[0], s, nullptr);
    case kChain:
      return entry<decltype(&tl_dtg_chain)>(e)(n, i[0], i[1], i[2], i[3], i[4], i[5], o[0], s,
                                               nullptr);
    case kBwd:
      return entry<decltype(&tl_dtg_chain_bwd)>(e)(n, i[0], i[1], i[2], i[3], i[4], i[5], o[0],
                                                   o[1], o[2], o[3], o[4], o[5], s, nullptr);
    default:
      return entry<decltype(&tl_dtg_chain_fwd_bwd)>(kFwdBwd)(
          n, i[0], i[1], i[2], i[3], i[4], i[5], i[6], o[0], o[1], o[2], o[3], o[4], o[5], o[6], s,
          nullptr);
  }
}

// Whether a mode, transform or tracer sees torch's own calls in this thread.
bool watched() {
  const c10::DispatchKeySet in = c10::impl::tls_local_dispatch_key_set().included_;
  return at::impl::torch_function_mode_enabled() || in.has(c10::DispatchKey::Python) ||
         in.has(c10::DispatchKey::Tracer) || in.has(c10::DispatchKey::Functionalize) ||
         in.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
         in.has(c10::DispatchKey::FuncTorchVmapMode);
}

// The fields of one call: common n and device.
struct Fields {
  int64_t n = -1;
  c10::Device device = c10::Device(c10::DeviceType::CPU);

  // A plain float64 device tensor [ncomp, n] (or [n] for one component) with
  // unit stride along the points, of the same n and device as the others.
  bool take(const at::Tensor& t, int ncomp, tl_cfield* f) {
    if (!t.defined() || t.scalar_type() != at::kDouble || t.layout() != at::kStrided ||
        t.device().type() != c10::DeviceType::CUDA)
      return false;
    const c10::DispatchKeySet ks = t.key_set();
    if (ks.has(c10::DispatchKey::Python) || ks.has(c10::DispatchKey::FuncTorchBatched) ||
        ks.has(c10::DispatchKey::FuncTorchGradWrapper) || ks.has(c10::DispatchKey::Negative) ||
        ks.has(c10::DispatchKey::Conjugate) || ks.has(c10::DispatchKey::ZeroTensor) ||
        ks.has(c10::DispatchKey::Functionalize))
      return false;
    const int64_t dim = t.dim();
    const bool flat = dim == 1 && ncomp == 1;
    if (!flat && (dim != 2 || t.size(0) != ncomp)) return false;
    const int64_t m = t.size(dim - 1);
    if (m < 1 || (m > 1 && t.stride(dim - 1) != 1)) return false;
    if (n < 0) {
      n = m;
      device = t.device();
    } else if (m != n || t.device() != device) {
      return false;
    }
    f->ptr = static_cast<const double*>(t.data_ptr());
    f->ld = ncomp == 1 ? m : t.stride(0);
    return true;
  }
  bool take(PyObject* o, int ncomp, tl_cfield* f) {
    return THPVariable_CheckExact(o) && take(THPVariable_Unpack(o), ncomp, f);
  }
  bool take(PyObject* o, int ncomp, tl_field* f) {
    tl_cfield c;
    if (!take(o, ncomp, &c)) return false;
    *f = {const_cast<double*>(c.ptr), c.ld};
    return true;
  }
  // The library launches on the current device.
  bool current() const { return device.index() == c10::hip::current_device(); }
  void* stream() const { return c10::hip::getCurrentHIPStream(device.index()).stream(); }

  at::Tensor make(int ncomp, bool flat, tl_field* f) const {
    const auto opt = at::TensorOptions().dtype(at::kDouble).device(device);
    at::Tensor t = flat ? at::empty({n}, opt) : at::empty({ncomp, n}, opt);
    *f = {static_cast<double*>(t.data_ptr()), n};
    return t;
  }
};

bool is_flat(const at::Tensor& t) { return t.dim() == 1; }

// Raises the error of a status (the message is this thread's).
PyObject* raise(tl_status st) {
  PyObject* r = PyObject_CallFunction(g_check, "i", static_cast<int>(st));
  Py_XDECREF(r);
  return nullptr;
}

// call(entry, want, inputs..., outputs...): outputs that are None are made where
// the bit of `want` is set.  The output, or for several a tuple with None for
// those left out; None if this is not the plain case.
PyObject* py_call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  const long e = nargs > 1 ? PyLong_AsLong(args[0]) : -1;
  const long want = nargs > 1 ? PyLong_AsLong(args[1]) : 0;
  if (PyErr_Occurred()) return nullptr;
  if (e < 0 || e >= kEntries || nargs != 2 + kSpec[e].nin + kSpec[e].nout) Py_RETURN_NONE;
  const Spec& sp = kSpec[e];
  PyObject* const* in = args + 2;
  PyObject* const* out = in + sp.nin;
  Fields f;
  tl_cfield cin[7];
  tl_field cout[7] = {};
  for (int i = 0; i < sp.nin; ++i)
    if (!f.take(in[i], sp.in[i], &cin[i])) Py_RETURN_NONE;
  bool any = false;
  for (int i = 0; i < sp.nout; ++i) {
    if (out[i] != Py_None && !f.take(out[i], sp.out[i], &cout[i])) Py_RETURN_NONE;
    any = any || out[i] != Py_None || (want >> i & 1);
  }
  if (!any || watched() || !f.current()) Py_RETURN_NONE;
  const bool flat = is_flat(THPVariable_Unpack(in[sp.alpha]));
  std::array<at::Tensor, 7> made;
  tl_status st;
  {
    pybind11::gil_scoped_release nogil;
    for (int i = 0; i < sp.nout; ++i)
      if (out[i] == Py_None && (want >> i & 1))
        made[i] = f.make(sp.out[i], flat && sp.out[i] == 1, &cout[i]);
    st = call(static_cast<Entry>(e), f.n, cin, cout, f.stream());
  }
  if (st != TL_OK) return raise(st);
  const auto result = [&](int i) {
    if (!made[i].defined()) {
      Py_INCREF(out[i]);
      return out[i];
    }
    return THPVariable_Wrap(made[i]);
  };
  if (sp.nout == 1) return result(0);
  PyObject* t = PyTuple_New(sp.nout);
  if (t == nullptr) return nullptr;
  for (int i = 0; i < sp.nout; ++i) {
    PyObject* r = result(i);
    if (r == nullptr) {
      Py_DECREF(t);
      return nullptr;
    }
    PyTuple_SET_ITEM(t, i, r);
  }
  return t;
  END_HANDLE_TH_ERRORS
}

// fields(what, comps, inputs..., outputs...): an expression (what < 0: its id is
// -1 - what) or a generated entry point (what: its address).  comps: one byte a
// field, the inputs', then the outputs', then the number of inputs.  As call().
typedef tl_status (*Generated)(int64_t, const tl_cfield*, int32_t, const tl_field*, int32_t, void*,
                               const tl_tune*);
PyObject* py_fields(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs < 4 || !PyBytes_CheckExact(args[1])) Py_RETURN_NONE;
  const long long what = PyLong_AsLongLong(args[0]);
  if (PyErr_Occurred()) return nullptr;
  const unsigned char* comps = reinterpret_cast<unsigned char*>(PyBytes_AS_STRING(args[1]));
  const Py_ssize_t all = PyBytes_GET_SIZE(args[1]) - 1;
  if (all < 1 || all > 16 || nargs != 2 + all) Py_RETURN_NONE;
  const int nin = comps[all], nout = static_cast<int>(all) - nin;
  if (nin < 1 || nin > 8 || nout < 1 || nout > 8) Py_RETURN_NONE;
  PyObject* const* in = args + 2;
  PyObject* const* out = in + nin;
  Fields f;
  tl_cfield cin[8];
  tl_field cout[8];
  for (int i = 0; i < nin; ++i)
    if (!f.take(in[i], comps[i], &cin[i])) Py_RETURN_NONE;
  for (int i = 0; i < nout; ++i)
    if (out[i] != Py_None && !f.take(out[i], comps[nin + i], &cout[i])) Py_RETURN_NONE;
  if (watched() || !f.current()) Py_RETURN_NONE;
  const bool flat = is_flat(THPVariable_Unpack(in[what < 0 ? nin - 1 : 0]));
  std::array<at::Tensor, 8> made;
  tl_status st;
  {
    pybind11::gil_scoped_release nogil;
    for (int i = 0; i < nout; ++i)
      if (out[i] == Py_None)
        made[i] = f.make(comps[nin + i], flat && comps[nin + i] == 1, &cout[i]);
    st = what < 0 ? g_expr(static_cast<int32_t>(-1 - what), f.n, cin, nin, cout[0], f.stream(), nullptr)
                  : reinterpret_cast<Generated>(static_cast<uintptr_t>(what))(
                        f.n, cin, nin, cout, nout, f.stream(), nullptr);
  }
  if (st != TL_OK) return raise(st);
  PyObject* t = PyTuple_New(nout);
  if (t == nullptr) return nullptr;
  for (int i = 0; i < nout; ++i) {
    PyObject* r = made[i].defined() ? THPVariable_Wrap(made[i]) : out[i];
    if (r == nullptr) {
      Py_DECREF(t);
      return nullptr;
    }
    if (!made[i].defined()) Py_INCREF(r);
    PyTuple_SET_ITEM(t, i, r);
  }
  return t;
  END_HANDLE_TH_ERRORS
}

// noalloc(domains): a list of dicts with every field given; the list of outputs.
PyObject* g_keys[7] = {};  // "g", "dg", "beta", "dbeta", "K", "alpha", "dtg"
PyObject* py_noalloc(PyObject*, PyObject* domains) {
  HANDLE_TH_ERRORS
  if (!PyList_CheckExact(domains)) Py_RETURN_NONE;
  const Py_ssize_t nd = PyList_GET_SIZE(domains);
  if (nd < 1 || watched()) Py_RETURN_NONE;
  std::vector<tl_domain> doms(nd);
  std::vector<at::Tensor> hold;  // the buffers, while other threads may run
  hold.reserve(7 * nd);
  c10::Device device(c10::DeviceType::CPU);
  PyObject* outs = PyList_New(nd);
  if (outs == nullptr) return nullptr;
  bool plain = true;
  for (Py_ssize_t d = 0; plain && d < nd; ++d) {
    PyObject* x = PyList_GET_ITEM(domains, d);
    plain = PyDict_CheckExact(x);
    Fields f;
    tl_cfield c[6];
    static const int comps[7] = {6, 18, 3, 9, 6, 1, 6};
    for (int k = 0; plain && k < 7; ++k) {
      PyObject* t = PyDict_GetItemWithError(x, g_keys[k]);
      plain = t != nullptr && (k < 6 ? f.take(t, comps[k], &c[k]) : f.take(t, 6, &doms[d].dtg));
      if (!plain) break;
      hold.push_back(THPVariable_Unpack(t));
      if (k == 6) {
        Py_INCREF(t);
        PyList_SET_ITEM(outs, d, t);
      }
    }
    if (!plain) break;
    if (d == 0) device = f.device;
    plain = f.device == device && (d > 0 || f.current());
    doms[d].n = f.n;
    doms[d].g = c[0];
    doms[d].dg = c[1];
    doms[d].beta = c[2];
    doms[d].dbeta = c[3];
    doms[d].K = c[4];
    doms[d].alpha = c[5];
  }
  if (!plain) {
    Py_DECREF(outs);
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  void* stream = c10::hip::getCurrentHIPStream(device.index()).stream();
  tl_status st;
  {
    pybind11::gil_scoped_release nogil;
    st = g_noalloc(doms.data(), static_cast<int32_t>(nd), nullptr, stream);
  }
  if (st != TL_OK) {
    Py_DECREF(outs);
    return raise(st);
  }
  return outs;
  END_HANDLE_TH_ERRORS
}

// plan_launch(plan, device): runs a plan on the current stream; True, or None if
// another device is current.
PyObject* py_plan_launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 2) Py_RETURN_NONE;
  void* plan = PyLong_AsVoidPtr(args[0]);
  const long device = PyLong_AsLong(args[1]);
  if (PyErr_Occurred()) return nullptr;
  if (plan == nullptr || device != c10::hip::current_device()) Py_RETURN_NONE;
  void* stream = c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(device)).stream();
  tl_status st;
  {
    pybind11::gil_scoped_release nogil;
    st = g_plan_launch(static_cast<tl_batch_plan*>(plan), stream);
  }
  if (st != TL_OK) return raise(st);
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// ---- The fused chain as an autograd node ------------------------------------

// Whether the calls of this thread are being recorded (ops.record).  A backward
// pass runs on the caller's thread where the engine's own are switched off, and
// its call is then recorded as any other.
thread_local bool t_recording = false;

PyObject* py_recording(PyObject*, PyObject* on) {
  const int v = PyObject_IsTrue(on);
  if (v < 0) return nullptr;
  t_recording = v != 0;
  Py_RETURN_NONE;
}

// Takes the inputs of an entry, which it has checked once already.
bool take_all(Entry e, const at::Tensor* const* t, Fields* f, tl_cfield* c) {
  for (int i = 0; i < kSpec[e].nin; ++i)
    if (!f->take(*t[i], kSpec[e].in[i], &c[i])) return false;
  return true;
}

// Throws the error that is set in the interpreter, which this thread may give up
// before it is handled.
[[noreturn]] void throw_python() {
  python_error e;
  e.persist();
  throw std::move(e);
}

// The error of a failed call, as _abi.check gives it; from a thread that may
// not hold the interpreter.
void check_native(tl_status st) {
  if (st == TL_OK) return;
  pybind11::gil_scoped_acquire gil;
  raise(st);
  throw_python();
}

// The adjoint through the Python entry point, for a saved tensor that a hook has
// changed, a gradient that is not a plain tensor or a call that is recorded.
torch::autograd::variable_list backward_python(const at::Tensor* const* in, const bool* wanted) {
  pybind11::gil_scoped_acquire gil;
  torch::autograd::variable_list grads(6);
  PyObject* args = PyTuple_New(12);
  if (args == nullptr) throw_python();
  for (int i = 0; i < 6; ++i) {
    PyObject* t = THPVariable_Wrap(*in[i]);
    if (t == nullptr) {
      Py_DECREF(args);
      throw_python();
    }
    PyTuple_SET_ITEM(args, i, t);
    PyTuple_SET_ITEM(args, 6 + i, PyBool_FromLong(wanted[i]));
  }
  PyObject* m = PyImport_ImportModule("paper_1804_10120_amd.autograd");
  PyObject* fn = m ? PyObject_GetAttrString(m, "_backward") : nullptr;
  PyObject* r = fn ? PyObject_CallObject(fn, args) : nullptr;
  Py_XDECREF(fn);
  Py_XDECREF(m);
  Py_DECREF(args);
  if (r == nullptr) throw_python();
  for (int i = 0; i < 6; ++i) {
    PyObject* t = PyTuple_GET_ITEM(r, i);
    if (t != Py_None) grads[i] = THPVariable_Unpack(t);
  }
  Py_DECREF(r);
  return grads;
}

// A gradient may be taken once: a second derivative raises, as for a Python
// function marked once_differentiable.
torch::autograd::variable_list once(torch::autograd::variable_list grads) {
  at::AutoGradMode on(true);
  for (auto& g : grads)
    if (g.defined()) g = g.detach().set_requires_grad(true);
  torch::autograd::DelayedError error(
      "trying to differentiate twice a function that was marked with @once_differentiable",
      static_cast<int64_t>(grads.size()));
  return error.apply(std::move(grads));
}

struct DtgChain : torch::autograd::Function<DtgChain> {
  static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& g,
                            const at::Tensor& dg, const at::Tensor& beta, const at::Tensor& dbeta,
                            const at::Tensor& K, const at::Tensor& alpha) {
    const at::Tensor* in[] = {&g, &dg, &beta, &dbeta, &K, &alpha};
    Fields f;
    tl_cfield c[6];
    tl_field o;
    TORCH_CHECK(take_all(kChain, in, &f, c), "dtg_chain: inputs changed during the call");
    at::Tensor out = f.make(6, false, &o);
    check_native(call(kChain, f.n, c, &o, f.stream()));
    ctx->save_for_backward({g, dg, beta, K, alpha});
    return out;
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx,
                                                 torch::autograd::variable_list w) {
    const auto saved = ctx->get_saved_variables();
    const at::Tensor cot = w[0].contiguous();
    const at::Tensor* in[] = {&saved[0], &saved[1], &saved[2], &saved[3], &saved[4], &cot};
    torch::autograd::variable_list grads(6);
    bool wanted[6], any = false;
    for (int i = 0; i < 6; ++i) any = (wanted[i] = ctx->needs_input_grad(i)) || any;
    if (!any) return grads;
    {
      at::AutoGradMode off(false);
      Fields f;
      tl_cfield c[6];
      tl_field o[6] = {};
      if (t_recording || watched() || !take_all(kBwd, in, &f, c) || !f.current()) {
        grads = backward_python(in, wanted);
      } else {
        const bool flat = is_flat(saved[4]);
        for (int i = 0; i < 6; ++i)
          if (wanted[i]) grads[i] = f.make(kSpec[kBwd].out[i], flat && i == 5, &o[i]);
        check_native(call(kBwd, f.n, c, o, f.stream()));
      }
    }
    if (at::GradMode::is_enabled() && w[0].requires_grad()) return once(std::move(grads));
    return grads;
  }
};

// dtg_chain(g, dg, beta, dbeta, K, alpha): the differentiable chain.
PyObject* py_dtg_chain(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 6 || watched()) Py_RETURN_NONE;
  Fields f;
  tl_cfield c[6];
  for (int i = 0; i < 6; ++i) {
    if (!f.take(args[i], kSpec[kChain].in[i], &c[i])) Py_RETURN_NONE;
    if (THPVariable_Unpack(args[i])._fw_grad(0).defined()) Py_RETURN_NONE;
  }
  if (!f.current()) Py_RETURN_NONE;
  at::Tensor out;
  {
    pybind11::gil_scoped_release nogil;
    out = DtgChain::apply(THPVariable_Unpack(args[0]), THPVariable_Unpack(args[1]),
                          THPVariable_Unpack(args[2]), THPVariable_Unpack(args[3]),
                          THPVariable_Unpack(args[4]), THPVariable_Unpack(args[5]));
  }
  return THPVariable_Wrap(out);
  END_HANDLE_TH_ERRORS
}

// init(addresses, check): the entry points' addresses in the order of Entry, then
// tl_expr, tl_batch_run_noalloc and tl_batch_plan_launch.
PyObject* py_init(PyObject*, PyObject* args) {
  PyObject* addresses;
  PyObject* check;
  if (!PyArg_ParseTuple(args, "O!O", &PyTuple_Type, &addresses, &check)) return nullptr;
  if (PyTuple_GET_SIZE(addresses) != kEntries + 3) {
    PyErr_SetString(PyExc_ValueError, "init: wrong number of addresses");
    return nullptr;
  }
  void* a[kEntries + 3];
  for (int i = 0; i < kEntries + 3; ++i) {
    a[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (a[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: null address");
      return nullptr;
    }
  }
  for (int i = 0; i < kEntries; ++i) g_entry[i] = a[i];
  g_expr = reinterpret_cast<decltype(g_expr)>(a[kEntries]);
  g_noalloc = reinterpret_cast<decltype(g_noalloc)>(a[kEntries + 1]);
  g_plan_launch = reinterpret_cast<decltype(g_plan_launch)>(a[kEntries + 2]);
  Py_INCREF(check);
  Py_XSETREF(g_check, check);
  Py_RETURN_NONE;
}

#define TL_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f))
PyMethodDef kMethods[] = {
    {"init", py_init, METH_VARARGS, nullptr},
    {"call", TL_FAST(py_call), METH_FASTCALL, nullptr},
    {"fields", TL_FAST(py_fields), METH_FASTCALL, nullptr},
    {"noalloc", py_noalloc, METH_O, nullptr},
    {"plan_launch", TL_FAST(py_plan_launch), METH_FASTCALL, nullptr},
    {"dtg_chain", TL_FAST(py_dtg_chain), METH_FASTCALL, nullptr},
    {"recording", py_recording, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind(void) {
  static const char* const keys[7] = {"g", "dg", "beta", "dbeta", "K", "alpha", "dtg"};
  for (int k = 0; k < 7; ++k)
    if ((g_keys[k] = PyUnicode_InternFromString(keys[k])) == nullptr) return nullptr;
  return PyModule_Create(&kModule);
}
