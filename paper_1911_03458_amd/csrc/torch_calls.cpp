// The ordinary form of every operation's Python call -- plain contiguous tensors in, a new output
// tensor out, the current stream -- without the interpreter's share of it.
//
// binding.py's general path costs the host 9.5-12.5 us per call (three attribute chains and a shape
// tuple per tensor, torch.cuda.current_stream(), torch.empty(), ctypes): longer than most small kernels
// run, so programs that make one small call after another were bound by it (a 64x64 frame's block
// matching: 12.2 us a call around a kernel of 3.8 us).  Here the same checks, the allocation and the
// launch are one native call.  A call that is not of the ordinary form (an output or a stream given, a
// tensor subclass, a wrapped tensor of a transform, an active dispatch or function mode, a wrong shape,
// type or layout) is not judged here: call() returns None and binding.py's general path takes it,
// which accepts or refuses it as it says there.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <new>

#include "merit.h"

namespace {

// (binding.py takes their numbers from the module: OPS)
enum Op { CONV2D, CONV2D_PACKED, RESIDUAL, POOL2D, SAD, DEPTHWISE, SEPFILTER, BILATERAL, CORRELATION };
constexpr struct {
  const char *name;
  Op op;
} kOps[] = {{"merit_conv2d", CONV2D},       {"merit_conv2d_packed", CONV2D_PACKED},  {"merit_conv2d_residual", RESIDUAL},
            {"merit_pool2d", POOL2D},       {"merit_sad_search", SAD},               {"merit_conv2d_depthwise", DEPTHWISE},
            {"merit_sepfilter", SEPFILTER}, {"merit_bilateral", BILATERAL},          {"merit_correlation", CORRELATION}};

struct Shape {
  int64_t d[MERIT_MAX_DIMS];
  int n;
  at::IntArrayRef ref() const { return at::IntArrayRef(d, static_cast<size_t>(n)); }
};

// What a plan's calls need and never changes while the plan lives (binding.Plan owns the handle and drops
// this object when it destroys it).
struct Spec {
  merit_plan *plan;
  Shape out, a, b;
};

const char *kSpec = "merit.spec";

void free_spec(PyObject *capsule) { delete static_cast<Spec *>(PyCapsule_GetPointer(capsule, kSpec)); }

bool read_shape(PyObject *seq, Shape *s) {
  if (!PyTuple_Check(seq) || PyTuple_GET_SIZE(seq) > MERIT_MAX_DIMS) return false;
  s->n = static_cast<int>(PyTuple_GET_SIZE(seq));
  for (int i = 0; i < s->n; ++i) {
    s->d[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(seq, i));
    if (s->d[i] == -1 && PyErr_Occurred()) return false;
  }
  return true;
}

// spec(handle, out_shape, a_shape, b_shape) -> capsule
PyObject *make_spec(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Spec *s = n == 4 ? new (std::nothrow) Spec() : nullptr;
  if (s) {
    s->plan = static_cast<merit_plan *>(PyLong_AsVoidPtr(args[0]));
    if (!PyErr_Occurred() && read_shape(args[1], &s->out) && read_shape(args[2], &s->a) && read_shape(args[3], &s->b)) {
      PyObject *c = PyCapsule_New(s, kSpec, free_spec);
      if (c) return c;
    }
    delete s;
  }
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "spec(handle, out_shape, a_shape, b_shape)");
  return nullptr;
}

// Keys of tensors whose storage is not what it seems, or that a transform watches.
constexpr c10::DispatchKeySet kNotPlain({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                         c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                         c10::DispatchKey::Conjugate, c10::DispatchKey::Negative});

// The device tensor in `o` if it is an ordinary one of this type, else nullptr.
const at::Tensor *plain(PyObject *o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.scalar_type() != type) return nullptr;
  const c10::TensorImpl *impl = t.unsafeGetTensorImpl();
  if (impl->key_set().has_any(kNotPlain) || !impl->has_storage() || impl->has_symbolic_sizes_strides()) return nullptr;
  return t.is_contiguous() ? &t : nullptr;
}

const at::Tensor *plain(PyObject *o, at::ScalarType type, const Shape &shape) {
  const at::Tensor *t = plain(o, type);
  return t && t->sizes() == shape.ref() ? t : nullptr;
}

// call(op, spec, tensor...[, norm]) -> the output tensor(s); the status as an int if the library refuses;
// None if the call is not of the ordinary form.
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const long op = n >= 2 ? PyLong_AsLong(args[0]) : -1;
  if (op == -1 && PyErr_Occurred()) return nullptr;
  static const int tensors[] = {2, 2, 3, 1, 2, 2, 3, 3, 2};
  if (op < CONV2D || op > CORRELATION || n != 2 + tensors[op] + (op == BILATERAL)) {
    PyErr_SetString(PyExc_TypeError, "call(op, spec, tensor...[, norm])");
    return nullptr;
  }
  const Spec *s = static_cast<const Spec *>(PyCapsule_GetPointer(args[1], kSpec));
  if (!s) return nullptr;
  if (c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;

  const bool fp32 = op == POOL2D || op == SEPFILTER || op == BILATERAL;
  const at::ScalarType type = op == SAD ? at::kByte : fp32 ? at::kFloat : at::kHalf;
  const at::Tensor *t[3] = {nullptr, nullptr, nullptr};
  for (int i = 0; i < tensors[op]; ++i) {
    const Shape *shape = &s->b;
    if (i == 0) shape = op == SAD ? &s->b : &s->a;      // (block matching takes the current frame first)
    else if (op == SAD) shape = &s->a;
    else if (op == RESIDUAL && i == 2) shape = &s->out;
    t[i] = op == CONV2D_PACKED && i == 1 ? plain(args[2 + i], type) : plain(args[2 + i], type, *shape);
    if (!t[i]) Py_RETURN_NONE;
  }
  double norm = 0;
  if (op == BILATERAL) {
    if (!PyFloat_CheckExact(args[5])) Py_RETURN_NONE;
    norm = PyFloat_AS_DOUBLE(args[5]);
  }
  if (op == CONV2D_PACKED) {
    int64_t bytes = 0;      // (a tile request may have changed it)
    if (merit_plan_packed_weights_bytes(s->plan, &bytes) != MERIT_OK || t[1]->numel() * 2 != bytes) Py_RETURN_NONE;
  }

  const at::TensorOptions opts =
      at::TensorOptions().dtype(op == SAD ? at::kInt : type).device(t[0]->device());
  at::Tensor y = at::empty(s->out.ref(), opts), mv;
  if (op == SAD) mv = at::empty({s->out.d[0], s->out.d[1], 2}, opts);
  void *p[3] = {t[0]->data_ptr(), t[1] ? t[1]->data_ptr() : nullptr, t[2] ? t[2]->data_ptr() : nullptr};
  void *out = y.data_ptr(), *out2 = op == SAD ? mv.data_ptr() : nullptr;
  void *stream = c10::hip::getCurrentHIPStream().stream();

  merit_status st = MERIT_ERR_INVALID_ARG;
  Py_BEGIN_ALLOW_THREADS      // as a ctypes call does: a launch may wait for room in the queue
  switch (op) {
    case CONV2D: st = merit_conv2d(s->plan, p[0], p[1], out, stream); break;
    case CONV2D_PACKED: st = merit_conv2d_packed(s->plan, p[0], p[1], out, stream); break;
    case RESIDUAL: st = merit_conv2d_residual(s->plan, p[0], p[1], p[2], out, stream); break;
    case POOL2D: st = merit_pool2d(s->plan, p[0], out, stream); break;
    case SAD: st = merit_sad_search(s->plan, p[0], p[1], out, out2, stream); break;
    case DEPTHWISE: st = merit_conv2d_depthwise(s->plan, p[0], p[1], out, stream); break;
    case SEPFILTER: st = merit_sepfilter(s->plan, p[0], p[1], p[2], out, stream); break;
    case BILATERAL: st = merit_bilateral(s->plan, p[0], p[1], p[2], norm, out, stream); break;
    case CORRELATION: st = merit_correlation(s->plan, p[0], p[1], out, stream); break;
  }
  Py_END_ALLOW_THREADS
  if (st != MERIT_OK) return PyLong_FromLong(st);
  if (op != SAD) return THPVariable_Wrap(std::move(y));
  PyObject *first = THPVariable_Wrap(std::move(y));
  PyObject *second = first ? THPVariable_Wrap(std::move(mv)) : nullptr;
  PyObject *pair = second ? PyTuple_Pack(2, first, second) : nullptr;
  Py_XDECREF(first);
  Py_XDECREF(second);
  return pair;
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"spec", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(make_spec)), METH_FASTCALL, nullptr},
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls() {
  PyObject *m = PyModule_Create(&module), *ops = m ? PyDict_New() : nullptr;
  bool ok = ops != nullptr;
  for (const auto &o : kOps) {
    PyObject *v = ok ? PyLong_FromLong(o.op) : nullptr;
    ok = v && PyDict_SetItemString(ops, o.name, v) == 0;
    Py_XDECREF(v);
  }
  ok = ok && PyObject_SetAttrString(m, "OPS", ops) == 0 && PyModule_AddStringConstant(m, "TORCH", MERIT_TORCH) == 0;
  Py_XDECREF(ops);
  if (!ok) Py_CLEAR(m);
  return m;
}
