// CPython module `_qwam_call`: the per-token calls of qwam.py (quantize_act,
// quantize_act_deflated, asp_linear, asp_layer) without ctypes.
//
// A few-token call runs for 5-10 us on the GPU; marshalling one through ctypes
// took 14 us of Python (nine tensor checks of the layer, four or five of the
// arguments, the struct, the stream lookup), which was the whole time of such
// a call.  The same checks here take under 1 us.  Every check runs on every
// call, on the tensors that the layer holds at that time; nothing is kept
// between calls.
//
// Each function returns its outputs, the library's status as an int when the
// library refused the call, or None when an argument is not what the fast path
// takes (a wrong device, type, shape or stride): qwam.py then goes the long
// way, which names the argument that is wrong.  asp_linear and asp_layer go
// there with an explicit stream too; an activation call does not, because the
// workspace of its stream made it dearer there than without one (26 us of host
// time against 16).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <initializer_list>
#include <memory>

#include "../../include/qwam.h"

namespace {

// entry points of the libqwam that qwam.py loaded
decltype(&qwam_quantize_act_ws) g_quantize;
decltype(&qwam_quantize_act_workspace) g_workspace;
decltype(&qwam_asp_linear) g_linear;
decltype(&qwam_asp_layer) g_layer;

enum Attr { kK, kN, kR, kGroup, kHadamard, kWq, kWs, kInv, kL1t, kL2t, kBias, kL1, kWsp, kL1f, kAttrs };
const char* const kAttrNames[kAttrs] = {"K",   "N",   "r",    "group", "hadamard", "wq",  "ws",
                                        "inv_smooth", "L1t", "L2t", "bias",  "L1",       "wsp", "L1f"};
PyObject* g_names[kAttrs];
PyObject *g_cuda_stream, *g_device_index;

// the data pointer of a contiguous GPU tensor of this type and shape; false otherwise
bool data_of(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape, void** out) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != type || t.dim() != static_cast<int64_t>(shape.size())) return false;
  int64_t i = 0;
  for (const int64_t s : shape)
    if (t.size(i++) != s) return false;
  if (!t.is_contiguous()) return false;
  *out = t.data_ptr();
  return true;
}

// A layer's struct, and references that keep its tensors alive during the call.
struct Layer {
  PyObject* held[kAttrs] = {};
  qwam_layer c = {};
  ~Layer() {
    for (PyObject* o : held) Py_XDECREF(o);
  }
  bool read_int(Attr a, int32_t& v) {
    if (!PyLong_Check(held[a])) return false;
    const long x = PyLong_AsLong(held[a]);
    if (x == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    v = static_cast<int32_t>(x);
    return v == x;
  }
  template <typename T>
  bool read(Attr a, at::ScalarType type, std::initializer_list<int64_t> shape, const T*& p, bool optional) {
    if (optional && held[a] == Py_None) return true;
    void* q = nullptr;
    if (!data_of(held[a], type, shape, &q)) return false;
    p = static_cast<const T*>(q);
    return true;
  }
  bool load(PyObject* o) {
    for (int a = 0; a < kAttrs; ++a) {
      held[a] = PyObject_GetAttr(o, g_names[a]);
      if (held[a] == nullptr) {
        PyErr_Clear();
        return false;
      }
    }
    if (!read_int(kK, c.K) || !read_int(kN, c.N) || !read_int(kR, c.r) || !read_int(kGroup, c.group) ||
        !read_int(kHadamard, c.hadamard) || c.K <= 0 || c.group <= 0)
      return false;
    const int64_t G = c.K / c.group;
    return read(kWq, at::kByte, {c.N, c.K / 2}, c.wq, false) && read(kWs, at::kFloat, {G, c.N}, c.ws, false) &&
           read(kInv, at::kFloat, {c.K}, c.inv_smooth, false) && read(kL1t, at::kBFloat16, {c.r, c.K}, c.L1t, false) &&
           read(kL2t, at::kBFloat16, {c.N, c.r}, c.L2t, false) && read(kBias, at::kBFloat16, {c.N}, c.bias, true) &&
           read(kL1, at::kBFloat16, {c.K, c.r}, c.L1, true) && read(kWsp, at::kInt, {G, c.N}, c.wsp, true) &&
           read(kL1f, at::kBFloat16, {c.K / 64, c.r / 16, 2, 64, 8}, c.L1f, true);
  }
};

// the number of rows of a 2-d GPU tensor; -1 for anything else
int64_t rows_of(PyObject* o) {
  if (!THPVariable_Check(o)) return -1;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.dim() == 2 && t.size(0) <= INT32_MAX ? t.size(0) : -1;
}

// the rows of `like` and an output of `cols` columns on its device, or `given`
bool output(PyObject* given, const at::Tensor& like, at::ScalarType type, int64_t rows, int64_t cols, PyObject** obj,
            void** data) {
  if (given == nullptr || given == Py_None) {
    const at::Tensor t = at::empty({rows, cols}, like.options().dtype(type));
    *data = t.data_ptr();
    *obj = THPVariable_Wrap(t);
    return *obj != nullptr;
  }
  if (!data_of(given, type, {rows, cols}, data)) return false;
  Py_INCREF(given);
  *obj = given;
  return true;
}

struct Held {
  PyObject* o = nullptr;
  ~Held() { Py_XDECREF(o); }
  PyObject* release() {
    PyObject* r = o;
    o = nullptr;
    return r;
  }
};

PyObject* none_or_error() {
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the handle of a torch.cuda.Stream of the current device; false for another device's
bool stream_of(PyObject* o, hipStream_t* out) {
  Held handle, device;
  handle.o = PyObject_GetAttr(o, g_cuda_stream);
  device.o = handle.o == nullptr ? nullptr : PyObject_GetAttr(o, g_device_index);
  if (device.o == nullptr) return false;
  *out = static_cast<hipStream_t>(PyLong_AsVoidPtr(handle.o));
  const long index = PyLong_AsLong(device.o);
  return !PyErr_Occurred() && index == c10::hip::current_device();
}

// quantize(layer, x, out, deflated, stream) -> (xq, xs, t); stream a torch.cuda.Stream or None
PyObject* py_quantize(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 5) Py_RETURN_NONE;
  Layer L;
  const int64_t M = rows_of(args[1]);
  void* x;
  if (M < 0 || !L.load(args[0]) || !data_of(args[1], at::kBFloat16, {M, L.c.K}, &x)) return none_or_error();
  PyObject* given[3] = {nullptr, nullptr, nullptr};
  if (args[2] != Py_None) {
    if (!PyTuple_Check(args[2]) || PyTuple_GET_SIZE(args[2]) != 3) return none_or_error();
    for (int i = 0; i < 3; ++i) given[i] = PyTuple_GET_ITEM(args[2], i);
  }
  const at::Tensor& xt = THPVariable_Unpack(args[1]);
  hipStream_t given_stream = nullptr;
  const bool explicit_stream = args[4] != Py_None;
  if (explicit_stream && (!stream_of(args[4], &given_stream) || xt.get_device() != c10::hip::current_device()))
    return none_or_error();
  Held xq, xs, t;
  void *pq, *ps, *pt;
  if (!output(given[0], xt, at::kByte, M, L.c.K / 2, &xq.o, &pq) ||
      !output(given[1], xt, at::kFloat, L.c.K / L.c.group, M, &xs.o, &ps) ||
      !output(given[2], xt, at::kBFloat16, M, L.c.r, &t.o, &pt))
    return none_or_error();
  const int32_t deflated = PyObject_IsTrue(args[3]) == 1;
  // few tokens and a large K: the call splits K over workgroups through a
  // workspace, from the pool of the stream the call runs on (dropped below: the
  // next user of that memory runs behind the call's kernels)
  const int64_t need = g_workspace(&L.c, static_cast<int32_t>(M), deflated);
  at::Tensor ws;
  std::unique_ptr<void, void (*)(void*)> ws_stream(nullptr, c10::hip::HIPCachingAllocator::raw_delete);
  if (need > 0) {
    if (explicit_stream)
      ws_stream.reset(c10::hip::HIPCachingAllocator::raw_alloc_with_stream(static_cast<size_t>(need), given_stream));
    else
      ws = at::empty({need}, xt.options().dtype(at::kByte));
  }
  void* const pw = need <= 0 ? nullptr : explicit_stream ? ws_stream.get() : ws.data_ptr();
  void* stream = explicit_stream ? given_stream : current_stream();
  qwam_status st;
  Py_BEGIN_ALLOW_THREADS
  st = g_quantize(&L.c, static_cast<int32_t>(M), deflated, static_cast<const uint16_t*>(x), static_cast<uint8_t*>(pq),
                  static_cast<float*>(ps), static_cast<uint16_t*>(pt), pw, need > 0 ? need : 0, stream);
  Py_END_ALLOW_THREADS
  if (st != QWAM_OK) return PyLong_FromLong(st);
  return PyTuple_Pack(3, xq.o, xs.o, t.o);
  END_HANDLE_TH_ERRORS
}

// linear(layer, xq, xs, t, out) -> y
PyObject* py_linear(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 5) Py_RETURN_NONE;
  Layer L;
  const int64_t M = rows_of(args[1]);
  void *xq, *xs, *t, *py;
  if (M < 0 || !L.load(args[0]) || !data_of(args[1], at::kByte, {M, L.c.K / 2}, &xq) ||
      !data_of(args[2], at::kFloat, {L.c.K / L.c.group, M}, &xs) || !data_of(args[3], at::kBFloat16, {M, L.c.r}, &t))
    return none_or_error();
  Held y;
  if (!output(args[4], THPVariable_Unpack(args[1]), at::kBFloat16, M, L.c.N, &y.o, &py)) return none_or_error();
  void* stream = current_stream();
  qwam_status st;
  Py_BEGIN_ALLOW_THREADS
  st = g_linear(&L.c, static_cast<int32_t>(M), static_cast<const uint8_t*>(xq), static_cast<const float*>(xs),
                static_cast<const uint16_t*>(t), static_cast<uint16_t*>(py), stream);
  Py_END_ALLOW_THREADS
  if (st != QWAM_OK) return PyLong_FromLong(st);
  return y.release();
  END_HANDLE_TH_ERRORS
}

// layer(layer, x, out) -> y (without the optional activation outputs)
PyObject* py_layer(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 3) Py_RETURN_NONE;
  Layer L;
  const int64_t M = rows_of(args[1]);
  void *x, *py;
  if (M < 0 || !L.load(args[0]) || !data_of(args[1], at::kBFloat16, {M, L.c.K}, &x)) return none_or_error();
  Held y;
  if (!output(args[2], THPVariable_Unpack(args[1]), at::kBFloat16, M, L.c.N, &y.o, &py)) return none_or_error();
  void* stream = current_stream();
  qwam_status st;
  Py_BEGIN_ALLOW_THREADS
  st = g_layer(&L.c, static_cast<int32_t>(M), static_cast<const uint16_t*>(x), static_cast<uint16_t*>(py), nullptr,
               nullptr, nullptr, stream);
  Py_END_ALLOW_THREADS
  if (st != QWAM_OK) return PyLong_FromLong(st);
  return y.release();
  END_HANDLE_TH_ERRORS
}

// bind(addresses of qwam_quantize_act_ws, qwam_quantize_act_workspace, qwam_asp_linear, qwam_asp_layer)
PyObject* py_bind(PyObject*, PyObject* args) {
  unsigned long long a[4];
  if (!PyArg_ParseTuple(args, "KKKK", &a[0], &a[1], &a[2], &a[3])) return nullptr;
  g_quantize = reinterpret_cast<decltype(&qwam_quantize_act_ws)>(a[0]);
  g_workspace = reinterpret_cast<decltype(&qwam_quantize_act_workspace)>(a[1]);
  g_linear = reinterpret_cast<decltype(&qwam_asp_linear)>(a[2]);
  g_layer = reinterpret_cast<decltype(&qwam_asp_layer)>(a[3]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    {"quantize", reinterpret_cast<PyCFunction>(py_quantize), METH_FASTCALL, nullptr},
    {"linear", reinterpret_cast<PyCFunction>(py_linear), METH_FASTCALL, nullptr},
    {"layer", reinterpret_cast<PyCFunction>(py_layer), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qwam_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qwam_call() {
  for (int a = 0; a < kAttrs; ++a)
    if ((g_names[a] = PyUnicode_InternFromString(kAttrNames[a])) == nullptr) return nullptr;
  if ((g_cuda_stream = PyUnicode_InternFromString("cuda_stream")) == nullptr ||
      (g_device_index = PyUnicode_InternFromString("device_index")) == nullptr)
    return nullptr;
  return PyModule_Create(&module);
}
