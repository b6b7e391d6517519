// The per-call part of runner.LinearLUT and of the multi-matrix call in native code: the output tensor and the
// arguments of one or two library calls, without Python objects in between.
//
// A decode call of a small matrix is bound by its host time: 7.2 us a pass (256 x 256, 2 bit), of which 2.6 are the
// launch, whose arguments go to the device, 1.75 torch.empty called from Python, and the rest argument
// handling in Python and ctypes.  Here: 4.6 us; the two documented calls one after the other 11.9 -> 7.6 us.
//
// Every function returns None for what is not the ordinary case (tensor subclasses, tensors of other devices, active
// modes, types that do not go together): the caller then takes the path through binding.py, which also words the
// errors.  The library's functions come as addresses from binding.py, so that there is one copy of the library.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <cstdint>
#include <cstring>
#include <limits>

#include "tmac.h"

namespace {

decltype(&tmac_mpgemv_fused) g_mpgemv_fused;
decltype(&tmac_precompute_lut) g_precompute_lut;
decltype(&tmac_mpgemm) g_mpgemm;
decltype(&tmac_mpgemm_fused) g_mpgemm_fused;
decltype(&tmac_fused_workspace_bytes) g_fused_workspace_bytes;
decltype(&tmac_mpgemv_fused_multi) g_mpgemv_fused_multi;
PyObject* g_error;       // TmacError
PyTypeObject* g_wdesc;   // the ctypes structure tmac_wdesc

// A dense tensor of the GPU with nothing wrapped around it.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  static const c10::DispatchKeySet allowed({c10::DispatchKey::CUDA, c10::DispatchKey::ADInplaceOrView, c10::DispatchKey::AutogradCUDA,
                                            c10::DispatchKey::AutocastCUDA});
  return t.defined() && t.is_cuda() && (t.key_set().raw_repr() & ~allowed.raw_repr()) == 0 ? &t : nullptr;
}

bool take_desc(PyObject* o, tmac_wdesc* desc) {
  if (!PyObject_TypeCheck(o, g_wdesc)) return false;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return false;
  const bool whole = b.len == (Py_ssize_t)sizeof(*desc);
  if (whole) memcpy(desc, b.buf, sizeof(*desc));
  PyBuffer_Release(&b);
  return whole;
}

bool modes_active() { return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set(); }

// Without the interpreter's lock, as in torch's own functions: a call's allocation may wait for the device, and what it
// waits for may need another Python thread.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// What all calls have in common.
struct Call {
  tmac_wdesc desc;
  const at::Tensor *packed, *A, *act_scale = nullptr;
  int32_t N;
  tmac_act_t act;
  tmac_out_t out_t;
  float weight_scale;
  at::TensorOptions options;
  int64_t width;
  at::Tensor out;
  void* stream;

  const float* scale() const { return act_scale ? static_cast<const float*>(act_scale->data_ptr()) : nullptr; }

  // desc, packed, A, M, out_t, act, act_scale, weight_scale, device; false: not the ordinary case, or an error is set
  bool take(PyObject* const* a) {
    if (modes_active() || !take_desc(a[0], &desc)) return false;
    if (!(packed = plain(a[1])) || !(A = plain(a[2])) || A->dim() != 2) return false;
    if (!PyLong_CheckExact(a[3]) || !PyLong_CheckExact(a[4]) || !PyFloat_CheckExact(a[7])) return false;
    const long long M = PyLong_AsLongLong(a[3]), type = PyLong_AsLongLong(a[4]);
    if (PyErr_Occurred() || M < 0 || type < 0 || type > 2 || A->size(0) > std::numeric_limits<int32_t>::max()) return false;
    out_t = (tmac_out_t)type;
    N = (int32_t)A->size(0);
    const bool i8 = A->scalar_type() == at::kChar;
    if (!i8 && A->scalar_type() != at::kHalf) return false;
    act = i8 ? TMAC_ACT_I8 : TMAC_ACT_F16;
    if (a[5] != Py_None) {
      if (!PyLong_CheckExact(a[5])) return false;
      const long long x = PyLong_AsLongLong(a[5]);
      if (PyErr_Occurred() || x < 0 || x > 2 || (x == TMAC_ACT_I8) != i8) return false;
      act = (tmac_act_t)x;
    }
    if (a[6] != Py_None && !(act_scale = plain(a[6]))) return false;
    weight_scale = (float)PyFloat_AS_DOUBLE(a[7]);
    at::Device device(at::kCUDA);
    if (THPDevice_Check(a[8])) device = reinterpret_cast<THPDevice*>(a[8])->device;
    else if (!PyUnicode_Check(a[8]) || PyUnicode_CompareWithASCIIString(a[8], "cuda") != 0) return false;
    const at::ScalarType dt = out_t == TMAC_OUT_F32 ? at::kFloat : out_t == TMAC_OUT_F16 ? at::kHalf : at::kInt;
    options = at::TensorOptions().dtype(dt).device(device);
    width = M;
    stream = c10::hip::getCurrentHIPStream().stream();
    return true;
  }

  void allocate() { out = at::empty({A->size(0), width}, options); }
};

PyObject* refuse(tmac_status status, const char* where) {
  PyObject* e = PyObject_CallFunction(g_error, "is", (int)status, where);
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  return nullptr;
}

PyObject* ordinary_only() {
  if (PyErr_Occurred()) PyErr_Clear();  // (an argument that the general path words the error for)
  Py_RETURN_NONE;
}

// forward_fused(desc, packed, A, M, out_t, act, act_scale, weight_scale, device)
PyObject* forward_fused(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c;
  if (n != 9 || !c.take(a)) return ordinary_only();
  const void* packed = c.packed->data_ptr();
  const void* A = c.A->data_ptr();
  const float* scale = c.scale();
  const int64_t lda = c.A->stride(0);
  tmac_status st;
  {
    const Unlocked unlocked;
    c.allocate();
    st = g_mpgemv_fused(&c.desc, packed, A, c.act, c.N, lda, scale, c.weight_scale, c.out.data_ptr(), c.out_t, c.out.stride(0), c.stream);
  }
  return st == TMAC_OK ? THPVariable_Wrap(std::move(c.out)) : refuse(st, "tmac_mpgemv_fused");
  END_HANDLE_TH_ERRORS
}

// forward(desc, packed, A, M, out_t, None, act_scale, weight_scale, device, lut, lut_t, workspace, K, group, g)
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 15) return ordinary_only();
  const at::Tensor *lut = plain(a[9]), *ws = plain(a[11]);
  if (!lut || !ws) return ordinary_only();
  long long v[4];
  const int from[4] = {10, 12, 13, 14};
  for (int i = 0; i < 4; ++i) {
    if (!PyLong_CheckExact(a[from[i]])) return ordinary_only();
    v[i] = PyLong_AsLongLong(a[from[i]]);
    if (PyErr_Occurred() || v[i] < 0 || v[i] > std::numeric_limits<int32_t>::max()) return ordinary_only();
  }
  Call c;
  if (!c.take(a)) return ordinary_only();
  const void* packed = c.packed->data_ptr();
  const void* A = c.A->data_ptr();
  const float* scale = c.scale();
  void *lut_ptr = lut->data_ptr(), *ws_ptr = ws->data_ptr();
  const size_t lut_bytes = lut->nbytes(), ws_bytes = ws->nbytes();
  const int64_t lda = c.A->stride(0);
  const tmac_lut_t lut_t = (tmac_lut_t)v[0];
  tmac_status first, second = TMAC_OK;
  {
    const Unlocked unlocked;
    c.allocate();
    first = g_precompute_lut(A, c.act, c.N, (int32_t)v[1], lda, (int32_t)v[3], (int32_t)v[2], lut_t, lut_ptr, lut_bytes, c.stream);
    if (first == TMAC_OK)
      second = g_mpgemm(&c.desc, packed, lut_ptr, lut_t, c.N, scale, c.weight_scale, c.out.data_ptr(), c.out_t, c.out.stride(0), ws_ptr,
                        ws_bytes, c.stream);
  }
  if (first != TMAC_OK) return refuse(first, "tmac_precompute_lut");
  return second == TMAC_OK ? THPVariable_Wrap(std::move(c.out)) : refuse(second, "tmac_mpgemm");
  END_HANDLE_TH_ERRORS
}

// forward_one_call(desc, packed, A, M, out_t, None, act_scale, weight_scale, device, workspace)
PyObject* forward_one_call(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 10) return ordinary_only();
  const at::Tensor* ws = plain(a[9]);
  if (!ws) return ordinary_only();
  Call c;
  if (!c.take(a)) return ordinary_only();
  const size_t need = g_fused_workspace_bytes(&c.desc, c.N, c.act);
  if (need == 0 || (size_t)ws->numel() < need) return ordinary_only();  // (a workspace is made there)
  const void* packed = c.packed->data_ptr();
  const void* A = c.A->data_ptr();
  const float* scale = c.scale();
  void* const ws_ptr = ws->data_ptr();
  const size_t ws_bytes = ws->nbytes();
  const int64_t lda = c.A->stride(0);
  tmac_status st;
  {
    const Unlocked unlocked;
    c.allocate();
    st = g_mpgemm_fused(&c.desc, packed, A, c.act, c.N, lda, scale, c.weight_scale, c.out.data_ptr(), c.out_t, c.out.stride(0), ws_ptr,
                        ws_bytes, c.stream);
  }
  return st == TMAC_OK ? THPVariable_Wrap(std::move(c.out)) : refuse(st, "tmac_mpgemm_fused");
  END_HANDLE_TH_ERRORS
}

// multi(items, N, out_t, act): tmac_mpgemv_fused_multi on the current stream; items as there, in a list or tuple of tuples
PyObject* multi(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4 || modes_active() || !(PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0]))) return ordinary_only();
  // a tuple of its own: another thread may change a list while the library runs, and what it reads by address lives until
  // it returns
  const THPObjectPtr held(PySequence_Tuple(a[0]));
  if (!held) return nullptr;
  const Py_ssize_t count = PyTuple_GET_SIZE(held.get());
  if (count < 1 || count > TMAC_MULTI_MAX || !PyLong_CheckExact(a[1]) || !PyLong_CheckExact(a[2])) return ordinary_only();
  const long long N = PyLong_AsLongLong(a[1]), out_t = PyLong_AsLongLong(a[2]);
  long long act = -1;
  if (a[3] != Py_None) {
    if (!PyLong_CheckExact(a[3])) return ordinary_only();
    act = PyLong_AsLongLong(a[3]);
    if (act < 0 || act > 2) return ordinary_only();
  }
  if (PyErr_Occurred() || N < 1 || N > std::numeric_limits<int32_t>::max() || out_t < 0 || out_t > 2) return ordinary_only();
  tmac_wdesc descs[TMAC_MULTI_MAX];
  tmac_gemv_item items[TMAC_MULTI_MAX];
  for (Py_ssize_t i = 0; i < count; ++i) {
    PyObject* const t = PyTuple_GET_ITEM(held.get(), i);
    if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) < 4 || PyTuple_GET_SIZE(t) > 6) return ordinary_only();
    const Py_ssize_t len = PyTuple_GET_SIZE(t);
    const at::Tensor *packed = plain(PyTuple_GET_ITEM(t, 1)), *A = plain(PyTuple_GET_ITEM(t, 2)), *out = plain(PyTuple_GET_ITEM(t, 3));
    if (!take_desc(PyTuple_GET_ITEM(t, 0), &descs[i]) || !packed || !A || !out || A->dim() != 2 || out->dim() != 2) return ordinary_only();
    const bool i8 = A->scalar_type() == at::kChar;
    if (!i8 && A->scalar_type() != at::kHalf) return ordinary_only();
    if (act < 0) act = i8 ? TMAC_ACT_I8 : TMAC_ACT_F16;
    if ((act == TMAC_ACT_I8) != i8) return ordinary_only();
    const at::Tensor* scale = nullptr;
    if (len > 4 && PyTuple_GET_ITEM(t, 4) != Py_None && !(scale = plain(PyTuple_GET_ITEM(t, 4)))) return ordinary_only();
    float weight_scale = 1.f;
    if (len > 5) {
      if (!PyFloat_CheckExact(PyTuple_GET_ITEM(t, 5))) return ordinary_only();
      weight_scale = (float)PyFloat_AS_DOUBLE(PyTuple_GET_ITEM(t, 5));
    }
    items[i] = tmac_gemv_item{&descs[i], packed->data_ptr(), A->data_ptr(), A->stride(0),
                              scale ? static_cast<const float*>(scale->data_ptr()) : nullptr, weight_scale, out->data_ptr(), out->stride(0)};
  }
  void* const stream = c10::hip::getCurrentHIPStream().stream();
  tmac_status st;
  {
    const Unlocked unlocked;
    st = g_mpgemv_fused_multi(items, (int32_t)count, (tmac_act_t)act, (int32_t)N, (tmac_out_t)out_t, stream, nullptr);
  }
  if (st != TMAC_OK) return refuse(st, "tmac_mpgemv_fused_multi");
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// bind(TmacError, tmac_wdesc, addresses of tmac_mpgemv_fused, tmac_precompute_lut, tmac_mpgemm, tmac_mpgemm_fused,
// tmac_fused_workspace_bytes, tmac_mpgemv_fused_multi)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *error, *wdesc;
  unsigned long long f[6];
  if (!PyArg_ParseTuple(args, "OO!KKKKKK", &error, &PyType_Type, &wdesc, &f[0], &f[1], &f[2], &f[3], &f[4], &f[5])) return nullptr;
  Py_INCREF(error);
  Py_INCREF(wdesc);
  g_error = error;
  g_wdesc = reinterpret_cast<PyTypeObject*>(wdesc);
  g_mpgemv_fused = reinterpret_cast<decltype(g_mpgemv_fused)>(f[0]);
  g_precompute_lut = reinterpret_cast<decltype(g_precompute_lut)>(f[1]);
  g_mpgemm = reinterpret_cast<decltype(g_mpgemm)>(f[2]);
  g_mpgemm_fused = reinterpret_cast<decltype(g_mpgemm_fused)>(f[3]);
  g_fused_workspace_bytes = reinterpret_cast<decltype(g_fused_workspace_bytes)>(f[4]);
  g_mpgemv_fused_multi = reinterpret_cast<decltype(g_mpgemv_fused_multi)>(f[5]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"forward_fused", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(forward_fused)), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(forward)), METH_FASTCALL, nullptr},
    {"forward_one_call", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(forward_one_call)), METH_FASTCALL, nullptr},
    {"multi", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(multi)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tmac_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tmac_calls() {
  PyObject* const m = PyModule_Create(&module);
  // (torch's classes are compiled in: binding.py uses the module with this version only)
  if (m && PyModule_AddStringConstant(m, "torch_version", TMAC_TORCH_VERSION) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
