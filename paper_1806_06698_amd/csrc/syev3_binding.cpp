// syev3_binding.cpp -- the Python binding's common calls in native code.
//
// Each function takes the arguments of a valid call on plain tensors (the
// checks that the Python code makes attribute by attribute), allocates the
// outputs and calls the C entry point.  Anything else (a wrong shape, dtype
// or device, a tensor subclass, an active mode, an error code) returns None
// with nothing launched, and the Python code, which handles every case,
// reports or handles it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "syev3.h"

namespace {

// No mode is active that could change what a tensor operation does.
bool no_modes() {
  return !at::impl::torch_function_mode_enabled() &&
         !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
         !c10::impl::tls_is_dispatch_key_included(
             c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

// The tensor of an exact torch.Tensor on the GPU that is no wrapper of
// another (its data pointer is what it shows); NULL otherwise.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.is_neg() ||
      t.is_conj())
    return nullptr;
  const c10::DispatchKeySet ks = t.key_set();
  using K = c10::DispatchKey;
  for (K k : {K::Python, K::PythonTLSSnapshot, K::FuncTorchBatched, K::FuncTorchGradWrapper,
              K::Functionalize, K::Batched, K::ZeroTensor})
    if (ks.has(k)) return nullptr;
  return &t;
}

// (n, ld) of an SoA input, shape (6, n) with n >= 1, unit column stride and
// disjoint rows; false for anything else.
bool soa_geometry(const at::Tensor& a, int64_t* n, int64_t* ld) {
  if (a.dim() != 2 || a.size(0) != 6 || a.size(1) < 1) return false;
  *n = a.size(1);
  *ld = a.stride(0);
  return (*n == 1 || a.stride(1) == 1) && *ld >= *n;
}

bool same_kind(const at::Tensor& t, const at::Tensor& a) {
  return t.scalar_type() == a.scalar_type() && t.device() == a.device();
}

// An SoA output of the input's type and device: (rows, n), unit column
// stride, row stride >= n.
bool soa_output(const at::Tensor& t, int64_t rows, int64_t n, const at::Tensor& a) {
  return t.dim() == 2 && t.size(0) == rows && t.size(1) == n && same_kind(t, a) &&
         (n == 1 || t.stride(1) == 1) && t.stride(0) >= n;
}

// A packed output: exactly these sizes and strides (those of a single value
// do not matter).
bool packed_output(const at::Tensor& t, at::IntArrayRef sizes, at::IntArrayRef strides,
                   const at::Tensor& a) {
  return t.sizes() == sizes && same_kind(t, a) && (t.numel() <= 1 || t.strides() == strides);
}

hipStream_t current_stream(const at::Tensor& a) {
  return c10::hip::getCurrentHIPStream(a.get_device()).stream();
}

// A C call without the interpreter lock, as through ctypes.
template <typename F>
int unlocked(F f) {
  PyThreadState* s = PyEval_SaveThread();
  const int rc = f();
  PyEval_RestoreThread(s);
  return rc;
}

PyObject* pair(PyObject* lam, PyObject* V) {
  PyObject* r = lam && V ? PyTuple_Pack(2, lam, V) : nullptr;
  Py_XDECREF(lam);
  Py_XDECREF(V);
  return r;
}

// solve(A, layout, vectors, flags, refine, out) -> (lam, V or None), or None.
// layout: the C code (SYEV3_SOA, _AOS, _AOS9).
PyObject* solve_impl(PyObject* const* args) {
  const at::Tensor* pa = plain(args[0]);
  if (!pa || !no_modes()) Py_RETURN_NONE;
  const at::Tensor& a = *pa;
  const long layout = PyLong_AsLong(args[1]);
  const int vecs = PyObject_IsTrue(args[2]), refine = PyObject_IsTrue(args[4]);
  const unsigned long flags = PyLong_Check(args[3]) ? PyLong_AsUnsignedLong(args[3]) : ~0ul;
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (flags > 0xffffffffu || layout < SYEV3_SOA || layout > SYEV3_AOS9) Py_RETURN_NONE;
  int dtype;
  if (a.scalar_type() == at::kDouble) dtype = SYEV3_F64;
  else if (a.scalar_type() == at::kFloat) dtype = refine ? SYEV3_F32_REFINE : SYEV3_F32;
  else Py_RETURN_NONE;

  int64_t n = 0, ld = 0;
  if (layout == SYEV3_SOA) {
    if (!soa_geometry(a, &n, &ld)) Py_RETURN_NONE;
  } else {
    const int64_t width = layout == SYEV3_AOS ? 6 : 9;
    const bool full = layout == SYEV3_AOS9 && a.dim() == 3 && a.size(1) == 3 && a.size(2) == 3;
    if (!full && !(a.dim() == 2 && a.size(1) == width)) Py_RETURN_NONE;
    n = a.size(0);
    if (n < 1 || !a.is_contiguous()) Py_RETURN_NONE;
  }

  at::Tensor lam, V;
  if (args[5] == Py_None) {
    if (layout == SYEV3_SOA) {
      const at::Tensor buf = at::empty({vecs ? 12 : 3, n}, a.options());
      lam = buf.narrow(0, 0, 3);
      if (vecs) V = buf.narrow(0, 3, 9);
    } else {
      lam = at::empty({n, 3}, a.options());
      if (vecs) V = at::empty({n, 3, 3}, a.options());
    }
  } else {
    PyObject* out = args[5];
    if (!PyTuple_CheckExact(out) || PyTuple_GET_SIZE(out) != 2) Py_RETURN_NONE;
    const at::Tensor* l = plain(PyTuple_GET_ITEM(out, 0));
    const at::Tensor* v = vecs ? plain(PyTuple_GET_ITEM(out, 1)) : nullptr;
    if (!l || (vecs && !v)) Py_RETURN_NONE;
    if (layout == SYEV3_SOA) {
      if (!soa_output(*l, 3, n, a) || (vecs && !soa_output(*v, 9, n, a))) Py_RETURN_NONE;
    } else if (!packed_output(*l, {n, 3}, {3, 1}, a) ||
               (vecs && !packed_output(*v, {n, 3, 3}, {9, 3, 1}, a))) {
      Py_RETURN_NONE;
    }
    lam = *l;
    if (vecs) V = *v;
  }
  const hipStream_t stream = current_stream(a);
  const void* A = a.data_ptr();
  void *L = lam.data_ptr(), *W = vecs ? V.data_ptr() : nullptr;
  const int rc =
      layout == SYEV3_SOA
          ? unlocked([&] {
              return batched_syev3_strided(n, A, ld, L, lam.stride(0), W, vecs ? V.stride(0) : 0,
                                           dtype, (uint32_t)flags, stream);
            })
          : unlocked([&] {
              return batched_syev3_ex(n, A, 0, (int)layout, L, W, dtype, (uint32_t)flags, stream);
            });
  if (rc != SYEV3_OK) Py_RETURN_NONE;
  if (args[5] == Py_None) {
    PyObject* v = vecs ? THPVariable_Wrap(V) : (Py_INCREF(Py_None), Py_None);
    return pair(THPVariable_Wrap(lam), v);
  }
  PyObject *l = PyTuple_GET_ITEM(args[5], 0), *v = vecs ? PyTuple_GET_ITEM(args[5], 1) : Py_None;
  return PyTuple_Pack(2, l, v);
}

// segments(requests, stream_device, stream) -> True, or None.  requests: a
// list or tuple of (A, lam, V) or (A, lam, V, flags) lists or tuples;
// stream_device: the index of the stream's device and its handle, or None
// for the current stream of the requests' device.
PyObject* segments_impl(PyObject* const* args) {
  PyObject* list = args[0];
  if (!(PyList_CheckExact(list) || PyTuple_CheckExact(list)) || !no_modes()) Py_RETURN_NONE;
  const Py_ssize_t k = PySequence_Fast_GET_SIZE(list);
  if (k < 1 || k > SYEV3_SEGMENTS_MAX) Py_RETURN_NONE;
  std::vector<syev3_segment> segs((size_t)k);
  const at::Tensor* first = nullptr;
  for (Py_ssize_t i = 0; i < k; ++i) {
    PyObject* item = PySequence_Fast_GET_ITEM(list, i);
    if (!(PyList_CheckExact(item) || PyTuple_CheckExact(item))) Py_RETURN_NONE;
    const Py_ssize_t m = PySequence_Fast_GET_SIZE(item);
    if (m != 3 && m != 4) Py_RETURN_NONE;
    PyObject** q = PySequence_Fast_ITEMS(item);
    const at::Tensor* a = plain(q[0]);
    const at::Tensor* l = plain(q[1]);
    const at::Tensor* v = q[2] == Py_None ? nullptr : plain(q[2]);
    if (!a || !l || (q[2] != Py_None && !v)) Py_RETURN_NONE;
    if (!first) first = a;
    unsigned long flags = 0;
    if (m == 4) {
      flags = PyLong_Check(q[3]) ? PyLong_AsUnsignedLong(q[3]) : ~0ul;
      if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
      }
    }
    int64_t n, ld;
    if (a->device() != first->device() || flags > 0xffffffffu || !soa_geometry(*a, &n, &ld) ||
        !packed_output(*l, {3, n}, {n, 1}, *a) || (v && !packed_output(*v, {9, n}, {n, 1}, *a)))
      Py_RETURN_NONE;
    int dtype;
    if (a->scalar_type() == at::kDouble) dtype = SYEV3_F64;
    else if (a->scalar_type() == at::kFloat) dtype = SYEV3_F32_REFINE;
    else Py_RETURN_NONE;
    segs[(size_t)i] = syev3_segment{n, a->data_ptr(), ld, l->data_ptr(),
                                    v ? v->data_ptr() : nullptr, dtype, (uint32_t)flags};
  }
  hipStream_t stream;
  if (args[1] == Py_None) {
    stream = current_stream(*first);
  } else {
    const long dev = PyLong_AsLong(args[1]);
    void* handle = PyLong_AsVoidPtr(args[2]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    if (dev != first->get_device()) Py_RETURN_NONE;
    stream = (hipStream_t)handle;
  }
  const int rc =
      unlocked([&] { return syev3_solve_segments_noalloc((int32_t)k, segs.data(), stream); });
  if (rc != SYEV3_OK) Py_RETURN_NONE;
  Py_RETURN_TRUE;
}

// An allocation that fails raises in Python as torch's own would: the Python
// code makes the same call again.
template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != N) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return F(args);
  } catch (...) {
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"solve", (PyCFunction)(void (*)(void))guarded<solve_impl, 6>, METH_FASTCALL, nullptr},
    {"segments", (PyCFunction)(void (*)(void))guarded<segments_impl, 3>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  PyObject* m = PyModule_Create(&module);
  // the torch these calls were compiled against
  if (m && PyModule_AddStringConstant(m, "torch_version", SYEV3_TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
