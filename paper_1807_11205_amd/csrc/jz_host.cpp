// The binding's part of a call that every launch pays for: looking the tensors over and calling the C ABI.  A sequence of short layers is bound by it:
// in Python a call of jz_conv2d_fwd took 5.3 us of host time, of which the library and the launch are two; its kernel takes 4.
//
// Only what is certain is done here: ordinary tensors on the GPU that meet every condition.  Anything else (subclasses, wrappers without
// storage, wrong types or sizes, empty tensors) is left to the Python code, which says what is wrong.
#include <Python.h>
#include <stdint.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "jz.h"

namespace {

// the address of an ordinary, contiguous GPU tensor of this type and size (any size: numel < 0); 0: look closer
uint64_t address(PyObject* o, PyObject* dtype, long long numel) {
  if (!THPVariable_CheckExact(o) || (dtype && !THPDtype_Check(dtype))) return 0;
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || (dtype && t.scalar_type() != reinterpret_cast<THPDtype*>(dtype)->scalar_type) ||
        !t.is_contiguous() || (numel >= 0 && t.numel() != numel))
      return 0;
    return reinterpret_cast<uint64_t>(t.data_ptr());
  } catch (...) {
    return 0;
  }
}

// ptr(tensor, dtype, elements or None) -> address or None
PyObject* ptr(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3) Py_RETURN_NONE;
  long long numel = -1;
  if (a[2] != Py_None) {
    numel = PyLong_Check(a[2]) ? PyLong_AsLongLong(a[2]) : -1;
    if (numel <= 0) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
  }
  const uint64_t p = address(a[0], a[1], numel);
  if (p == 0) Py_RETURN_NONE;
  return PyLong_FromUnsignedLongLong(p);
}

bool workspace(PyObject* o, uint64_t* p, uint64_t* bytes) {  // a contiguous GPU tensor of any type, or None
  *p = *bytes = 0;
  if (o == Py_None) return true;
  *p = address(o, nullptr, -1);
  if (*p == 0) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  *bytes = (uint64_t)t.numel() * t.element_size();
  return true;
}

// ws(tensor) -> (address, bytes) or None
PyObject* ws(PyObject*, PyObject* o) {
  uint64_t p, bytes;
  if (o == Py_None || !workspace(o, &p, &bytes)) Py_RETURN_NONE;
  return Py_BuildValue("(KK)", (unsigned long long)p, (unsigned long long)bytes);
}

bool elements(int a, int b, int c, int d, long long* out) {
  long long n = a;
  return !__builtin_mul_overflow(n, (long long)b, &n) && !__builtin_mul_overflow(n, (long long)c, &n) && !__builtin_mul_overflow(n, (long long)d, &n) &&
         (*out = n) > 0;
}

constexpr long LOOK = 1 << 20;  // conv's answer where it made no call

// conv(function, operation, descriptor, first operand, second operand, output, workspace, dtype, stream, handle) -> status or LOOK; handle(stream) is the
// stream's handle, asked for last
PyObject* conv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10 || !PyObject_CheckBuffer(a[2])) return PyLong_FromLong(LOOK);
  Py_buffer view;
  if (PyObject_GetBuffer(a[2], &view, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return PyLong_FromLong(LOOK);
  }
  long status = LOOK;
  const uint64_t fn = PyLong_AsUnsignedLongLong(a[0]);
  const long op = PyLong_AsLong(a[1]);
  const jz_conv_desc* const d = static_cast<const jz_conv_desc*>(view.buf);
  if (PyErr_Occurred()) {
    PyErr_Clear();
  } else if (view.len == (Py_ssize_t)sizeof(jz_conv_desc) && d->stride_h > 0 && d->stride_w > 0 && op >= 0 && op <= 2) {
    const long long ph = (long long)d->H + 2ll * d->pad_h - d->R, pw = (long long)d->W + 2ll * d->pad_w - d->S;
    const long long P = ph / d->stride_h + 1, Q = pw / d->stride_w + 1;
    long long nx, nw, ny;
    if (ph >= 0 && pw >= 0 && P <= INT32_MAX && Q <= INT32_MAX && elements(d->N, d->H, d->W, d->C, &nx) && elements(d->K, d->R, d->S, d->C, &nw) &&
        elements(d->N, (int)P, (int)Q, d->K, &ny)) {
      const uint64_t p0 = address(a[3], a[7], op == JZ_BWD_DATA ? ny : nx), p1 = address(a[4], a[7], op == JZ_BWD_WEIGHT ? ny : nw);
      const uint64_t p2 = address(a[5], a[7], op == JZ_FWD ? ny : op == JZ_BWD_DATA ? nx : nw);
      uint64_t wp, wn;
      if (p0 && p1 && p2 && workspace(a[6], &wp, &wn)) {
        PyObject* const handle = PyObject_CallOneArg(a[9], a[8]);
        const uint64_t stream = handle ? PyLong_AsUnsignedLongLongMask(handle) : 0;
        Py_XDECREF(handle);
        if (PyErr_Occurred()) {
          PyBuffer_Release(&view);
          return nullptr;
        }
        auto* const call = reinterpret_cast<int (*)(const jz_conv_desc*, const void*, const void*, void*, void*, size_t, void*)>(fn);
        auto v = [](uint64_t p) { return reinterpret_cast<void*>(p); };
        Py_BEGIN_ALLOW_THREADS
        status = call(d, v(p0), v(p1), v(p2), v(wp), (size_t)wn, v(stream));
        Py_END_ALLOW_THREADS
      }
    }
  }
  PyBuffer_Release(&view);
  return PyLong_FromLong(status);
}

// invoke(function, (integers and addresses ...), stream) -> status: an entry point without floating-point arguments, at most 24 before the stream
template <size_t... I>
int spread(uint64_t fn, const uint64_t* v, std::index_sequence<I...>) {
  return reinterpret_cast<int (*)(decltype((void)I, uint64_t())...)>(fn)(v[I]...);
}
constexpr Py_ssize_t MOST = 24;
template <size_t N>
int call_n(uint64_t fn, const uint64_t* v, size_t n) {
  if constexpr (N <= (size_t)MOST + 1) return n == N ? spread(fn, v, std::make_index_sequence<N>{}) : call_n<N + 1>(fn, v, n);
  return JZ_ERR_UNSUPPORTED;
}
PyObject* invoke(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3 || !PyTuple_Check(a[1]) || PyTuple_GET_SIZE(a[1]) > MOST) {
    PyErr_SetString(PyExc_TypeError, "invoke(function, tuple of at most 24 integers, stream)");
    return nullptr;
  }
  const Py_ssize_t m = PyTuple_GET_SIZE(a[1]);
  uint64_t v[MOST + 1];
  for (Py_ssize_t i = 0; i < m; ++i) v[i] = PyLong_AsUnsignedLongLongMask(PyTuple_GET_ITEM(a[1], i));
  v[m] = PyLong_AsUnsignedLongLongMask(a[2]);
  const uint64_t fn = PyLong_AsUnsignedLongLong(a[0]);
  if (PyErr_Occurred()) return nullptr;
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call_n<1>(fn, v, (size_t)m + 1);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyMethodDef methods[] = {{"ptr", reinterpret_cast<PyCFunction>(ptr), METH_FASTCALL, nullptr},
                         {"ws", ws, METH_O, nullptr},
                         {"conv", reinterpret_cast<PyCFunction>(conv), METH_FASTCALL, nullptr},
                         {"invoke", reinterpret_cast<PyCFunction>(invoke), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_jz_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__jz_host() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddIntConstant(m, "LOOK", LOOK) != 0) return nullptr;
  return m;
}
