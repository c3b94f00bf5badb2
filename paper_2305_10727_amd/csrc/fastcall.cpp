// Python extension module _fastcall: calls the library's C functions from Python at a fraction of ctypes' cost.
//
// A launch of a small layer takes the GPU 3 us; ctypes with a dozen arguments (a c_void_p object per tensor, a conversion per
// argument, two Python calls for the stream) took the host 5.  A FastCall object holds a function pointer and a signature and
// converts its arguments in one pass: about half a microsecond, of a dozen arguments.
//
// Signature, one letter per C parameter:
//   p  tensor, integer address or None (NULL)
//   t  tensor on the GPU and contiguous (else ValueError), or None
//   i  integer (int, int64_t, an enum)
//   s  torch's current stream; takes no argument
// All of them travel in integer registers or 8-byte stack slots, so a function of any such parameters can be called through
// one function type (x86-64 System V: the callee reads its parameters, the caller cleans up).
//
// Tensors are read, and results allocated (empty()), through torch's C++ interface: data_ptr() by way of Python takes 60 ns a tensor, torch.empty
// by way of its Python arguments 1.8 us, which for the calls that prepare a layer's weights was half of what the host did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/ops/empty.h>
#include <stddef.h>
#include <string.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

constexpr int kMaxArgs = 24;
typedef int (*fn_t)(long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long, long);

struct FastCall {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  fn_t fn;
  PyObject* name;
  int n, wanted, raw;  // C parameters, Python arguments; raw: return the status instead of raising
  char sig[kMaxArgs + 1];
};

PyObject *s_data_ptr, *s_is_cuda, *s_is_contiguous;
PyObject *g_get_device, *g_get_stream, *g_raise;  // set by setup()

bool address_of(PyObject* o, bool check, long* out) {
  if (o == Py_None) {
    *out = 0;
    return true;
  }
  if (THPVariable_CheckExact(o)) {  // (a subclass of Tensor, or what has a tensor's methods, answers for itself below)
    try {
      const at::Tensor& t = THPVariable_Unpack(o);
      if (check && !t.is_cuda()) {
        PyErr_SetString(PyExc_ValueError, "gpusq works on device tensors only");
        return false;
      }
      if (check && !t.is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "gpusq needs contiguous tensors");
        return false;
      }
      *out = (long)(uintptr_t)t.data_ptr();
      return true;
    } catch (...) {
      torch::translate_exception_to_python(std::current_exception());
      return false;
    }
  }
  if (!check && PyLong_Check(o)) {
    *out = (long)PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
  }
  if (check) {
    PyObject* cuda = PyObject_GetAttr(o, s_is_cuda);
    if (!cuda) return false;
    const bool on_gpu = cuda == Py_True;
    Py_DECREF(cuda);
    if (!on_gpu) {
      PyErr_SetString(PyExc_ValueError, "gpusq works on device tensors only");
      return false;
    }
    PyObject* whole = PyObject_CallMethodNoArgs(o, s_is_contiguous);
    if (!whole) return false;
    const bool contiguous = whole == Py_True;
    Py_DECREF(whole);
    if (!contiguous) {
      PyErr_SetString(PyExc_ValueError, "gpusq needs contiguous tensors");
      return false;
    }
  }
  PyObject* p = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!p) return false;
  *out = (long)PyLong_AsUnsignedLongLongMask(p);
  Py_DECREF(p);
  return !PyErr_Occurred();
}

bool current_stream(long* out) {
  PyObject* dev = PyObject_CallNoArgs(g_get_device);
  if (!dev) return false;
  PyObject* s = PyObject_CallOneArg(g_get_stream, dev);
  Py_DECREF(dev);
  if (!s) return false;
  *out = (long)PyLong_AsUnsignedLongLongMask(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  FastCall* f = (FastCall*)self;
  const Py_ssize_t given = PyVectorcall_NARGS(nargsf);
  if (given != f->wanted || (kwnames && PyTuple_GET_SIZE(kwnames) != 0))
    return PyErr_Format(PyExc_TypeError, "%U takes %d positional arguments", f->name, f->wanted);
  long a[kMaxArgs] = {0};
  int at = 0;
  for (int i = 0; i < f->n; ++i) {
    switch (f->sig[i]) {
      case 's':
        if (!current_stream(&a[i])) return nullptr;
        break;
      case 'i':
        a[i] = PyLong_AsLong(args[at++]);
        if (a[i] == -1 && PyErr_Occurred()) return nullptr;
        break;
      default:
        if (!address_of(args[at++], f->sig[i] == 't', &a[i])) return nullptr;
    }
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f->fn(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15], a[16], a[17], a[18], a[19], a[20],
                 a[21], a[22], a[23]);
  Py_END_ALLOW_THREADS
  if (f->raw) return PyLong_FromLong(status);
  if (status == 0) Py_RETURN_NONE;
  PyObject* code = PyLong_FromLong(status);
  if (!code) return nullptr;
  PyObject* argv[2] = {code, f->name};
  PyObject* r = PyObject_Vectorcall(g_raise, argv, 2, nullptr);  // raises
  Py_DECREF(code);
  return r;
}

void dealloc(PyObject* self) {
  Py_XDECREF(((FastCall*)self)->name);
  Py_TYPE(self)->tp_free(self);
}

// FastCall(name, address, signature, raw=False)
PyObject* make(PyTypeObject* type, PyObject* args, PyObject*) {
  PyObject* name;
  unsigned long long address;
  const char* sig;
  int raw = 0;
  if (!PyArg_ParseTuple(args, "UKs|p", &name, &address, &sig, &raw)) return nullptr;
  const size_t n = strlen(sig);
  if (n > kMaxArgs || strspn(sig, "ptis") != n) {
    PyErr_SetString(PyExc_ValueError, "signature: up to 24 of p, t, i, s");
    return nullptr;
  }
  FastCall* f = (FastCall*)type->tp_alloc(type, 0);
  if (!f) return nullptr;
  f->vectorcall = call;
  f->fn = (fn_t)address;
  Py_INCREF(name);
  f->name = name;
  f->n = (int)n;
  f->wanted = 0;
  f->raw = raw;
  memcpy(f->sig, sig, n + 1);
  for (size_t i = 0; i < n; ++i) f->wanted += sig[i] != 's';
  return (PyObject*)f;
}

PyTypeObject g_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// setup(get_device, get_stream, on_error): the current device's number, the raw stream of a device, what a status other
// than 0 is handed to (with the function's name) and must raise
PyObject* setup(PyObject*, PyObject* args) {
  PyObject *dev, *stream, *err;
  if (!PyArg_ParseTuple(args, "OOO", &dev, &stream, &err)) return nullptr;
  Py_INCREF(dev);
  Py_INCREF(stream);
  Py_INCREF(err);
  Py_XSETREF(g_get_device, dev);
  Py_XSETREF(g_get_stream, stream);
  Py_XSETREF(g_raise, err);
  Py_RETURN_NONE;
}

// empty(like, dtype, *sizes): torch.empty(sizes, dtype=dtype, device=like.device)
PyObject* empty(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  constexpr int kMaxDims = 4;
  if (n < 3 || n > 2 + kMaxDims || !THPVariable_Check(args[0]) || !THPDtype_Check(args[1])) {
    PyErr_SetString(PyExc_TypeError, "empty(like, dtype, *sizes): a tensor, a dtype, up to 4 sizes");
    return nullptr;
  }
  int64_t sizes[kMaxDims];
  for (Py_ssize_t i = 2; i < n; ++i) {
    sizes[i - 2] = PyLong_AsLongLong(args[i]);
    if (sizes[i - 2] == -1 && PyErr_Occurred()) return nullptr;
  }
  const auto options = at::TensorOptions().dtype(((THPDtype*)args[1])->scalar_type).device(THPVariable_Unpack(args[0]).device());
  at::Tensor t;
  {
    pybind11::gil_scoped_release unlocked;
    t = at::empty(at::IntArrayRef(sizes, (size_t)(n - 2)), options);
  }
  return THPVariable_Wrap(std::move(t));
  END_HANDLE_TH_ERRORS
}

PyMethodDef g_methods[] = {{"empty", (PyCFunction)(void (*)(void))empty, METH_FASTCALL, "empty(like, dtype, *sizes)"},
                           {"setup", setup, METH_VARARGS, "setup(get_device, get_stream, on_error)"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", "C functions as cheap Python callables", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  g_type.tp_name = "_fastcall.FastCall";
  g_type.tp_basicsize = sizeof(FastCall);
  g_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
  g_type.tp_vectorcall_offset = offsetof(FastCall, vectorcall);
  g_type.tp_call = PyVectorcall_Call;
  g_type.tp_new = make;
  g_type.tp_dealloc = dealloc;
  if (PyType_Ready(&g_type) < 0) return nullptr;
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  PyObject* m = PyModule_Create(&g_module);
  if (!m || !s_data_ptr || !s_is_cuda || !s_is_contiguous) return nullptr;
  Py_INCREF(&g_type);
  if (PyModule_AddObject(m, "FastCall", (PyObject*)&g_type) < 0) return nullptr;
  return m;
}
