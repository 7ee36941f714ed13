// Calls of the C ABI from Python without ctypes: one object per library function, which turns its arguments into machine words
// and jumps.  A forward pass of a few tokens is five calls, each of which took longer on the host (3.8 to 4.7 us, 2.2 of them the
// launch) than its kernel on the GPU.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <utility>

namespace {

constexpr int kMaxWords = 20;

// What the Python side hands over: raises the error of a status; the pointer of something that is no plain tensor; torch's current
// device; the raw handle of a device's current stream
PyObject *g_fail = nullptr, *g_pointer = nullptr, *g_device = nullptr, *g_stream = nullptr;

struct Function {
  PyObject_HEAD
  vectorcallfunc call;
  void* address;
  PyObject* name;
  Py_ssize_t n_args;
  // one letter per argument: d descriptor, t tensor or None, w workspace tensor (its pointer and number of elements),
  // i integer, s stream or None
  char kinds[kMaxWords];
};

// The library's functions take pointers, sizes and 32-bit integers and return a 32-bit status: on x86-64 every argument
// travels in a 64-bit register or stack slot.
template <size_t>
using Word = uint64_t;
template <size_t... I>
int32_t jump(void* f, const uint64_t* w, std::index_sequence<I...>) {
  return reinterpret_cast<int32_t (*)(Word<I>...)>(f)(w[I]...);
}
using Jump = int32_t (*)(void*, const uint64_t*);
template <size_t N>
int32_t jump_n(void* f, const uint64_t* w) {
  return jump(f, w, std::make_index_sequence<N>());
}
template <size_t... N>
constexpr auto jumps(std::index_sequence<N...>) {
  struct Table {
    Jump of[sizeof...(N)];
  };
  return Table{{jump_n<N>...}};
}
constexpr auto kJumps = jumps(std::make_index_sequence<kMaxWords + 1>());

// the device pointer of a contiguous GPU tensor (0 for None); false with an exception set
bool pointer_of(PyObject* o, uint64_t* p) {
  if (o == Py_None) {
    *p = 0;
    return true;
  }
  if (THPVariable_CheckExact(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
      PyErr_SetString(PyExc_ValueError, "expected a contiguous GPU tensor");
      return false;
    }
    *p = (uint64_t)t.data_ptr();
    return true;
  }
  PyObject* r = PyObject_CallOneArg(g_pointer, o);
  if (!r) return false;
  *p = r == Py_None ? 0 : PyLong_AsUnsignedLongLong(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

bool elements_of(PyObject* o, uint64_t* n) {
  if (THPVariable_CheckExact(o)) {
    *n = (uint64_t)THPVariable_Unpack(o).numel();
    return true;
  }
  PyObject* r = PyObject_CallMethod(o, "numel", nullptr);
  if (!r) return false;
  *n = PyLong_AsUnsignedLongLong(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

bool stream_of(PyObject* o, uint64_t* s) {
  PyObject* r;
  if (o == Py_None) {
    PyObject* device = PyObject_CallNoArgs(g_device);
    if (!device) return false;
    r = PyObject_CallOneArg(g_stream, device);
    Py_DECREF(device);
  } else {
    r = PyObject_GetAttrString(o, "cuda_stream");
  }
  if (!r) return false;
  *s = PyLong_AsUnsignedLongLong(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

PyObject* call_function(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  HANDLE_TH_ERRORS
  Function* f = (Function*)self;
  if ((kwnames && PyTuple_GET_SIZE(kwnames) > 0) || PyVectorcall_NARGS(nargsf) != f->n_args) {
    PyErr_Format(PyExc_TypeError, "%U takes exactly %zd arguments", f->name, f->n_args);
    return nullptr;
  }
  uint64_t w[kMaxWords];
  int n = 0;
  for (Py_ssize_t i = 0; i < f->n_args; ++i) {
    PyObject* o = args[i];
    bool ok = true;
    switch (f->kinds[i]) {
      case 'd': {  // the caller holds the descriptor, and its memory does not move
        Py_buffer b;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return nullptr;
        w[n++] = (uint64_t)b.buf;
        ok = b.len >= (Py_ssize_t)(6 * sizeof(int32_t));
        PyBuffer_Release(&b);
        if (!ok) PyErr_SetString(PyExc_TypeError, "expected a descriptor");
        break;
      }
      case 't': ok = pointer_of(o, &w[n++]); break;
      case 'w':
        ok = pointer_of(o, &w[n]) && elements_of(o, &w[n + 1]);
        n += 2;
        break;
      case 'i': {
        PyObject* v = PyNumber_Index(o);
        if (!v) return nullptr;
        w[n++] = PyLong_AsUnsignedLongLongMask(v);
        Py_DECREF(v);
        ok = !PyErr_Occurred();
        break;
      }
      default: ok = stream_of(o, &w[n++]); break;
    }
    if (!ok) return nullptr;
  }
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = kJumps.of[n](f->address, w);
  Py_END_ALLOW_THREADS
  if (status != 0) {
    PyObject* r = PyObject_CallFunction(g_fail, "Oi", f->name, (int)status);
    if (!r) return nullptr;
    Py_DECREF(r);
  }
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

void free_function(PyObject* self) {
  Py_XDECREF(((Function*)self)->name);
  Py_TYPE(self)->tp_free(self);
}

PyTypeObject g_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// function(name, address, kinds)
PyObject* make_function(PyObject*, PyObject* args) {
  PyObject* name;
  unsigned long long address;
  const char* kinds;
  if (!PyArg_ParseTuple(args, "UKs", &name, &address, &kinds)) return nullptr;
  const size_t n = strlen(kinds);
  size_t words = n;
  for (const char* k = kinds; *k; ++k) words += *k == 'w';
  if (words > kMaxWords || strspn(kinds, "dtwis") != n) {
    PyErr_SetString(PyExc_ValueError, "bad argument kinds");
    return nullptr;
  }
  Function* f = PyObject_New(Function, &g_type);
  if (!f) return nullptr;
  f->call = call_function;
  f->address = (void*)(uintptr_t)address;
  Py_INCREF(name);
  f->name = name;
  f->n_args = (Py_ssize_t)n;
  memcpy(f->kinds, kinds, n);
  return (PyObject*)f;
}

// setup(fail, pointer, device, stream)
PyObject* setup(PyObject*, PyObject* args) {
  PyObject* v[4];
  if (!PyArg_ParseTuple(args, "OOOO", &v[0], &v[1], &v[2], &v[3])) return nullptr;
  PyObject** to[4] = {&g_fail, &g_pointer, &g_device, &g_stream};
  for (int i = 0; i < 4; ++i) {
    Py_INCREF(v[i]);
    Py_XDECREF(*to[i]);
    *to[i] = v[i];
  }
  Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"function", make_function, METH_VARARGS, nullptr}, {"setup", setup, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, g_methods};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
  g_type.tp_name = "paper_2505_14864_amd._fastcall.Function";
  g_type.tp_basicsize = sizeof(Function);
  g_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
  g_type.tp_vectorcall_offset = offsetof(Function, call);
  g_type.tp_call = PyVectorcall_Call;
  g_type.tp_dealloc = free_function;
  if (PyType_Ready(&g_type) < 0) return nullptr;
  return PyModule_Create(&g_module);
}
