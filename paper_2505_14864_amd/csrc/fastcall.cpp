// Calls of the C ABI from Python without ctypes: one object per library function, which turns its arguments into machine words
// and jumps.  Only plain arguments are taken here; a call with any other one (a subclass of Tensor, a ctypes integer, and all that is
// refused) goes through ctypes as a whole, which decides what is accepted and how the rest is refused.  A forward pass of a few tokens is five calls, each of which took longer on the host (3.8 to 4.7 us, 2.2 of them the
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

// What the Python side hands over: raises the error of a status; the descriptor's type; torch's current device, by the call that
// initialises torch's GPU state (and refuses to in a forked child) and by the quick one that follows; the raw handle of a device's
// current stream
PyObject *g_fail = nullptr, *g_desc = nullptr, *g_first_device = nullptr, *g_device = nullptr, *g_stream = nullptr;
bool g_initialised = false;  // in this process

struct Function {
  PyObject_HEAD
  vectorcallfunc call;
  void* address;
  PyObject* name;
  PyObject* by_ctypes;  // the same call with the same arguments
  Py_ssize_t n_args;
  // one letter per argument: d descriptor, t contiguous GPU tensor or None, w workspace tensor (its pointer and number of
  // elements), i int, s stream or None
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

enum Taken { kPlain, kOther, kError };  // kError: with an exception set

Taken descriptor_of(PyObject* o, uint64_t* p) {
  if ((PyObject*)Py_TYPE(o) != g_desc) return kOther;
  Py_buffer b;  // the caller holds the descriptor, and its memory does not move
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return kError;
  *p = (uint64_t)b.buf;
  PyBuffer_Release(&b);
  return kPlain;
}

Taken tensor_of(PyObject* o, uint64_t* p, uint64_t* n) {
  if (!THPVariable_CheckExact(o)) return kOther;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) return kOther;
  *p = (uint64_t)t.data_ptr();
  if (n) *n = (uint64_t)t.numel();
  return kPlain;
}

Taken integer_of(PyObject* o, uint64_t* v) {
  if (!PyLong_Check(o)) return kOther;
  *v = PyLong_AsUnsignedLongLongMask(o);
  return PyErr_Occurred() ? kError : kPlain;
}

Taken stream_of(PyObject* o, uint64_t* s) {
  PyObject* r;
  if (o == Py_None) {
    PyObject* device = PyObject_CallNoArgs(g_initialised ? g_device : g_first_device);
    if (!device) return kError;
    g_initialised = true;
    r = PyObject_CallOneArg(g_stream, device);
    Py_DECREF(device);
  } else {
    r = PyObject_GetAttrString(o, "cuda_stream");
  }
  if (!r) return kError;
  const Taken taken = integer_of(r, s);
  Py_DECREF(r);
  return taken;
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
    Taken taken = kPlain;
    switch (f->kinds[i]) {
      case 'd': taken = descriptor_of(o, &w[n++]); break;
      case 't':
        if (o == Py_None) w[n] = 0;
        else taken = tensor_of(o, &w[n], nullptr);
        ++n;
        break;
      case 'w':
        taken = tensor_of(o, &w[n], &w[n + 1]);
        n += 2;
        break;
      case 'i': taken = integer_of(o, &w[n++]); break;
      default: taken = stream_of(o, &w[n++]); break;
    }
    if (taken == kOther) return PyObject_Vectorcall(f->by_ctypes, args, (size_t)f->n_args, nullptr);
    if (taken == kError) return nullptr;
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
  Py_XDECREF(((Function*)self)->by_ctypes);
  Py_TYPE(self)->tp_free(self);
}

PyTypeObject g_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// function(name, address, kinds, by_ctypes)
PyObject* make_function(PyObject*, PyObject* args) {
  PyObject *name, *by_ctypes;
  unsigned long long address;
  const char* kinds;
  if (!PyArg_ParseTuple(args, "UKsO", &name, &address, &kinds, &by_ctypes)) return nullptr;
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
  Py_INCREF(by_ctypes);
  f->by_ctypes = by_ctypes;
  f->n_args = (Py_ssize_t)n;
  memcpy(f->kinds, kinds, n);
  return (PyObject*)f;
}

// setup(fail, desc, first_device, device, stream)
PyObject* setup(PyObject*, PyObject* args) {
  PyObject* v[5];
  if (!PyArg_ParseTuple(args, "OOOOO", &v[0], &v[1], &v[2], &v[3], &v[4])) return nullptr;
  PyObject** to[5] = {&g_fail, &g_desc, &g_first_device, &g_device, &g_stream};
  for (int i = 0; i < 5; ++i) {
    Py_INCREF(v[i]);
    Py_XDECREF(*to[i]);
    *to[i] = v[i];
  }
  Py_RETURN_NONE;
}

// forked(): this process is a child
PyObject* forked(PyObject*, PyObject*) {
  g_initialised = false;
  Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"function", make_function, METH_VARARGS, nullptr},
                           {"setup", setup, METH_VARARGS, nullptr},
                           {"forked", forked, METH_NOARGS, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
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
