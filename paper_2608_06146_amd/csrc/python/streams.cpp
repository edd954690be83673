// Python's calls of padoc_session_open / _close, for streams that open and
// close by the hundred in every decode step.
//
// Such a call is tens of nanoseconds of work; through ctypes it costs 0.9 to
// 1.4 us of argument objects, conversions and releases of the interpreter
// lock, and a step of 64 branches makes 128 of them (a whole step with its
// opens and closes, 512 rows over 8 pages: 148 us, 86 with these).  Here the
// arguments are converted as ctypes converts them (int(), then the low 32
// bits) and the lock is kept.  The library is not linked: ctypes, which loads
// it on first use, hands over the two addresses.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

namespace {

using OpenFn = int (*)(void*, int32_t, int32_t, int32_t*);
using CloseFn = int (*)(void*, int32_t);

struct Streams {
  PyObject_HEAD
  void* session;
  OpenFn open;
  CloseFn close;
};

bool low32(PyObject* o, int32_t& v) {
  unsigned long x;
  if (PyLong_Check(o)) {
    x = PyLong_AsUnsignedLongMask(o);
  } else {
    PyObject* i = PyNumber_Long(o);
    if (!i) return false;
    x = PyLong_AsUnsignedLongMask(i);
    Py_DECREF(i);
  }
  if (x == (unsigned long)-1 && PyErr_Occurred()) return false;
  v = (int32_t)(uint32_t)x;
  return true;
}

PyObject* streams_new(PyTypeObject* type, PyObject* args, PyObject*) {
  unsigned long long session, open, close;
  if (!PyArg_ParseTuple(args, "KKK", &session, &open, &close)) return nullptr;
  Streams* s = reinterpret_cast<Streams*>(type->tp_alloc(type, 0));
  if (!s) return nullptr;
  s->session = reinterpret_cast<void*>((uintptr_t)session);
  s->open = reinterpret_cast<OpenFn>((uintptr_t)open);
  s->close = reinterpret_cast<CloseFn>((uintptr_t)close);
  return reinterpret_cast<PyObject*>(s);
}

void streams_dealloc(PyObject* self) {
  PyTypeObject* type = Py_TYPE(self);
  type->tp_free(self);
  Py_DECREF(type);
}

// The new stream's id, or the (negative) status.
PyObject* streams_open(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Streams* s = reinterpret_cast<Streams*>(self);
  int32_t parent, fork, id = 0;
  if (n != 2) return PyErr_Format(PyExc_TypeError, "open takes 2 arguments, got %zd", n);
  if (!low32(a[0], parent) || !low32(a[1], fork)) return nullptr;
  const int st = s->open(s->session, parent, fork, &id);
  return PyLong_FromLong(st ? st : id);
}

// The status.
PyObject* streams_close(PyObject* self, PyObject* arg) {
  Streams* s = reinterpret_cast<Streams*>(self);
  int32_t id;
  if (!low32(arg, id)) return nullptr;
  return PyLong_FromLong(s->close(s->session, id));
}

PyMethodDef kMethods[] = {
    {"open", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(streams_open)), METH_FASTCALL, nullptr},
    {"close", streams_close, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyType_Slot kSlots[] = {{Py_tp_new, reinterpret_cast<void*>(streams_new)},
                        {Py_tp_dealloc, reinterpret_cast<void*>(streams_dealloc)},
                        {Py_tp_methods, kMethods},
                        {0, nullptr}};

PyType_Spec kSpec = {"paper_2608_06146_amd._streams.Streams", sizeof(Streams), 0, Py_TPFLAGS_DEFAULT, kSlots};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_streams", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__streams() {
  PyObject* m = PyModule_Create(&kModule);
  if (!m) return nullptr;
  PyObject* t = PyType_FromSpec(&kSpec);
  if (!t || PyModule_AddObject(m, "Streams", t) < 0) {
    Py_XDECREF(t);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
