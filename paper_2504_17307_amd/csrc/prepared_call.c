/* One marshalled call of the C ABI as a Python object: calling it makes that call again (uccl_prepare).  A call of
 * few small messages is bound by the host, and ctypes spends a seventh of it on taking C arguments out of their objects
 * and putting them into a frame each time.  Here they lie ready (loops of prepared calls, us each, by ctypes / here /
 * the same loop in C: a reset 3.02 / 2.76 / 2.68, 14 records of 4 KiB 3.73 / 3.45 / 3.34, or in a process in which HIP
 * launches faster 2.49 / 2.26 / 2.18 and 2.81 / 2.36 / 2.28; a call of no records 0.10). */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <structmember.h>

enum { MOST = 13 };

typedef struct {
  PyObject_HEAD
  vectorcallfunc call;
  void* fn;
  int n;
  uint64_t a[MOST];
  PyObject *failed, *keeps;   /* called with a code other than 0; what the caller gave */
  PyObject *holds, *name;     /* what else the arguments point into; of the function (either may be NULL) */
  PyObject *dict, *weak;
} Prepared;

/* Every argument of the ABI's functions is a pointer or a whole number of at most 64 bits: each takes one integer
 * register or one 8-byte stack slot of the x86-64 System V convention, of which the callee reads as much as its
 * type has. */
#if !defined(__x86_64__) || defined(_WIN32)
#error "prepared calls rely on the x86-64 System V calling convention"
#endif
typedef uint64_t W;
static int invoke(const Prepared* p) {
  const W* a = p->a;
  void* f = p->fn;
  switch (p->n) {
    case 0: return ((int (*)(void))f)();
    case 1: return ((int (*)(W))f)(a[0]);
    case 2: return ((int (*)(W, W))f)(a[0], a[1]);
    case 3: return ((int (*)(W, W, W))f)(a[0], a[1], a[2]);
    case 4: return ((int (*)(W, W, W, W))f)(a[0], a[1], a[2], a[3]);
    case 5: return ((int (*)(W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4]);
    case 6: return ((int (*)(W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5]);
    case 7: return ((int (*)(W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6]);
    case 8: return ((int (*)(W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]);
    case 9: return ((int (*)(W, W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8]);
    case 10: return ((int (*)(W, W, W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]);
    case 11: return ((int (*)(W, W, W, W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10]);
    case 12: return ((int (*)(W, W, W, W, W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11]);
    default: return ((int (*)(W, W, W, W, W, W, W, W, W, W, W, W, W))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12]);
  }
}

static PyObject* prepared_vectorcall(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* names) {
  (void)args;
  if (PyVectorcall_NARGS(nargsf) != 0 || (names != NULL && PyTuple_GET_SIZE(names) != 0)) {
    PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
    return NULL;
  }
  const Prepared* const p = (const Prepared*)self;
  int code;
  Py_BEGIN_ALLOW_THREADS   /* a launch may wait for room in its stream's queue */
  code = invoke(p);
  Py_END_ALLOW_THREADS
  if (code != 0) {
    PyObject* const r = PyObject_CallFunction(p->failed, "i", code);
    Py_XDECREF(r);
    if (r == NULL) return NULL;
  }
  Py_RETURN_NONE;
}

static PyObject* prepared_new(PyTypeObject* type, PyObject* args, PyObject* kw) {
  unsigned long long fn;
  PyObject *values, *failed, *keeps, *holds = NULL, *name = NULL;
  if (kw != NULL && PyDict_GET_SIZE(kw) != 0) {
    PyErr_SetString(PyExc_TypeError, "no keyword arguments");
    return NULL;
  }
  if (!PyArg_ParseTuple(args, "KO!OO|OO", &fn, &PyTuple_Type, &values, &failed, &keeps, &holds, &name)) return NULL;
  const Py_ssize_t n = PyTuple_GET_SIZE(values);
  if (fn == 0 || n > MOST || !PyCallable_Check(failed)) {
    PyErr_SetString(PyExc_ValueError, "a function's address, at most 13 whole numbers, a callable and what to keep");
    return NULL;
  }
  Prepared* const p = (Prepared*)type->tp_alloc(type, 0);
  if (p == NULL) return NULL;
  p->call = prepared_vectorcall;
  p->fn = (void*)(uintptr_t)fn;
  p->n = (int)n;
  Py_INCREF(failed);
  p->failed = failed;
  Py_INCREF(keeps);
  p->keeps = keeps;
  Py_XINCREF(holds);
  p->holds = holds;
  Py_XINCREF(name);
  p->name = name;
  for (Py_ssize_t i = 0; i < n; ++i) {
    p->a[i] = PyLong_AsUnsignedLongLongMask(PyTuple_GET_ITEM(values, i));
    if (PyErr_Occurred()) {
      Py_DECREF(p);
      return NULL;
    }
  }
  return (PyObject*)p;
}

static int prepared_traverse(PyObject* self, visitproc visit, void* arg) {
  Py_VISIT(((Prepared*)self)->failed);
  Py_VISIT(((Prepared*)self)->keeps);
  Py_VISIT(((Prepared*)self)->holds);
  Py_VISIT(((Prepared*)self)->name);
  Py_VISIT(((Prepared*)self)->dict);
  return 0;
}
static int prepared_clear(PyObject* self) {
  Py_CLEAR(((Prepared*)self)->failed);
  Py_CLEAR(((Prepared*)self)->keeps);
  Py_CLEAR(((Prepared*)self)->holds);
  Py_CLEAR(((Prepared*)self)->name);
  Py_CLEAR(((Prepared*)self)->dict);
  return 0;
}
static void prepared_dealloc(PyObject* self) {
  PyObject_GC_UnTrack(self);
  if (((Prepared*)self)->weak != NULL) PyObject_ClearWeakRefs(self);
  prepared_clear(self);
  Py_TYPE(self)->tp_free(self);
}

static PyMemberDef members[] = {{"keeps", T_OBJECT_EX, offsetof(Prepared, keeps), READONLY, NULL},
                                {"__name__", T_OBJECT_EX, offsetof(Prepared, name), 0, NULL},
                                {NULL, 0, 0, 0, NULL}};
static PyGetSetDef getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, NULL, NULL}, {NULL, NULL, NULL, NULL, NULL}};
static PyTypeObject prepared_type = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "paper_2504_17307_amd._prepared.Prepared",
    .tp_basicsize = sizeof(Prepared),
    .tp_dealloc = prepared_dealloc,
    .tp_vectorcall_offset = offsetof(Prepared, call),
    .tp_call = PyVectorcall_Call,
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_traverse = prepared_traverse,
    .tp_clear = prepared_clear,
    .tp_members = members,
    .tp_getset = getset,
    .tp_dictoffset = offsetof(Prepared, dict),
    .tp_weaklistoffset = offsetof(Prepared, weak),
    .tp_new = prepared_new,
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_prepared", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__prepared(void) {
  if (PyType_Ready(&prepared_type) < 0) return NULL;
  PyObject* const m = PyModule_Create(&module);
  if (m == NULL) return NULL;
  Py_INCREF(&prepared_type);
  if (PyModule_AddObject(m, "Prepared", (PyObject*)&prepared_type) < 0) {
    Py_DECREF(&prepared_type);
    Py_DECREF(m);
    return NULL;
  }
  return m;
}
