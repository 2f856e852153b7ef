/* The call of a bound program (fc_run_bound) as a Python type, for binding.BoundRun: a program of one short kernel takes
 * little longer on the device than Python and ctypes take to issue it (a call with its launch 2.7 to 2.8 us through this type, 3.0 to
 * 3.3 through a Python method and ctypes).  Knows two things: a function and the program it is called with. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

typedef struct {
  PyObject_HEAD
  PyObject *owner;                         /* keeps the program alive */
  const void *program;                     /* NULL: not armed */
  int (*run)(const void *program, void *stream);
} Bound;

static PyObject *bound_new(PyTypeObject *type, PyObject *args, PyObject *kwargs) {
  Bound *self = (Bound *)type->tp_alloc(type, 0);
  (void)args; (void)kwargs;
  return (PyObject *)self;                 /* zeroed: not armed */
}

static int bound_init(PyObject *self, PyObject *args, PyObject *kwargs) {
  (void)self; (void)args; (void)kwargs;
  return 0;
}

static void bound_dealloc(Bound *self) {
  Py_CLEAR(self->owner);
  Py_TYPE(self)->tp_free((PyObject *)self);
}

/* _arm(owner, program, run): from now on a call is run(program, stream) */
static PyObject *bound_arm(Bound *self, PyObject *args) {
  PyObject *owner;
  unsigned long long program, run;
  if (!PyArg_ParseTuple(args, "OKK", &owner, &program, &run)) return NULL;
  Py_INCREF(owner);
  Py_XSETREF(self->owner, owner);
  self->program = (const void *)(size_t)program;
  self->run = (int (*)(const void *, void *))(size_t)run;
  Py_RETURN_NONE;
}

static PyObject *bound_call(Bound *self, PyObject *args, PyObject *kwargs) {
  const Py_ssize_t n = PyTuple_GET_SIZE(args);
  PyObject *stream = n == 1 ? PyTuple_GET_ITEM(args, 0) : NULL;
  const int plain = n <= 1 && (kwargs == NULL || PyDict_GET_SIZE(kwargs) == 0) && (stream == NULL || stream == Py_None || PyLong_Check(stream));
  if (!plain || self->program == NULL) {   /* the Python method sees to everything else */
    PyObject *method = PyObject_GetAttrString((PyObject *)self, "_call");
    if (method == NULL) return NULL;
    PyObject *result = PyObject_Call(method, args, kwargs);
    Py_DECREF(method);
    return result;
  }
  void *on = NULL;
  if (stream != NULL && stream != Py_None) {
    const unsigned long long value = PyLong_AsUnsignedLongLongMask(stream);
    if (value == (unsigned long long)-1 && PyErr_Occurred()) return NULL;
    on = (void *)(size_t)value;
  }
  const void *program = self->program;
  int (*run)(const void *, void *) = self->run;
  PyObject *owner = self->owner;           /* stays while the call runs, whatever other threads do to self */
  Py_INCREF(owner);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = run(program, on);
  Py_END_ALLOW_THREADS
  Py_DECREF(owner);
  if (rc != 0) return PyObject_CallMethod((PyObject *)self, "_failed", "i", rc);
  Py_RETURN_NONE;
}

static PyMethodDef bound_methods[] = {{"_arm", (PyCFunction)bound_arm, METH_VARARGS, "what a call runs"}, {NULL, NULL, 0, NULL}};

static PyTypeObject BoundType = {
    PyVarObject_HEAD_INIT(NULL, 0)
    .tp_name = "paper_2407_13585_amd._bound_call.Bound",
    .tp_basicsize = sizeof(Bound),
    .tp_dealloc = (destructor)bound_dealloc,
    .tp_call = (ternaryfunc)bound_call,
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE,
    .tp_methods = bound_methods,
    .tp_init = bound_init,
    .tp_new = bound_new,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bound_call", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__bound_call(void) {
  PyObject *m;
  if (PyType_Ready(&BoundType) < 0) return NULL;
  m = PyModule_Create(&module);
  if (m == NULL) return NULL;
  Py_INCREF(&BoundType);
  if (PyModule_AddObject(m, "Bound", (PyObject *)&BoundType) < 0) {
    Py_DECREF(&BoundType);
    Py_DECREF(m);
    return NULL;
  }
  return m;
}
