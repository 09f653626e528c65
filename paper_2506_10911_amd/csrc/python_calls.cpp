// The calls a training loop makes every step, for CPython: argument marshalling in C++ instead of
// ctypes.  The functions of libnoloco.so are handed over by address when the binding loads, so this
// module links against nothing.  A step of a small arena is bound by the host: through ctypes
// plan_groups took 6.2 us and outer_step 12.5 us, of which the C ABI itself takes 4.5.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <numpy/arrayobject.h>

#include <cstdint>
#include <cstring>

#include "noloco.h"

namespace {

decltype(&noloco_plan_groups) plan_groups_fn = nullptr;
decltype(&noloco_outer_step) outer_step_fn = nullptr;
decltype(&noloco_replica_spread) spread_fn = nullptr;
decltype(&noloco_replica_spread_noalloc) spread_noalloc_fn = nullptr;
PyObject* to_int32 = nullptr;      // callable: anything array-like -> contiguous int32 numpy array
PyObject* data_ptr_name = nullptr;

// Address of a device buffer: None, an integer, or an object with data_ptr().
bool address_of(PyObject* x, void** out) {
  if (x == Py_None) { *out = nullptr; return true; }
  PyObject* value = nullptr;
  if (PyLong_CheckExact(x)) {
    value = Py_NewRef(x);
  } else {
    PyObject* method = PyObject_GetAttr(x, data_ptr_name);
    if (method != nullptr) {
      value = PyObject_CallNoArgs(method);
      Py_DECREF(method);
      if (value != nullptr && !PyLong_CheckExact(value)) {      // whatever int() takes
        PyObject* made = PyNumber_Long(value);
        Py_DECREF(value);
        value = made;
      }
    } else if (PyErr_ExceptionMatches(PyExc_AttributeError)) {
      PyErr_Clear();
      value = PyNumber_Long(x);
    }
  }
  if (value == nullptr) return false;
  *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(value)));
  Py_DECREF(value);
  return !PyErr_Occurred();
}

// `values` as a contiguous int32 array, converted if it is anything else.  (numpy's own view: its buffer
// protocol builds a format string, 1 us each time.)
struct Int32Array {
  PyArrayObject* array = nullptr;
  ~Int32Array() { Py_XDECREF(array); }
  static bool fits(PyObject* x) {
    return PyArray_Check(x) && PyArray_TYPE(reinterpret_cast<PyArrayObject*>(x)) == NPY_INT32 &&
           PyArray_NDIM(reinterpret_cast<PyArrayObject*>(x)) > 0 && PyArray_ISCARRAY_RO(reinterpret_cast<PyArrayObject*>(x));
  }
  bool open(PyObject* values) {
    if (fits(values)) {
      array = reinterpret_cast<PyArrayObject*>(Py_NewRef(values));
      return true;
    }
    PyObject* made = PyObject_CallOneArg(to_int32, values);
    if (made == nullptr) return false;
    if (fits(made)) {
      array = reinterpret_cast<PyArrayObject*>(made);
      return true;
    }
    // ascontiguousarray() keeps an array that is contiguous at an odd address: it is copied to an aligned one
    array = reinterpret_cast<PyArrayObject*>(PyArray_FROMANY(made, NPY_INT32, 1, 0, NPY_ARRAY_IN_ARRAY));
    Py_DECREF(made);
    return array != nullptr;
  }
  int32_t* data() const { return static_cast<int32_t*>(PyArray_DATA(array)); }
  int32_t rows() const { return static_cast<int32_t>(PyArray_DIM(array, 0)); }
};

bool float_at(PyObject* seq, Py_ssize_t i, float* out) {
  PyObject* item = nullptr;
  if (PyTuple_CheckExact(seq) && i < PyTuple_GET_SIZE(seq)) {
    item = Py_NewRef(PyTuple_GET_ITEM(seq, i));
  } else if (PyObject* key = PyLong_FromSsize_t(i)) {
    item = PyObject_GetItem(seq, key);
    Py_DECREF(key);
  }
  if (item == nullptr) return false;
  PyObject* value = PyNumber_Float(item);
  Py_DECREF(item);
  if (value == nullptr) return false;
  *out = static_cast<float>(PyFloat_AS_DOUBLE(value));
  Py_DECREF(value);
  return true;
}

bool counted(Py_ssize_t got, Py_ssize_t want) {
  if (got == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, got);
  return false;
}

// plan_groups(seed, step, W, n, members, offsets): the last two are int32 arrays to fill
PyObject* plan_groups(PyObject*, PyObject* const* args, Py_ssize_t count) {
  if (!counted(count, 6)) return nullptr;
  const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[0]), step = PyLong_AsUnsignedLongLongMask(args[1]);
  const int32_t W = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(args[2]));
  const int32_t n = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(args[3]));
  if (PyErr_Occurred()) return nullptr;
  Int32Array members, offsets;
  if (!members.open(args[4]) || !offsets.open(args[5])) return nullptr;
  noloco_status status;
  Py_BEGIN_ALLOW_THREADS
  status = plan_groups_fn(seed, step, W, n, members.data(), offsets.data());
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// outer_step((plan, worker_stride, W, theta_dtype), phi, delta, theta, hparams, members, offsets, stream)
PyObject* outer_step(PyObject*, PyObject* const* args, Py_ssize_t count) {
  if (!counted(count, 8)) return nullptr;
  PyObject* layout = args[0];
  void *plan, *phi, *delta, *theta, *stream;
  if (!address_of(PyTuple_GET_ITEM(layout, 0), &plan) || !address_of(args[1], &phi) || !address_of(args[2], &delta) ||
      !address_of(args[3], &theta) || !address_of(args[7], &stream))
    return nullptr;
  noloco_arena arena;
  std::memset(&arena, 0, sizeof(arena));       // the step does not read the segments
  arena.phi = static_cast<float*>(phi);
  arena.delta = static_cast<float*>(delta);
  arena.theta = theta;
  arena.worker_stride = PyLong_AsLongLong(PyTuple_GET_ITEM(layout, 1));
  arena.W = static_cast<int32_t>(PyLong_AsLongLong(PyTuple_GET_ITEM(layout, 2)));
  arena.theta_dtype = static_cast<int32_t>(PyLong_AsLongLong(PyTuple_GET_ITEM(layout, 3)));
  noloco_hparams hp;
  if (PyErr_Occurred() || !float_at(args[4], 0, &hp.alpha) || !float_at(args[4], 1, &hp.beta) ||
      !float_at(args[4], 2, &hp.gamma))
    return nullptr;
  Int32Array members, offsets;
  if (!members.open(args[5]) || !offsets.open(args[6])) return nullptr;
  const int32_t groups = offsets.rows() - 1;
  noloco_status status;
  Py_BEGIN_ALLOW_THREADS
  status = outer_step_fn(static_cast<noloco_launch_plan*>(plan), &arena, &hp, members.data(), offsets.data(), groups, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyObject* spread(decltype(spread_fn) fn, PyObject* const* args, Py_ssize_t count) {
  if (!counted(count, 5)) return nullptr;
  void *plan, *x, *out, *stream;
  if (!address_of(PyTuple_GET_ITEM(args[0], 0), &plan) || !address_of(args[1], &x) || !address_of(args[3], &out) ||
      !address_of(args[4], &stream))
    return nullptr;
  const int32_t x_dtype = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(args[2]));
  if (PyErr_Occurred()) return nullptr;
  noloco_status status;
  Py_BEGIN_ALLOW_THREADS
  status = fn(static_cast<noloco_launch_plan*>(plan), x, x_dtype, static_cast<double*>(out), stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// replica_spread((plan, ...), x, x_dtype, out_std, stream)
PyObject* replica_spread(PyObject*, PyObject* const* args, Py_ssize_t count) { return spread(spread_fn, args, count); }
PyObject* replica_spread_noalloc(PyObject*, PyObject* const* args, Py_ssize_t count) {
  return spread(spread_noalloc_fn, args, count);
}

// bind(addresses of noloco_plan_groups, _outer_step, _replica_spread, _replica_spread_noalloc, to_int32)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t count) {
  if (!counted(count, 5)) return nullptr;
  void* fn[4];
  for (int i = 0; i < 4; ++i)
    if (!address_of(args[i], &fn[i])) return nullptr;
  plan_groups_fn = reinterpret_cast<decltype(plan_groups_fn)>(fn[0]);
  outer_step_fn = reinterpret_cast<decltype(outer_step_fn)>(fn[1]);
  spread_fn = reinterpret_cast<decltype(spread_fn)>(fn[2]);
  spread_noalloc_fn = reinterpret_cast<decltype(spread_noalloc_fn)>(fn[3]);
  Py_XDECREF(to_int32);
  to_int32 = Py_NewRef(args[4]);
  Py_RETURN_NONE;
}

template <typename F> PyCFunction fast(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"bind", fast(bind), METH_FASTCALL, nullptr},
    {"plan_groups", fast(plan_groups), METH_FASTCALL, nullptr},
    {"outer_step", fast(outer_step), METH_FASTCALL, nullptr},
    {"replica_spread", fast(replica_spread), METH_FASTCALL, nullptr},
    {"replica_spread_noalloc", fast(replica_spread_noalloc), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  import_array();
  data_ptr_name = PyUnicode_InternFromString("data_ptr");
  return data_ptr_name == nullptr ? nullptr : PyModule_Create(&module);
}
