// Conversion of Python lists for the ctypes binding (loaded with PyDLL: the GIL is held).
#include <Python.h>

#include <stdint.h>

// The n ints of `list` to `out`.  1, or 0 with no exception set where an element is not exactly an int, is
// out of range, or the list has another length: the caller then converts by Python's own means.
extern "C" int32_t oxy_ints_of_list(PyObject* list, int64_t* out, int64_t n) {
  if (!PyList_CheckExact(list) || PyList_GET_SIZE(list) != n) return 0;
  for (int64_t i = 0; i < n; ++i) {
    PyObject* o = PyList_GET_ITEM(list, i);
    if (!PyLong_CheckExact(o)) return 0;
    int overflow = 0;
    out[i] = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) return 0;
  }
  return 1;
}
