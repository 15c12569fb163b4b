// Python extension module _tables: lists of radius tables to the flat int32 array of a mask descriptor.
// A walk over the list objects themselves: 30 tables of 10 x 10 integers take 7 us where list, chain
// and array in Python take 48.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

// radius_tables(rows, K) -> bytearray of int32 [H][K][K], or None where `rows` is anything but a list (tuple)
// of H > 0 lists of K lists of K integers that fit: the caller's general path takes those, and names the error.
static PyObject* radius_tables(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  if (n_args != 2) { PyErr_SetString(PyExc_TypeError, "radius_tables(rows, K)"); return nullptr; }
  const Py_ssize_t K = PyLong_AsSsize_t(args[1]);
  if (K == -1 && PyErr_Occurred()) return nullptr;
  auto is_seq = [](PyObject* o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); };
  PyObject* const rows = args[0];
  if (!is_seq(rows)) Py_RETURN_NONE;
  const Py_ssize_t H = PySequence_Fast_GET_SIZE(rows);
  if (H < 1 || K < 1 || K > 1024 || H > (1 << 20)) Py_RETURN_NONE;
  PyObject* const out = PyByteArray_FromStringAndSize(nullptr, H * K * K * (Py_ssize_t)sizeof(int32_t));
  if (!out) return nullptr;
  int32_t* p = (int32_t*)PyByteArray_AS_STRING(out);
  // (nothing below runs Python code, so the lists cannot change under the walk)
  for (Py_ssize_t h = 0; h < H; ++h) {
    PyObject* const table = PySequence_Fast_GET_ITEM(rows, h);
    if (!is_seq(table) || PySequence_Fast_GET_SIZE(table) != K) goto general;
    for (Py_ssize_t k = 0; k < K; ++k) {
      PyObject* const row = PySequence_Fast_GET_ITEM(table, k);
      if (!is_seq(row) || PySequence_Fast_GET_SIZE(row) != K) goto general;
      PyObject* const* const item = PySequence_Fast_ITEMS(row);
      for (Py_ssize_t j = 0; j < K; ++j) {
        if (!PyLong_CheckExact(item[j])) goto general;
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(item[j], &overflow);
        if (overflow || v < INT32_MIN || v > INT32_MAX) goto general;
        *p++ = (int32_t)v;
      }
    }
  }
  return out;
general:
  Py_DECREF(out);
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"radius_tables", (PyCFunction)(void (*)(void))radius_tables, METH_FASTCALL, "radius tables as int32 bytes, or None"},
    {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tables", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

PyMODINIT_FUNC PyInit__tables() { return PyModule_Create(&module); }
