// _mccall: calls a function of libmooncake_hip.so with the arguments of a Python wrapper (binding.py), laid out here instead of
// through ctypes.  Small calls are bound by the host: an attention call of the tiny fp32 request was 7.3 us of it, now 4.9, 4 of
// them in the library.  Marshalling only; the library itself is loaded by binding.py, which hands the address over.
//
//   call(address, kinds, *arguments) -> status        one letter of `kinds` per argument:
//     p  device (or pinned) tensor: its data_ptr(); None: a null pointer
//     s  a ctypes structure: its address; None: a null pointer
//     i  an integer (32 or 64 bits; the function takes the bits it has parameters for, as with ctypes)
//     I  a list of n integers as int32[n], or an integer address
//     Q  a list of n integers as int64[n], or an integer address
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include <vector>

#if !defined(__x86_64__)
#error "Function below rests on the x86-64 System V calling convention"
#endif

namespace {

constexpr int kMaxArgs = 20;
// every parameter is an integer or a pointer, so one signature does: registers and stack words the callee has no parameter for
// are not looked at (x86-64 calling convention, the caller clears the stack)
typedef int (*Function)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t,
                        uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t);

PyObject* g_data_ptr = nullptr;                            // "data_ptr"

// low 64 bits of an integer; false with an exception set for what is none
bool bits_of(PyObject* o, uint64_t* out) {
  if (!PyLong_Check(o)) {
    PyObject* index = PyNumber_Index(o);
    if (index == nullptr) return false;
    *out = PyLong_AsUnsignedLongLongMask(index);
    Py_DECREF(index);
  } else {
    *out = PyLong_AsUnsignedLongLongMask(o);
  }
  return !(*out == (uint64_t)-1 && PyErr_Occurred());
}

template <typename Int>
bool lay_out(PyObject* list, std::vector<uint64_t>& room) {
  const Py_ssize_t n = PyList_GET_SIZE(list);
  room.resize((size_t)n * sizeof(Int) / 8 + 1);
  Int* to = reinterpret_cast<Int*>(room.data());
  for (Py_ssize_t i = 0; i < n && i < PyList_GET_SIZE(list); ++i) {
    PyObject* item = PyList_GET_ITEM(list, i);
    uint64_t v;
    if (PyLong_Check(item)) {
      if (!bits_of(item, &v)) return false;
    } else {                                               // as int() takes it: numpy integers, floats
      Py_INCREF(item);
      PyObject* whole = PyNumber_Long(item);
      Py_DECREF(item);
      if (whole == nullptr) return false;
      const bool fine = bits_of(whole, &v);
      Py_DECREF(whole);
      if (!fine) return false;
    }
    to[i] = (Int)v;
  }
  return true;
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  if (n_args < 2 || !PyUnicode_Check(args[1])) {
    PyErr_SetString(PyExc_TypeError, "call(address, kinds, *arguments)");
    return nullptr;
  }
  Py_ssize_t n = 0;
  const char* kinds = PyUnicode_AsUTF8AndSize(args[1], &n);
  uint64_t address = 0;
  if (kinds == nullptr || !bits_of(args[0], &address)) return nullptr;
  if (n != n_args - 2 || n > kMaxArgs || address == 0) {
    PyErr_SetString(PyExc_TypeError, "one letter of kinds per argument, at most 20");
    return nullptr;
  }
  uint64_t a[kMaxArgs] = {0};
  std::vector<uint64_t> lists[2];
  int n_lists = 0;
  try {
    for (Py_ssize_t i = 0; i < n; ++i) {
      PyObject* o = args[i + 2];
      if (kinds[i] == 'p') {
        if (o == Py_None) continue;
        PyObject* ptr = PyObject_CallMethodNoArgs(o, g_data_ptr);
        if (ptr == nullptr) return nullptr;
        const bool fine = bits_of(ptr, &a[i]);
        Py_DECREF(ptr);
        if (!fine) return nullptr;
      } else if (kinds[i] == 's') {
        if (o == Py_None) continue;
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return nullptr;
        a[i] = reinterpret_cast<uint64_t>(view.buf);       // (the caller holds the object, which owns the memory)
        PyBuffer_Release(&view);
      } else if ((kinds[i] == 'I' || kinds[i] == 'Q') && PyList_CheckExact(o)) {
        if (n_lists == 2) {
          PyErr_SetString(PyExc_TypeError, "at most two lists");
          return nullptr;
        }
        std::vector<uint64_t>& room = lists[n_lists++];
        if (!(kinds[i] == 'I' ? lay_out<int32_t>(o, room) : lay_out<int64_t>(o, room))) return nullptr;
        a[i] = reinterpret_cast<uint64_t>(room.data());
      } else if (!bits_of(o, &a[i])) {
        return nullptr;
      }
    }
  } catch (const std::exception&) {                        // no memory for a list
    return PyErr_NoMemory();
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = reinterpret_cast<Function>(address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12],
                                               a[13], a[14], a[15], a[16], a[17], a[18], a[19]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyMethodDef g_methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call(address, kinds, *arguments) -> status"},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_mccall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mccall(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr == nullptr ? nullptr : PyModule_Create(&g_module);
}
