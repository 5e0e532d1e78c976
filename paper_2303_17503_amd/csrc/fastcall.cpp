// fastcall.cpp -- the argument checks of the calls that programs make once per ply, in native code.
//
// With small batches a ply takes the GPU 4 to 6 us, and the Python checks of the up to seven tensors of a call (dtype, device,
// contiguity, shape, pointer: 0.4 us each) took longer than that.  Each function here checks the tensors of one call exactly as
// binding.py does and calls the library's C entry point, whose address it is given; it returns the entry point's code, or None when
// anything is not as it has to be, and then the Python path runs and raises its error.  Nothing is kept between calls.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

// pointer of a contiguous cuda tensor of the given type and shape; false: not such a tensor (or one of a subclass)
bool take(PyObject* o, at::ScalarType type, int64_t d0, int64_t d1, void** out) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  const int64_t dim = d1 < 0 ? 1 : 2;
  if (t.scalar_type() != type || !t.is_cuda() || t.dim() != dim || t.size(0) != d0 || (dim == 2 && t.size(1) != d1) || !t.is_contiguous()) return false;
  *out = t.data_ptr();
  return true;
}
// the same, None gives a null pointer
bool take_or_null(PyObject* o, at::ScalarType type, int64_t d0, int64_t d1, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  return take(o, type, d0, d1, out);
}

template <class F>
PyObject* guarded(F&& f) {   // f: prepares and calls; returns -1000 when the Python path has to look at the call
  int rc = -1000;
  try {
    rc = f();
  } catch (...) {
    rc = -1000;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  if (rc == -1000) Py_RETURN_NONE;
  return PyLong_FromLong(rc);
}
template <class F>
int without_gil(F&& f) {   // launching can wait for room in the queue
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}
void* pointer(PyObject* o) { return PyLong_AsVoidPtr(o); }
uint32_t u32(PyObject* o) { return (uint32_t)PyLong_AsUnsignedLongLong(o); }

constexpr auto kInt = at::kInt;
constexpr auto kByte = at::kByte;
constexpr auto kFloat = at::kFloat;

// (address, handle, batch, actions)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&] {
    void* actions;
    if (n != 4) return -1000;
    void *fn = pointer(a[0]), *h = pointer(a[1]);
    const int64_t B = PyLong_AsLongLong(a[2]);
    if (PyErr_Occurred() || !take(a[3], kInt, B, -1, &actions)) return -1000;
    return without_gil([&] { return ((int (*)(void*, const int32_t*))fn)(h, (const int32_t*)actions); });
  });
}

// (address, handle, batch, actions, seed, t, start_t, out)
PyObject* step_sample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&] {
    void *actions, *start, *out;
    if (n != 8) return -1000;
    void *fn = pointer(a[0]), *h = pointer(a[1]);
    const int64_t B = PyLong_AsLongLong(a[2]);
    const uint32_t seed = u32(a[4]), t = u32(a[5]);
    if (PyErr_Occurred() || !take(a[3], kInt, B, -1, &actions) || !take_or_null(a[6], kInt, B, -1, &start) || !take(a[7], kInt, B, -1, &out)) return -1000;
    return without_gil([&] {
      return ((int (*)(void*, const int32_t*, uint32_t, uint32_t, const int32_t*, int32_t*))fn)(h, (const int32_t*)actions, seed, t, (const int32_t*)start,
                                                                                               (int32_t*)out);
    });
  });
}

// (address, handle, batch, seed, t, start_t, out)
PyObject* random_actions(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&] {
    void *start, *out;
    if (n != 7) return -1000;
    void *fn = pointer(a[0]), *h = pointer(a[1]);
    const int64_t B = PyLong_AsLongLong(a[2]);
    const uint32_t seed = u32(a[3]), t = u32(a[4]);
    if (PyErr_Occurred() || !take_or_null(a[5], kInt, B, -1, &start) || !take(a[6], kInt, B, -1, &out)) return -1000;
    return without_gil([&] { return ((int (*)(void*, uint32_t, uint32_t, const int32_t*, int32_t*))fn)(h, seed, t, (const int32_t*)start, (int32_t*)out); });
  });
}

// (address, handle, mask_pitch, obs_pitch, src, actions, dst, mask, obs, rewards, terminated)
PyObject* step_slots(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&] {
    void *src, *actions, *dst, *mask, *obs, *rew, *term;
    if (n != 11 || !THPVariable_CheckExact(a[4])) return -1000;
    void *fn = pointer(a[0]), *h = pointer(a[1]);
    const int64_t mask_pitch = PyLong_AsLongLong(a[2]), obs_pitch = PyLong_AsLongLong(a[3]);
    const at::Tensor& s = THPVariable_Unpack(a[4]);
    if (PyErr_Occurred() || s.dim() != 1 || s.size(0) > INT32_MAX) return -1000;
    const int64_t N = s.size(0);
    if (!take(a[4], kInt, N, -1, &src) || !take_or_null(a[5], kInt, N, -1, &actions) || !take(a[6], kInt, N, -1, &dst) ||
        !take_or_null(a[7], kByte, N, mask_pitch, &mask) || !take_or_null(a[8], kByte, N, obs_pitch, &obs) || !take_or_null(a[9], kFloat, N, 2, &rew) ||
        !take_or_null(a[10], kByte, N, -1, &term))
      return -1000;
    return without_gil([&] {
      return ((int (*)(void*, int32_t, const int32_t*, const int32_t*, const int32_t*, uint8_t*, uint8_t*, float*, uint8_t*))fn)(
          h, (int32_t)N, (const int32_t*)src, (const int32_t*)actions, (const int32_t*)dst, (uint8_t*)mask, (uint8_t*)obs, (float*)rew, (uint8_t*)term);
    });
  });
}

PyMethodDef kMethods[] = {
    {"step", (PyCFunction)(void*)step, METH_FASTCALL, nullptr},
    {"step_sample", (PyCFunction)(void*)step_sample, METH_FASTCALL, nullptr},
    {"random_actions", (PyCFunction)(void*)random_actions, METH_FASTCALL, nullptr},
    {"step_slots", (PyCFunction)(void*)step_slots, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__fastcall() { return PyModule_Create(&kModule); }
