// The part of the Python binding that runs on every call: argument checks on torch tensors, the
// current stream, and the call into the C ABI (include/pcgrl.h), without a Python frame, a ctypes
// conversion or a Python-level attribute lookup per argument.  A pcgrl_step from Python is bound by
// this path for every batch whose kernel takes less than it: 9 us a call when the same checks were
// made in Python and the call through ctypes (3 us of it the library and the launch), against a
// kernel of 4.5 us for 64 levels of 16x16.
//
// Only what is plainly right is handled here.  Anything else -- a wrong type, shape, device or
// layout, an argument that is missing, a tensor that torch itself refuses to look into (one without
// storage, say) -- makes the call return kLook, and the Python method then goes through the arguments
// one by one and says what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/pcgrl.h"

namespace {

constexpr long kLook = 1000;  // "look at the arguments": no library code is positive

struct Env {
  PyObject_HEAD pcgrl_ctx* ctx;
  int device;
  int64_t B, M, Hm, Wm;
  int64_t obs[4], onehot[4];  // the shape of an observation buffer, and of its one-hot cells
  int obs_dims;
};

// A tensor argument as a device pointer: contiguous, of this element type and on this device, with
// the `nd` sizes of `dims` behind `lead` leading ones (lead < 0: none, else the size of the one
// there is).
bool tensor(PyObject* o, const Env* e, c10::ScalarType type, int64_t lead, const int64_t* dims, int nd, void** out) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  const int extra = lead >= 0 ? 1 : 0;
  if (!t.is_cuda() || t.get_device() != e->device || t.scalar_type() != type || t.dim() != nd + extra) return false;
  if (extra && t.size(0) != lead) return false;
  for (int i = 0; i < nd; ++i)
    if (t.size(i + extra) != dims[i]) return false;
  if (!t.is_contiguous()) return false;
  *out = t.data_ptr();
  return true;
}
bool optional(PyObject* o, const Env* e, c10::ScalarType type, int64_t lead, const int64_t* dims, int nd, void** out) {
  *out = nullptr;
  return o == Py_None || tensor(o, e, type, lead, dims, nd, out);
}

void* stream_of(const Env* e) { return c10::hip::getCurrentHIPStream((c10::DeviceIndex)e->device).stream(); }

PyObject* look() { return PyLong_FromLong(kLook); }
template <typename F> PyObject* call(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// step(actions, obs, reward, done)
PyObject* env_step(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Env* e = reinterpret_cast<Env*>(self);
  void *act, *obs, *rew, *done;
  if (n != 4 || !e->ctx || !tensor(a[0], e, at::kInt, -1, &e->B, 1, &act) ||
      !optional(a[1], e, at::kByte, -1, e->obs, e->obs_dims, &obs) || !optional(a[2], e, at::kFloat, -1, &e->B, 1, &rew) ||
      !optional(a[3], e, at::kByte, -1, &e->B, 1, &done))
    return look();
  void* st = stream_of(e);
  return call([&] {
    return pcgrl_step(e->ctx, static_cast<const int32_t*>(act), static_cast<uint8_t*>(obs), static_cast<float*>(rew),
                      static_cast<uint8_t*>(done), st);
  });
}

// rollout(actions, obs, reward, done)
PyObject* env_rollout(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Env* e = reinterpret_cast<Env*>(self);
  if (n != 4 || !e->ctx || !THPVariable_Check(a[0]) || THPVariable_Unpack(a[0]).dim() != 2) return look();
  const int64_t T = THPVariable_Unpack(a[0]).size(0);
  int64_t slots = 1;
  if (a[1] != Py_None) {
    if (!THPVariable_Check(a[1]) || THPVariable_Unpack(a[1]).dim() != e->obs_dims + 1) return look();
    slots = THPVariable_Unpack(a[1]).size(0);
  }
  void *act, *obs, *rew, *done;
  if (T > (1 << 20) || slots > (1 << 20) || !tensor(a[0], e, at::kInt, T, &e->B, 1, &act) ||
      !optional(a[1], e, at::kByte, slots, e->obs, e->obs_dims, &obs) || !optional(a[2], e, at::kFloat, T, &e->B, 1, &rew) ||
      !optional(a[3], e, at::kByte, T, &e->B, 1, &done))
    return look();
  void* st = stream_of(e);
  return call([&] {
    return pcgrl_rollout(e->ctx, static_cast<const int32_t*>(act), (int32_t)T, static_cast<uint8_t*>(obs), (int32_t)slots,
                         static_cast<float*>(rew), static_cast<uint8_t*>(done), st);
  });
}

// reset(seed, obs): the seed as ctypes takes it, any Python integer modulo 2^64
PyObject* env_reset(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Env* e = reinterpret_cast<Env*>(self);
  void* obs;
  if (n != 2 || !e->ctx || !PyLong_Check(a[0]) || !optional(a[1], e, at::kByte, -1, e->obs, e->obs_dims, &obs)) return look();
  const unsigned long long seed = PyLong_AsUnsignedLongLongMask(a[0]);
  if (PyErr_Occurred()) return nullptr;
  void* st = stream_of(e);
  return call([&] { return pcgrl_reset(e->ctx, (uint64_t)seed, static_cast<uint8_t*>(obs), st); });
}

at::TensorOptions on_device(const Env* e, c10::ScalarType type) {
  return at::TensorOptions().dtype(type).device(at::Device(at::kCUDA, (c10::DeviceIndex)e->device));
}

// metrics(out) / exact_diameter(out) / observe(obs)
PyObject* env_metrics(PyObject* self, PyObject* o) {
  Env* e = reinterpret_cast<Env*>(self);
  const int64_t dims[2] = {e->B, e->M};
  void* out;
  if (!e->ctx || !tensor(o, e, at::kInt, -1, dims, 2, &out)) return look();
  void* st = stream_of(e);
  return call([&] { return pcgrl_metrics(e->ctx, static_cast<int32_t*>(out), st); });
}
PyObject* env_exact_diameter(PyObject* self, PyObject* o) {
  Env* e = reinterpret_cast<Env*>(self);
  void* out;
  if (!e->ctx || !tensor(o, e, at::kInt, -1, &e->B, 1, &out)) return look();
  void* st = stream_of(e);
  return call([&] { return pcgrl_exact_diameter(e->ctx, static_cast<int32_t*>(out), st); });
}
PyObject* env_observe(PyObject* self, PyObject* o) {
  Env* e = reinterpret_cast<Env*>(self);
  void* obs;
  if (!e->ctx || !tensor(o, e, at::kByte, -1, e->obs, e->obs_dims, &obs)) return look();
  void* st = stream_of(e);
  return call([&] { return pcgrl_observe(e->ctx, static_cast<uint8_t*>(obs), st); });
}

// unpack_obs(packed, out): the element type is that of `out`
PyObject* env_unpack_obs(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Env* e = reinterpret_cast<Env*>(self);
  void *packed, *out;
  if (n != 2 || !e->ctx || !tensor(a[0], e, at::kByte, -1, e->obs, e->obs_dims, &packed) || !THPVariable_Check(a[1])) return look();
  const c10::ScalarType type = THPVariable_Unpack(a[1]).scalar_type();
  const int code = type == at::kByte ? PCGRL_UNPACK_U8 : type == at::kHalf ? PCGRL_UNPACK_F16
                   : type == at::kBFloat16 ? PCGRL_UNPACK_BF16 : type == at::kFloat ? PCGRL_UNPACK_F32 : -1;
  if (code < 0 || !tensor(a[1], e, type, -1, e->onehot, 4, &out)) return look();
  void* st = stream_of(e);
  return call([&] { return pcgrl_unpack_obs(e->ctx, static_cast<const uint8_t*>(packed), out, code, st); });
}

// set_state(tiles, frozen, hw, pos)
PyObject* env_set_state(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  Env* e = reinterpret_cast<Env*>(self);
  const int64_t grid[3] = {e->B, e->Hm, e->Wm}, pair[2] = {e->B, 2};
  void *tiles, *frozen, *hw, *pos;
  if (n != 4 || !e->ctx || !tensor(a[0], e, at::kChar, -1, grid, 3, &tiles) ||
      !optional(a[1], e, at::kByte, -1, grid, 3, &frozen) || !tensor(a[2], e, at::kShort, -1, pair, 2, &hw) ||
      !tensor(a[3], e, at::kShort, -1, pair, 2, &pos))
    return look();
  void* st = stream_of(e);
  return call([&] {
    return pcgrl_set_state(e->ctx, static_cast<const int8_t*>(tiles), static_cast<const uint8_t*>(frozen),
                           static_cast<const int16_t*>(hw), static_cast<const int16_t*>(pos), st);
  });
}

// get_state() -> (rc, tiles, frozen, hw, pos, counters), new tensors
PyObject* env_get_state(PyObject* self, PyObject*) {
  Env* e = reinterpret_cast<Env*>(self);
  if (!e->ctx) return look();
  HANDLE_TH_ERRORS
  at::Tensor tiles = at::empty({e->B, e->Hm, e->Wm}, on_device(e, at::kChar));
  at::Tensor frozen = at::empty({e->B, e->Hm, e->Wm}, on_device(e, at::kByte));
  at::Tensor hw = at::empty({e->B, 2}, on_device(e, at::kShort));
  at::Tensor pos = at::empty({e->B, 2}, on_device(e, at::kShort));
  at::Tensor counters = at::empty({e->B, 3}, on_device(e, at::kInt));
  void* st = stream_of(e);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = pcgrl_get_state(e->ctx, static_cast<int8_t*>(tiles.data_ptr()), static_cast<uint8_t*>(frozen.data_ptr()),
                       static_cast<int16_t*>(hw.data_ptr()), static_cast<int16_t*>(pos.data_ptr()),
                       static_cast<int32_t*>(counters.data_ptr()), st);
  Py_END_ALLOW_THREADS
  return Py_BuildValue("(iNNNNN)", rc, THPVariable_Wrap(tiles), THPVariable_Wrap(frozen), THPVariable_Wrap(hw),
                       THPVariable_Wrap(pos), THPVariable_Wrap(counters));
  END_HANDLE_TH_ERRORS
}

PyObject* env_close(PyObject* self, PyObject*) {
  reinterpret_cast<Env*>(self)->ctx = nullptr;
  Py_RETURN_NONE;
}

// Env(ctx, device, M, max_h, max_w, obs_shape, onehot_shape)
PyObject* env_new(PyTypeObject* type, PyObject* args, PyObject*) {
  unsigned long long ctx;
  int device;
  long long M, Hm, Wm, h[4];
  PyObject* shape;
  if (!PyArg_ParseTuple(args, "KiLLLO!(LLLL)", &ctx, &device, &M, &Hm, &Wm, &PyTuple_Type, &shape, &h[0], &h[1], &h[2], &h[3]))
    return nullptr;
  const Py_ssize_t nd = PyTuple_Size(shape);
  if (nd < 1 || nd > 4) {
    PyErr_SetString(PyExc_ValueError, "an observation buffer has one to four dimensions");
    return nullptr;
  }
  Env* e = reinterpret_cast<Env*>(type->tp_alloc(type, 0));
  if (!e) return nullptr;
  e->ctx = reinterpret_cast<pcgrl_ctx*>((uintptr_t)ctx);
  e->device = device;
  e->M = M;
  e->Hm = Hm;
  e->Wm = Wm;
  e->obs_dims = (int)nd;
  for (int i = 0; i < 4; ++i) e->onehot[i] = h[i];
  for (Py_ssize_t i = 0; i < nd; ++i) e->obs[i] = PyLong_AsLongLong(PyTuple_GetItem(shape, i));
  e->B = e->obs[0];
  if (PyErr_Occurred()) {
    Py_DECREF(e);
    return nullptr;
  }
  return reinterpret_cast<PyObject*>(e);
}

// The tensor accessors and the stream lookup throw, and no C++ exception may reach the interpreter's
// frames: the process would end.  The Python checks make the same accesses and raise what torch says.
// (Nothing throws while the interpreter lock is released: the library's C entry points do not.)
template <auto F, typename... A> PyObject* guarded(PyObject* self, A... args) noexcept {
  try {
    return F(self, args...);
  } catch (...) {
    PyErr_Clear();  // (a tensor type written in Python leaves its exception behind)
    return look();
  }
}

template <auto F> PyCFunction one() { return guarded<F, PyObject*>; }
template <auto F> PyCFunction fast() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<F, PyObject* const*, Py_ssize_t>));
}
PyMethodDef env_methods[] = {
    {"step", fast<env_step>(), METH_FASTCALL, nullptr}, {"rollout", fast<env_rollout>(), METH_FASTCALL, nullptr},
    {"reset", fast<env_reset>(), METH_FASTCALL, nullptr}, {"unpack_obs", fast<env_unpack_obs>(), METH_FASTCALL, nullptr},
    {"set_state", fast<env_set_state>(), METH_FASTCALL, nullptr},
    {"metrics", one<env_metrics>(), METH_O, nullptr}, {"exact_diameter", one<env_exact_diameter>(), METH_O, nullptr},
    {"observe", one<env_observe>(), METH_O, nullptr}, {"get_state", env_get_state, METH_NOARGS, nullptr},
    {"close", env_close, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr},
};

PyTypeObject EnvType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "pcgrl_py", "Call path of the Python binding.", -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_pcgrl_py() {
  EnvType.tp_name = "pcgrl_py.Env";
  EnvType.tp_basicsize = sizeof(Env);
  EnvType.tp_flags = Py_TPFLAGS_DEFAULT;
  EnvType.tp_new = env_new;
  EnvType.tp_methods = env_methods;
  if (PyType_Ready(&EnvType) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&EnvType);
  if (PyModule_AddObject(m, "Env", reinterpret_cast<PyObject*>(&EnvType)) < 0 || PyModule_AddIntConstant(m, "LOOK", kLook) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
