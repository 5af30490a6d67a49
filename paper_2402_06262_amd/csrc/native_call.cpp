// Argument marshalling of the step and prompt entry points for the Python binding, without a Python-level call per tensor: a
// small step takes less time on the GPU than its fourteen data_ptr() and is_contiguous() calls, the stream lookup and the
// ctypes conversion of seventeen arguments took on the host.
//
// The library's functions are handed over by address (`bind`): which libroco.so is in use stays the business of binding.py.
// What the arguments may be does not change: tensors (contiguous, else ValueError), plain addresses, None where NULL is
// allowed, objects that binding.py's own conversion knows; a size or None, a stream, an address or None.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>

#include "../../include/roco.h"

namespace {

// ------------------------------------------------------------------ what binding.py hands over once
PyObject* g_tensor_types[2];  // torch.Tensor, torch.nn.Parameter: exactly these are read without a call
PyObject* g_params_type;      // binding.RocoParams
PyObject* g_pointer;          // binding._ptr: everything else
PyObject* g_current_stream;   // binding._stream: anything but an address, and the current stream before it is known how to ask
PyObject* g_raw_stream;       // torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice: set once the GPU is in use
PyObject* g_device;

struct Functions {
  decltype(&roco_prefill_compress) prefill;
  decltype(&roco_prefill_compress_gqa) prefill_gqa;
  decltype(&roco_prefill_compress_lse) prefill_lse;
  decltype(&roco_decode_step) decode;
  decltype(&roco_decode_step_static) decode_static;
  decltype(&roco_encode_block) block;
  decltype(&roco_encode_block_gqa) block_gqa;
  decltype(&roco_decode_step_gqa) decode_gqa;
} g_fn;

// ------------------------------------------------------------------ arguments
struct Failed {};  // a Python exception is set

const at::Tensor* tensor_of(PyObject* o) {
  PyObject* const type = reinterpret_cast<PyObject*>(Py_TYPE(o));
  return type == g_tensor_types[0] || type == g_tensor_types[1] ? &THPVariable_Unpack(o) : nullptr;
}

void* address_of_int(PyObject* o) { return reinterpret_cast<void*>(PyLong_AsUnsignedLongLongMask(o)); }

void* pointer(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (const at::Tensor* t = tensor_of(o)) {
    if (!t->is_contiguous()) {
      PyErr_SetString(PyExc_ValueError, "roco: tensors must be contiguous");
      throw Failed{};
    }
    return t->data_ptr();
  }
  if (PyLong_Check(o)) return address_of_int(o);
  PyObject* const r = PyObject_CallOneArg(g_pointer, o);
  if (r == nullptr) throw Failed{};
  void* p = nullptr;
  if (r != Py_None) {
    p = PyLong_AsVoidPtr(r);
    if (p == nullptr && PyErr_Occurred()) {
      Py_DECREF(r);
      throw Failed{};
    }
  }
  Py_DECREF(r);
  return p;
}

// The low 64 bits, as ctypes takes them: sizes from 2^63 on are sizes.
unsigned long long integer(PyObject* o) {
  if (PyLong_CheckExact(o)) return PyLong_AsUnsignedLongLongMask(o);
  PyObject* const n = PyNumber_Long(o);  // as int(o)
  if (n == nullptr) throw Failed{};
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return v;
}
int32_t int32_of(PyObject* o) { return static_cast<int32_t>(integer(o)); }

size_t bytes(PyObject* size, PyObject* workspace) {
  if (size != Py_None) return static_cast<size_t>(integer(size));
  if (const at::Tensor* t = tensor_of(workspace)) return t->nbytes();
  PyObject* const n = PyObject_GetAttrString(workspace, "nbytes");
  if (n == nullptr) throw Failed{};
  size_t v;
  try {
    v = static_cast<size_t>(integer(n));
  } catch (const Failed&) {
    Py_DECREF(n);
    throw;
  }
  Py_DECREF(n);
  return v;
}

void* stream_of(PyObject* o) {
  PyObject* r;
  if (o == Py_None && g_raw_stream != nullptr) {
    PyObject* const device = PyObject_CallNoArgs(g_device);
    if (device == nullptr) throw Failed{};
    r = PyObject_CallOneArg(g_raw_stream, device);
    Py_DECREF(device);
  } else if (PyLong_Check(o)) {
    return address_of_int(o);
  } else {
    r = PyObject_CallOneArg(g_current_stream, o);
  }
  if (r == nullptr) throw Failed{};
  void* const s = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  if (s == nullptr && PyErr_Occurred()) throw Failed{};
  return s;
}

// The parameters' structure, a ctypes object of binding.py's class (or one derived from it), read through the buffer it exports and
// copied: its first 44 bytes.
roco_params params_of(PyObject* o) {
  roco_params p;
  Py_buffer view;
  if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(g_params_type))) {
    PyErr_SetString(PyExc_TypeError, "roco: params must be a RocoParams");
    throw Failed{};
  }
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Failed{};
  std::memcpy(&p, view.buf, sizeof(p));  // (a derived structure has its own fields behind)
  PyBuffer_Release(&view);
  return p;
}

template <class Call> PyObject* guarded(Py_ssize_t n, Py_ssize_t expected, Call call) {
  if (n != expected) {
    PyErr_Format(PyExc_TypeError, "roco: %zd arguments expected, got %zd", expected, n);
    return nullptr;
  }
  try {
    return PyLong_FromLong(call());
  } catch (const Failed&) {
    return nullptr;
  } catch (const std::exception& e) {  // a tensor without memory (fake, vmapped, sparse)
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
struct NoGil {  // the launches may wait for room in the queue
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

// ------------------------------------------------------------------ entry points: the arguments of binding.py's functions in order
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 17, [&] {
    const roco_params p = params_of(a[0]);
    void* t[14];
    for (int i = 0; i < 14; ++i) t[i] = pointer(a[1 + i]);
    const size_t ws = bytes(a[15], a[14]);
    void* const s = stream_of(a[16]);
    NoGil g;
    return g_fn.decode(&p, t[0], t[1], t[2], static_cast<int32_t*>(t[3]), t[4], t[5], static_cast<float*>(t[6]),
                       static_cast<int32_t*>(t[7]), static_cast<int32_t*>(t[8]), static_cast<int32_t*>(t[9]), t[10],
                       static_cast<int32_t*>(t[11]), static_cast<int32_t*>(t[12]), t[13], ws, s);
  });
}
PyObject* decode_step_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 15, [&] {
    const roco_params p = params_of(a[0]);
    void* t[13];
    for (int i = 0; i < 13; ++i) t[i] = pointer(a[1 + i]);
    void* const s = stream_of(a[14]);
    NoGil g;
    return g_fn.decode_static(&p, t[0], t[1], t[2], static_cast<int32_t*>(t[3]), t[4], t[5], static_cast<float*>(t[6]),
                              static_cast<int32_t*>(t[7]), static_cast<int32_t*>(t[8]), static_cast<int32_t*>(t[9]), t[10],
                              static_cast<int32_t*>(t[11]), static_cast<int32_t*>(t[12]), s);
  });
}
// (params, integer, 14 pointers, workspace_bytes, stream): a block of tokens, or one token of a group of heads
template <class Fn> PyObject* step_of_many(Fn Functions::*fn, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 18, [&] {
    const roco_params p = params_of(a[0]);
    const int32_t count = int32_of(a[1]);
    void* t[14];
    for (int i = 0; i < 14; ++i) t[i] = pointer(a[2 + i]);
    const size_t ws = bytes(a[16], a[15]);
    void* const s = stream_of(a[17]);
    NoGil g;
    return (g_fn.*fn)(&p, count, t[0], t[1], t[2], static_cast<int32_t*>(t[3]), t[4], t[5], static_cast<float*>(t[6]),
                      static_cast<int32_t*>(t[7]), static_cast<int32_t*>(t[8]), static_cast<int32_t*>(t[9]), t[10],
                      static_cast<int32_t*>(t[11]), static_cast<int32_t*>(t[12]), t[13], ws, s);
  });
}
PyObject* encode_block(PyObject*, PyObject* const* a, Py_ssize_t n) { return step_of_many(&Functions::block, a, n); }
PyObject* decode_step_gqa(PyObject*, PyObject* const* a, Py_ssize_t n) { return step_of_many(&Functions::decode_gqa, a, n); }
PyObject* encode_block_gqa(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 19, [&] {
    const roco_params p = params_of(a[0]);
    const int32_t block = int32_of(a[1]), group = int32_of(a[2]);
    void* t[14];
    for (int i = 0; i < 14; ++i) t[i] = pointer(a[3 + i]);
    const size_t ws = bytes(a[17], a[16]);
    void* const s = stream_of(a[18]);
    NoGil g;
    return g_fn.block_gqa(&p, block, group, t[0], t[1], t[2], static_cast<int32_t*>(t[3]), t[4], t[5], static_cast<float*>(t[6]),
                          static_cast<int32_t*>(t[7]), static_cast<int32_t*>(t[8]), static_cast<int32_t*>(t[9]), t[10],
                          static_cast<int32_t*>(t[11]), static_cast<int32_t*>(t[12]), t[13], ws, s);
  });
}
PyObject* prefill_compress(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 16, [&] {
    const roco_params p = params_of(a[0]);
    void *in[4], *t[8];
    for (int i = 0; i < 4; ++i) in[i] = pointer(a[1 + i]);
    const int32_t L_max = int32_of(a[5]);
    for (int i = 0; i < 8; ++i) t[i] = pointer(a[6 + i]);
    const size_t ws = bytes(a[14], a[13]);
    void* const s = stream_of(a[15]);
    NoGil g;
    return g_fn.prefill(&p, in[0], in[1], in[2], static_cast<int32_t*>(in[3]), L_max, t[0], t[1], static_cast<float*>(t[2]),
                        static_cast<int32_t*>(t[3]), static_cast<int32_t*>(t[4]), static_cast<int32_t*>(t[5]), t[6], t[7], ws, s);
  });
}
PyObject* prefill_compress_gqa(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 17, [&] {
    const roco_params p = params_of(a[0]);
    const int32_t group = int32_of(a[1]);
    void *in[4], *t[8];
    for (int i = 0; i < 4; ++i) in[i] = pointer(a[2 + i]);
    const int32_t L_max = int32_of(a[6]);
    for (int i = 0; i < 8; ++i) t[i] = pointer(a[7 + i]);
    const size_t ws = bytes(a[15], a[14]);
    void* const s = stream_of(a[16]);
    NoGil g;
    return g_fn.prefill_gqa(&p, group, in[0], in[1], in[2], static_cast<int32_t*>(in[3]), L_max, t[0], t[1],
                            static_cast<float*>(t[2]), static_cast<int32_t*>(t[3]), static_cast<int32_t*>(t[4]),
                            static_cast<int32_t*>(t[5]), t[6], t[7], ws, s);
  });
}
PyObject* prefill_compress_lse(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 17, [&] {
    const roco_params p = params_of(a[0]);
    const int32_t group = int32_of(a[1]);
    void *in[4], *t[8];
    for (int i = 0; i < 4; ++i) in[i] = pointer(a[2 + i]);
    const int32_t L_max = int32_of(a[6]);
    for (int i = 0; i < 8; ++i) t[i] = pointer(a[7 + i]);
    const size_t ws = bytes(a[15], a[14]);
    void* const s = stream_of(a[16]);
    NoGil g;
    return g_fn.prefill_lse(&p, group, in[0], in[1], in[2], static_cast<int32_t*>(in[3]), L_max, static_cast<float*>(t[0]), t[1],
                            t[2], static_cast<float*>(t[3]), static_cast<int32_t*>(t[4]), static_cast<int32_t*>(t[5]),
                            static_cast<int32_t*>(t[6]), t[7], ws, s);
  });
}

// bind(addresses, tensor, parameter, RocoParams, _ptr, _stream); use_gpu(getCurrentRawStream, getDevice)
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[8];
  PyObject *tensor, *parameter, *params, *ptr, *stream;
  if (!PyArg_ParseTuple(args, "(KKKKKKKK)OOO!OO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &f[6], &f[7], &tensor, &parameter,
                        &PyType_Type, &params, &ptr, &stream))
    return nullptr;
  g_fn.prefill = reinterpret_cast<decltype(g_fn.prefill)>(f[0]);
  g_fn.prefill_gqa = reinterpret_cast<decltype(g_fn.prefill_gqa)>(f[1]);
  g_fn.prefill_lse = reinterpret_cast<decltype(g_fn.prefill_lse)>(f[2]);
  g_fn.decode = reinterpret_cast<decltype(g_fn.decode)>(f[3]);
  g_fn.decode_static = reinterpret_cast<decltype(g_fn.decode_static)>(f[4]);
  g_fn.block = reinterpret_cast<decltype(g_fn.block)>(f[5]);
  g_fn.block_gqa = reinterpret_cast<decltype(g_fn.block_gqa)>(f[6]);
  g_fn.decode_gqa = reinterpret_cast<decltype(g_fn.decode_gqa)>(f[7]);
  Py_INCREF(tensor); Py_INCREF(parameter); Py_INCREF(params); Py_INCREF(ptr); Py_INCREF(stream);
  Py_XSETREF(g_tensor_types[0], tensor);
  Py_XSETREF(g_tensor_types[1], parameter);
  Py_XSETREF(g_params_type, params);
  Py_XSETREF(g_pointer, ptr);
  Py_XSETREF(g_current_stream, stream);
  Py_RETURN_NONE;
}
PyObject* use_gpu(PyObject*, PyObject* args) {
  PyObject *raw, *device;
  if (!PyArg_ParseTuple(args, "OO", &raw, &device)) return nullptr;
  Py_INCREF(raw); Py_INCREF(device);
  Py_XSETREF(g_device, device);
  Py_XSETREF(g_raw_stream, raw);
  Py_RETURN_NONE;
}

PyObject* forget_gpu(PyObject*, PyObject*) {  // in a forked child
  Py_CLEAR(g_raw_stream);
  Py_CLEAR(g_device);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST(decode_step), FAST(decode_step_static), FAST(decode_step_gqa), FAST(encode_block), FAST(encode_block_gqa),
    FAST(prefill_compress), FAST(prefill_compress_gqa), FAST(prefill_compress_lse),
    {"bind", bind, METH_VARARGS, nullptr}, {"use_gpu", use_gpu, METH_VARARGS, nullptr},
    {"forget_gpu", forget_gpu, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
#undef FAST
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
