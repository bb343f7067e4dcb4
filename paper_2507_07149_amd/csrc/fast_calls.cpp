// The calls of a training step's inner loop from Python, in one native step each: argument checks, pointers, the current stream
// and the call.  Through ctypes and the checks in Python a call cost 5.8 us, most of it not the runtime's launch: quantize and
// dequantize of 262 K binary32 elements, whose kernels take 3.4 us each, 11.6 us, now 7.9; a weight gradient of one small tile 6.8 -> 5.4.
//
// Every function takes the arguments of the entry point of its name and returns its status, or None without having done anything where
// an argument is not what the usual call has: then the caller goes on with the general checks, which either raise or make the call.
// Usual are plain tensors (no subclasses, no wrappers of a tracer or of vmap) on a device, contiguous, of the right type and large enough.
#define PY_SSIZE_T_CLEAN
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "daf.h"

namespace {

struct Library {
  decltype(&daf_quantize_pack) quantize_pack;
  decltype(&daf_quantize_pack_static) quantize_pack_static;
  decltype(&daf_unpack_dequantize) unpack_dequantize;
  decltype(&daf_quantize_pack_metrics) quantize_pack_metrics;
  decltype(&daf_relu_quantize_pack) relu_quantize_pack;
  decltype(&daf_unpack_relu_backward) unpack_relu_backward;
  decltype(&daf_group_minmax) group_minmax;
  decltype(&daf_select_bits) select_bits;
  decltype(&daf_select_bits_from_scale) select_bits_from_scale;
  decltype(&daf_select_bits_workspace_bytes) select_bits_workspace_bytes;
  decltype(&daf_plan_update) plan_update;
  decltype(&daf_linear_quantize_pack) linear_quantize_pack;
  decltype(&daf_unpack_matmul_grad_weight) unpack_matmul_grad_weight;
  decltype(&daf_unpack_matmul_workspace_bytes) unpack_matmul_workspace_bytes;
  decltype(&daf_plan_num_elements) plan_num_elements;
  decltype(&daf_plan_num_groups) plan_num_groups;
  decltype(&daf_plan_packed_words) plan_packed_words;
} lib;
PyObject* plan_type = nullptr;
PyObject* handle_name = nullptr;
PyObject* stream_name = nullptr;

// What one call's arguments amount to; `ok` stays true as long as all of them are usual.
struct Call {
  bool ok = true;
  daf_plan_t* plan = nullptr;
  int64_t elements = 0, groups = 0;
  void* stream = nullptr;

  void with_plan(PyObject* o) {
    if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != plan_type) { ok = false; return; }
    PyObject* h = PyObject_GetAttr(o, handle_name);
    plan = h != nullptr && PyLong_CheckExact(h) ? static_cast<daf_plan_t*>(PyLong_AsVoidPtr(h)) : nullptr;
    Py_XDECREF(h);
    if (PyErr_Occurred()) PyErr_Clear();
    if (plan == nullptr) { ok = false; return; }
    elements = lib.plan_num_elements(plan);
    groups = lib.plan_num_groups(plan);
  }
  void with_stream(PyObject* o) {
    if (!ok) return;
    if (o == Py_None) {
      stream = c10::hip::getCurrentHIPStream().stream();
      return;
    }
    PyObject* h = PyObject_GetAttr(o, stream_name);
    if (h == nullptr || !PyLong_CheckExact(h)) ok = false;
    else stream = PyLong_AsVoidPtr(h);
    Py_XDECREF(h);
    if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
  }
  const at::Tensor* tensor(PyObject* o) {
    if (!ok) return nullptr;
    if (THPVariable_CheckExact(o)) {
      const at::Tensor& t = THPVariable_Unpack(o);
      if (t.defined() && !at::isTensorSubclassLike(t) && t.is_cuda() && t.has_storage() && t.is_contiguous()) return &t;
    }
    ok = false;
    return nullptr;
  }
  void* data(PyObject* o, at::ScalarType type, int64_t least) {
    const at::Tensor* t = tensor(o);
    if (t == nullptr || t->scalar_type() != type || t->numel() < least) { ok = false; return nullptr; }
    return t->data_ptr();
  }
  void* bytes(PyObject* o, int64_t least) {              // of any type
    const at::Tensor* t = tensor(o);
    if (t == nullptr || t->numel() * (int64_t)t->element_size() < least) { ok = false; return nullptr; }
    return t->data_ptr();
  }
  static int dtype_of(at::ScalarType type) {
    return type == at::kFloat ? DAF_F32 : type == at::kHalf ? DAF_F16 : type == at::kBFloat16 ? DAF_BF16 : -1;
  }
  // a tensor of the plan's size in one of the element formats; `dtype` -1: any, and it is told
  void* activation(PyObject* o, int& dtype) {
    const at::Tensor* t = tensor(o);
    const int d = t != nullptr ? dtype_of(t->scalar_type()) : -1;
    if (d < 0 || (dtype >= 0 && d != dtype) || t->numel() != elements) { ok = false; return nullptr; }
    dtype = d;
    return t->data_ptr();
  }
  struct Packed { uint32_t* words; float *min, *scale; };
  Packed packed(PyObject* words, PyObject* min, PyObject* scale) {
    Packed p;
    p.words = static_cast<uint32_t*>(data(words, at::kInt, ok ? lib.plan_packed_words(plan) : 0));
    p.min = static_cast<float*>(data(min, at::kFloat, groups));
    p.scale = static_cast<float*>(data(scale, at::kFloat, groups));
    return p;
  }
  const uint8_t* widths(PyObject* o) {                   // or None
    return o == Py_None ? nullptr : static_cast<const uint8_t*>(data(o, at::kByte, groups));
  }
  uint64_t seed(PyObject* o) {
    if (!PyLong_CheckExact(o)) { ok = false; return 0; }
    return PyLong_AsUnsignedLongLongMask(o);
  }
};

// Runs `make(call)`, which fills in the call and returns what is to be done without the interpreter's lock.
template <class Make>
PyObject* run(Py_ssize_t got, Py_ssize_t wanted, Make make) {
  try {
    Call c;
    if (got != wanted || plan_type == nullptr) c.ok = false;             // (nothing bound yet)
    if (c.ok) {
      auto call = make(c);
      if (c.ok) {
        int rc;
        // (An exception from the library's C functions ends the process, as it did on its way through ctypes: caught below, it would
        // come back to the interpreter without the lock.)
        auto without_the_lock = [&]() noexcept { rc = call(); };
        Py_BEGIN_ALLOW_THREADS
        without_the_lock();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
      }
    }
  } catch (...) {                                        // (a tensor that gives no pointer: the general way says so)
  }
  Py_RETURN_NONE;
}
using Args = PyObject* const*;

template <class F>
PyObject* quantize(F fn, Args a, Py_ssize_t n) {
  return run(n, 7, [&](Call& c) {
    c.with_plan(a[0]);
    int dt = -1;
    const void* x = c.activation(a[1], dt);
    const uint64_t seed = c.seed(a[2]);
    const auto p = c.packed(a[3], a[4], a[5]);
    c.with_stream(a[6]);
    return [=] { return fn(c.plan, x, static_cast<daf_dtype_t>(dt), seed, p.words, p.min, p.scale, c.stream); };
  });
}
PyObject* quantize_pack(PyObject*, Args a, Py_ssize_t n) { return quantize(lib.quantize_pack, a, n); }
PyObject* quantize_pack_static(PyObject*, Args a, Py_ssize_t n) { return quantize(lib.quantize_pack_static, a, n); }

PyObject* unpack_dequantize(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 7, [&](Call& c) {
    c.with_plan(a[0]);
    const auto p = c.packed(a[1], a[2], a[3]);
    int dt = -1;
    void* out = c.activation(a[4], dt);
    const uint8_t* bits = c.widths(a[5]);
    c.with_stream(a[6]);
    return [=] { return lib.unpack_dequantize(c.plan, p.words, p.min, p.scale, bits, out, static_cast<daf_dtype_t>(dt), c.stream); };
  });
}

PyObject* quantize_pack_metrics(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 8, [&](Call& c) {
    c.with_plan(a[0]);
    int dt = -1;
    const void* x = c.activation(a[1], dt);
    const uint64_t seed = c.seed(a[2]);
    const auto p = c.packed(a[3], a[4], a[5]);
    float* metrics = static_cast<float*>(c.data(a[6], at::kFloat, 3 * c.groups));
    c.with_stream(a[7]);
    return [=] { return lib.quantize_pack_metrics(c.plan, x, static_cast<daf_dtype_t>(dt), seed, p.words, p.min, p.scale, metrics, c.stream); };
  });
}

PyObject* relu_quantize_pack(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 8, [&](Call& c) {
    c.with_plan(a[0]);
    int dt = -1;
    const void* z = c.activation(a[1], dt);
    const uint64_t seed = c.seed(a[2]);
    void* y = c.activation(a[3], dt);
    const auto p = c.packed(a[4], a[5], a[6]);
    c.with_stream(a[7]);
    return [=] { return lib.relu_quantize_pack(c.plan, z, static_cast<daf_dtype_t>(dt), seed, y, p.words, p.min, p.scale, c.stream); };
  });
}

PyObject* unpack_relu_backward(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 8, [&](Call& c) {
    c.with_plan(a[0]);
    const auto p = c.packed(a[1], a[2], a[3]);
    int dt = -1;
    const void* grad_y = c.activation(a[4], dt);
    void* grad_z = c.activation(a[5], dt);
    const uint8_t* bits = c.widths(a[6]);
    c.with_stream(a[7]);
    return [=] { return lib.unpack_relu_backward(c.plan, p.words, p.min, p.scale, bits, grad_y, grad_z, static_cast<daf_dtype_t>(dt), c.stream); };
  });
}

PyObject* group_minmax(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 5, [&](Call& c) {
    c.with_plan(a[0]);
    int dt = -1;
    const void* x = c.activation(a[1], dt);
    float* lo = static_cast<float*>(c.data(a[2], at::kFloat, c.groups));
    float* hi = static_cast<float*>(c.data(a[3], at::kFloat, c.groups));
    c.with_stream(a[4]);
    return [=] { return lib.group_minmax(c.plan, x, static_cast<daf_dtype_t>(dt), lo, hi, c.stream); };
  });
}

PyObject* plan_update(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 3, [&](Call& c) {
    c.with_plan(a[0]);
    const uint8_t* bits = static_cast<const uint8_t*>(c.data(a[1], at::kByte, c.groups));
    if (c.ok && THPVariable_Unpack(a[1]).numel() != c.groups) c.ok = false;
    c.with_stream(a[2]);
    return [=] { return lib.plan_update(c.plan, bits, c.stream); };
  });
}

struct Classes {
  uint8_t of[4];
  int32_t n = 0;
};
Classes classes_of(Call& c, PyObject* o) {               // a list or tuple of up to four whole numbers
  Classes k;
  const bool list = PyList_CheckExact(o), tuple = PyTuple_CheckExact(o);
  const Py_ssize_t n = list ? PyList_GET_SIZE(o) : tuple ? PyTuple_GET_SIZE(o) : -1;
  if (n < 1 || n > 4) { c.ok = false; return k; }
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* v = list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i);
    if (!PyLong_CheckExact(v)) { c.ok = false; return k; }
    k.of[k.n++] = (uint8_t)PyLong_AsUnsignedLongLongMask(v);
  }
  return k;
}

// group_min, group_max (or group_scale, prev_bits), classes, out_bits, workspace, stream
PyObject* select(Args a, Py_ssize_t n, bool from_scale) {
  return run(n, 6, [&](Call& c) {
    const float* first = static_cast<const float*>(c.data(a[0], at::kFloat, 1));
    const int64_t G = c.ok ? THPVariable_Unpack(a[0]).numel() : 0;
    const float* max = nullptr;
    const uint8_t* prev = nullptr;
    int32_t uniform = 0;
    if (from_scale && PyLong_CheckExact(a[1])) {
      const long v = PyLong_AsLong(a[1]);
      if (PyErr_Occurred()) PyErr_Clear();
      if (v < 1 || v > 8) c.ok = false;
      uniform = (int32_t)v;
    } else {
      void* second = c.data(a[1], from_scale ? at::kByte : at::kFloat, G);
      if (c.ok && THPVariable_Unpack(a[1]).numel() != G) c.ok = false;
      if (from_scale) prev = static_cast<const uint8_t*>(second);
      else max = static_cast<const float*>(second);
    }
    const Classes k = classes_of(c, a[2]);
    uint8_t* out = static_cast<uint8_t*>(c.data(a[3], at::kByte, G));
    void* ws = c.data(a[4], at::kByte, c.ok ? lib.select_bits_workspace_bytes(G) : 0);
    c.with_stream(a[5]);
    return [=] {
      return from_scale ? lib.select_bits_from_scale(first, prev, uniform, G, k.of, k.n, out, ws, c.stream)
                        : lib.select_bits(first, max, G, k.of, k.n, out, ws, c.stream);
    };
  });
}
PyObject* select_bits(PyObject*, Args a, Py_ssize_t n) { return select(a, n, false); }
PyObject* select_bits_from_scale(PyObject*, Args a, Py_ssize_t n) { return select(a, n, true); }

// plan, x [M, K], weight [N, K], seed, out_y, out_words, out_min, out_scale, stream
PyObject* linear_quantize_pack(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 9, [&](Call& c) {
    c.with_plan(a[0]);
    const at::Tensor *x = c.tensor(a[1]), *w = c.tensor(a[2]);
    int64_t N = 0, K = 0;
    if (c.ok) {
      if (x->dim() != 2 || w->dim() != 2 || x->size(1) != w->size(1) || x->scalar_type() != w->scalar_type()) c.ok = false;
      else { N = w->size(0); K = x->size(1); }
      if (c.ok && x->size(0) * N != c.elements) c.ok = false;
    }
    int dt = c.ok ? Call::dtype_of(x->scalar_type()) : -1;
    if (dt < 0) c.ok = false;
    const uint64_t seed = c.seed(a[3]);
    void* y = c.activation(a[4], dt);
    const auto p = c.packed(a[5], a[6], a[7]);
    c.with_stream(a[8]);
    const void *px = c.ok ? x->data_ptr() : nullptr, *pw = c.ok ? w->data_ptr() : nullptr;
    return [=] { return lib.linear_quantize_pack(c.plan, px, pw, N, K, static_cast<daf_dtype_t>(dt), seed, y, p.words, p.min, p.scale, c.stream); };
  });
}

// plan, words, min, scale, grad_y [M, N], out_grad_w [N, K], workspace or None, bits or None, stream
PyObject* unpack_matmul_grad_weight(PyObject*, Args a, Py_ssize_t n) {
  return run(n, 9, [&](Call& c) {
    c.with_plan(a[0]);
    const auto p = c.packed(a[1], a[2], a[3]);
    const at::Tensor *gy = c.tensor(a[4]), *gw = c.tensor(a[5]);
    int64_t N = 0, K = 0;
    if (c.ok) {
      if (gy->dim() != 2 || gw->dim() != 2 || gw->scalar_type() != at::kFloat) c.ok = false;
      else { N = gw->size(0); K = gw->size(1); }
      if (c.ok && (gy->size(1) != N || K < 1 || gy->size(0) * K != c.elements)) c.ok = false;
    }
    const int dt = c.ok ? Call::dtype_of(gy->scalar_type()) : -1;
    if (dt < 0) c.ok = false;
    const int64_t need = c.ok ? lib.unpack_matmul_workspace_bytes(c.plan, N, K) : -1;
    if (need < 0) c.ok = false;
    void* ws = a[6] == Py_None ? nullptr : c.bytes(a[6], need);
    const uint8_t* bits = c.widths(a[7]);
    c.with_stream(a[8]);
    const void* pg = c.ok ? gy->data_ptr() : nullptr;
    float* out = c.ok ? static_cast<float*>(gw->data_ptr()) : nullptr;
    return [=] { return lib.unpack_matmul_grad_weight(c.plan, p.words, p.min, p.scale, bits, pg, N, K, static_cast<daf_dtype_t>(dt), out, ws, c.stream); };
  });
}

// bind({name: address}, Plan): where the library's functions are.
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *table, *type;
  if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &table, &type)) return nullptr;
  Library found;
  struct { const char* name; void* slot; } const slots[] = {
      {"daf_quantize_pack", &found.quantize_pack}, {"daf_quantize_pack_static", &found.quantize_pack_static},
      {"daf_unpack_dequantize", &found.unpack_dequantize}, {"daf_quantize_pack_metrics", &found.quantize_pack_metrics},
      {"daf_relu_quantize_pack", &found.relu_quantize_pack}, {"daf_unpack_relu_backward", &found.unpack_relu_backward},
      {"daf_group_minmax", &found.group_minmax}, {"daf_select_bits", &found.select_bits},
      {"daf_select_bits_from_scale", &found.select_bits_from_scale},
      {"daf_select_bits_workspace_bytes", &found.select_bits_workspace_bytes}, {"daf_plan_update", &found.plan_update},
      {"daf_linear_quantize_pack", &found.linear_quantize_pack},
      {"daf_unpack_matmul_grad_weight", &found.unpack_matmul_grad_weight},
      {"daf_unpack_matmul_workspace_bytes", &found.unpack_matmul_workspace_bytes},
      {"daf_plan_num_elements", &found.plan_num_elements}, {"daf_plan_num_groups", &found.plan_num_groups},
      {"daf_plan_packed_words", &found.plan_packed_words}};
  for (const auto& s : slots) {
    PyObject* v = PyDict_GetItemString(table, s.name);
    void* address = v != nullptr ? PyLong_AsVoidPtr(v) : nullptr;
    if (address == nullptr) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "no address for %s", s.name);
      return nullptr;
    }
    *static_cast<void**>(s.slot) = address;
  }
  lib = found;
  Py_INCREF(type);
  Py_XSETREF(plan_type, type);
  Py_RETURN_NONE;
}

#define DAF_FAST(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DAF_FAST(quantize_pack), DAF_FAST(quantize_pack_static), DAF_FAST(unpack_dequantize),
                         DAF_FAST(quantize_pack_metrics), DAF_FAST(relu_quantize_pack), DAF_FAST(unpack_relu_backward),
                         DAF_FAST(group_minmax), DAF_FAST(plan_update), DAF_FAST(select_bits), DAF_FAST(select_bits_from_scale),
                         DAF_FAST(linear_quantize_pack), DAF_FAST(unpack_matmul_grad_weight),
                         {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast_calls() {
  handle_name = PyUnicode_InternFromString("_h");
  stream_name = PyUnicode_InternFromString("cuda_stream");
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", DAF_TORCH_VERSION) < 0) Py_CLEAR(m);
  return m;
}
