// The Python binding's call path in native code: argument checks, workspace lookup and
// the C ABI call of one DecodeAttention method, without a Python statement per check.
//
// A method takes a call only when every argument is what the Python checks of
// paper_2607_09207_amd/__init__.py accept, and answers None for any other call (tensor
// subclasses, active modes, a workspace that is not allocated yet, a mismatch): the
// Python code then runs its own checks, which raise or go through ctypes.  Nothing is
// kept from one call for the next.
//
// Why: issuing a call took 16.2 us on the host (12.4 us of it checks in Python, 1 us the
// ctypes conversion) against 6 to 12 us of kernel time for the small calls; it takes
// 3.9 us here, nearly all of it the launch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rl_decode_attn.h"

namespace {

using at::Tensor;

// Entry points of the library, found by the caller (addresses) so that both bindings use
// the one that is loaded.
decltype(&rl_decode_attn_run) g_run;
decltype(&rl_decode_attn_run_grouped) g_grouped;
decltype(&rl_decode_attn_run_multi) g_multi;
decltype(&rl_decode_attn_run_noalloc) g_noalloc;
decltype(&rl_decode_attn_append) g_append;
PyObject* g_raw_stream;   // device index -> current stream (an int)

constexpr int kMaxDevices = 64;
PyObject* g_device_key[kMaxDevices];   // "cuda:0", ... : keys of the workspace dict

struct Layer {
  PyObject_HEAD
  rl_decode_attn_t handle;
  PyObject* workspaces;   // dict: device string -> uint8 tensor (the Python object's own)
  int64_t hq, hkv, d, page, max_batch, max_pages;
  int64_t stride[3];
  int64_t ws_bytes, grouped_ws_bytes;   // as allocated, alignment room included
  at::ScalarType q_dtype, kv_dtype, out_dtype;
  bool fp8;
};

at::ScalarType scalar_of(int code) {
  return code == RLDA_F32 ? at::kFloat : code == RLDA_BF16 ? at::kBFloat16 : at::kFloat8_e4m3fn;
}

// The tensor of an argument, or null: not a plain strided tensor.
const Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || !t.has_storage() || at::isTensorSubclassLike(t)) return nullptr;
  return &t;
}

bool plain(const Tensor* t, int dev, at::ScalarType type) {
  return t && t->is_cuda() && t->get_device() == dev && t->scalar_type() == type;
}
bool shaped(const Tensor* t, int dev, at::ScalarType type, at::IntArrayRef shape) {
  return plain(t, dev, type) && t->sizes() == shape && t->is_contiguous();
}

// One call's arguments that every method shares.
struct Call {
  int dev = -1;
  int64_t npages = 0;
  const Tensor *k = nullptr, *v = nullptr, *ks = nullptr, *vs = nullptr, *bt = nullptr, *lens = nullptr;
  Tensor ws;   // held: the dict's entry may be replaced while the call is without the GIL
  char* ws_ptr = nullptr;
  size_t ws_room = 0;
  void* stream = nullptr;
};

bool cache_ok(const Layer* L, const Tensor* t, int dev, int64_t npages) {
  if (!plain(t, dev, L->kv_dtype) || t->dim() != 4) return false;
  const auto sz = t->sizes(), st = t->strides();
  if (sz[1] != L->hkv || sz[2] != L->page || sz[3] != L->d || sz[0] < npages) return false;
  for (int i = 0; i < 3; ++i)
    if (sz[i] > 1 && st[i] != L->stride[i]) return false;
  return sz[3] <= 1 || st[3] == 1;
}

bool scale_ok(const Layer* L, const Tensor* t, int dev, int64_t npages) {
  return plain(t, dev, at::kFloat) && t->dim() == 2 && t->size(1) == L->hkv && t->size(0) >= npages &&
         t->is_contiguous();
}

// An int argument, or `none` for None; false: neither.
bool as_int(PyObject* o, int64_t none, int64_t* out) {
  if (o == Py_None) {
    *out = none;
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  const long long x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *out = x;
  return true;
}

// The arguments common to the methods, in order: k, v, block table, lengths, k scale,
// v scale, stream, page count; `batch` sequences on device `dev`.
bool common(const Layer* L, Call& c, PyObject* const* a, int dev, int64_t batch) {
  c.dev = dev;
  c.k = tensor(a[0]);
  c.v = tensor(a[1]);
  c.bt = tensor(a[2]);
  c.lens = tensor(a[3]);
  if (!c.k || !c.v || c.k->dim() != 4 || !as_int(a[7], c.k->size(0), &c.npages)) return false;
  if (c.npages < 0 || c.npages > INT32_MAX || batch < 0 || batch > L->max_batch) return false;
  if (!cache_ok(L, c.k, dev, c.npages) || !cache_ok(L, c.v, dev, c.npages)) return false;
  if (!shaped(c.bt, dev, at::kInt, {batch, L->max_pages}) || !shaped(c.lens, dev, at::kInt, {batch})) return false;
  if (L->fp8) {
    c.ks = tensor(a[4]);
    c.vs = tensor(a[5]);
    if (!scale_ok(L, c.ks, dev, c.npages) || !scale_ok(L, c.vs, dev, c.npages)) return false;
  } else if (a[4] != Py_None || a[5] != Py_None) {
    return false;
  }
  int64_t s = 0;
  if (a[6] == Py_None) {
    PyObject* idx = PyLong_FromLong(dev);
    PyObject* r = idx ? PyObject_CallFunctionObjArgs(g_raw_stream, idx, nullptr) : nullptr;
    Py_XDECREF(idx);
    const bool ok = r && as_int(r, 0, &s);
    Py_XDECREF(r);
    if (!ok) {
      PyErr_Clear();
      return false;
    }
  } else if (!as_int(a[6], 0, &s)) {
    PyObject* r = PyObject_GetAttrString(a[6], "cuda_stream");   // a torch.cuda.Stream
    const bool ok = r && as_int(r, 0, &s);
    Py_XDECREF(r);
    if (!ok) {
      PyErr_Clear();
      return false;
    }
  }
  c.stream = (void*)(intptr_t)s;
  return true;
}

// The workspace given, or the one the Python object keeps for the device.
bool workspace(const Layer* L, Call& c, PyObject* given, bool grouped) {
  const Tensor* t = nullptr;
  if (given != Py_None) {
    t = tensor(given);
  } else {
    if (c.dev >= kMaxDevices) return false;
    PyObject* o = PyDict_GetItem(L->workspaces, g_device_key[c.dev]);   // borrowed
    t = o ? tensor(o) : nullptr;
    if (t && t->numel() < (grouped ? L->grouped_ws_bytes : L->ws_bytes)) return false;
  }
  if (!plain(t, c.dev, at::kByte) || !t->is_contiguous()) return false;
  c.ws = *t;
  char* p = (char*)t->mutable_data_ptr();
  c.ws_ptr = (char*)(((uintptr_t)p + 255) / 256 * 256);
  const int64_t room = t->numel() - (c.ws_ptr - p);
  if (room < 0) return false;
  c.ws_room = (size_t)room;
  return true;
}

void* ptr(const Tensor* t) { return t ? t->mutable_data_ptr() : nullptr; }

// The output given, or a new tensor (rows, Hq, d) held by `fresh`.
const Tensor* output(const Layer* L, PyObject* given, const Tensor& q, int64_t rows, Tensor& fresh) {
  if (given == Py_None) {
    fresh = at::empty({rows, L->hq, L->d}, at::TensorOptions().dtype(L->out_dtype).device(q.device()));
    return &fresh;
  }
  const Tensor* o = tensor(given);
  return shaped(o, q.get_device(), L->out_dtype, {rows, L->hq, L->d}) ? o : nullptr;
}

// The call's answer: the output tensor, or the status of a call that failed.
PyObject* answer(rlda_status st, PyObject* given, const Tensor& fresh) {
  if (st != RLDA_OK) return PyLong_FromLong((long)st);
  if (given != Py_None) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(fresh);
}

// Runs `body` with C++ exceptions (a tensor without data, no memory) turned into "not
// taken": the Python path then meets, and reports, the same condition.
template <class F>
PyObject* guarded(F body) {
  try {
    PyObject* r = body();
    if (r) return r;
    if (PyErr_Occurred()) return nullptr;
  } catch (const std::exception&) {
  }
  Py_RETURN_NONE;
}

#define WITHOUT_GIL(call)    \
  rlda_status st;            \
  Py_BEGIN_ALLOW_THREADS     \
  st = (call);               \
  Py_END_ALLOW_THREADS

// run(q, k, v, block_table, seq_lens, k_scale, v_scale, stream, num_pages, out, workspace)
PyObject* layer_run(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n != 11) return PyErr_Format(PyExc_TypeError, "run takes 11 arguments");
  const Layer* L = (const Layer*)self;
  return guarded([&]() -> PyObject* {
    const Tensor* q = tensor(a[0]);
    if (!q || !q->is_cuda() || q->dim() != 3) return nullptr;
    const int dev = q->get_device();
    const int64_t B = q->size(0);
    Call c;
    if (!shaped(q, dev, L->q_dtype, {B, L->hq, L->d}) || !common(L, c, a + 1, dev, B) || !workspace(L, c, a[10], false))
      return nullptr;
    Tensor fresh;
    const Tensor* o = output(L, a[9], *q, B, fresh);
    if (!o) return nullptr;
    void *qp = ptr(q), *kp = ptr(c.k), *vp = ptr(c.v), *ksp = ptr(c.ks), *vsp = ptr(c.vs), *bp = ptr(c.bt),
         *lp = ptr(c.lens), *op = ptr(o);
    WITHOUT_GIL(g_run(L->handle, (int32_t)B, (int32_t)c.npages, qp, kp, vp, (const float*)ksp, (const float*)vsp,
                      (const int32_t*)bp, (const int32_t*)lp, op, c.ws_ptr, c.ws_room, c.stream));
    return answer(st, a[9], fresh);
  });
}

// grouped(q, k, v, block_table, seq_lens, k_scale, v_scale, stream, num_pages, out, workspace,
//         group_size, prefix_pages, prompt_pages_hint)
PyObject* layer_grouped(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n != 14) return PyErr_Format(PyExc_TypeError, "grouped takes 14 arguments");
  const Layer* L = (const Layer*)self;
  return guarded([&]() -> PyObject* {
    const Tensor* q = tensor(a[0]);
    if (!q || !q->is_cuda() || q->dim() != 3) return nullptr;
    const int dev = q->get_device();
    const int64_t B = q->size(0);
    Call c;
    int64_t gs = 0, hint = -1;
    const Tensor* pp = tensor(a[12]);
    if (!as_int(a[11], 0, &gs) || a[13] == Py_None || !as_int(a[13], -1, &hint) || gs < 1 || gs > INT32_MAX ||
        hint < INT32_MIN || hint > INT32_MAX)
      return nullptr;
    if (!shaped(q, dev, L->q_dtype, {B, L->hq, L->d}) || !common(L, c, a + 1, dev, B) ||
        !shaped(pp, dev, at::kInt, {(B + gs - 1) / gs}) || !workspace(L, c, a[10], true))
      return nullptr;
    Tensor fresh;
    const Tensor* o = output(L, a[9], *q, B, fresh);
    if (!o) return nullptr;
    void *qp = ptr(q), *kp = ptr(c.k), *vp = ptr(c.v), *ksp = ptr(c.ks), *vsp = ptr(c.vs), *bp = ptr(c.bt),
         *lp = ptr(c.lens), *op = ptr(o), *ppp = ptr(pp);
    WITHOUT_GIL(g_grouped(L->handle, (int32_t)B, (int32_t)c.npages, (int32_t)gs, (const int32_t*)ppp, (int32_t)hint, qp,
                          kp, vp, (const float*)ksp, (const float*)vsp, (const int32_t*)bp, (const int32_t*)lp, op,
                          c.ws_ptr, c.ws_room, c.stream, nullptr, nullptr));
    return answer(st, a[9], fresh);
  });
}

// multi(q, k, v, block_table, seq_lens, k_scale, v_scale, stream, num_pages, out, workspace,
//       q_start, max_q_len)
PyObject* layer_multi(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n != 13) return PyErr_Format(PyExc_TypeError, "multi takes 13 arguments");
  const Layer* L = (const Layer*)self;
  return guarded([&]() -> PyObject* {
    const Tensor *q = tensor(a[0]), *qs = tensor(a[11]);
    if (!q || !q->is_cuda() || q->dim() != 3 || !qs || qs->dim() != 1) return nullptr;
    const int dev = q->get_device();
    const int64_t total = q->size(0), B = qs->size(0) - 1;
    Call c;
    int64_t mq = 0;
    if (total > INT32_MAX || a[12] == Py_None || !as_int(a[12], 0, &mq) || mq < INT32_MIN || mq > INT32_MAX)
      return nullptr;
    if (!shaped(q, dev, L->q_dtype, {total, L->hq, L->d}) || !shaped(qs, dev, at::kInt, {B + 1}) ||
        !common(L, c, a + 1, dev, B) || !workspace(L, c, a[10], false))
      return nullptr;
    Tensor fresh;
    const Tensor* o = output(L, a[9], *q, total, fresh);
    if (!o) return nullptr;
    void *qp = ptr(q), *kp = ptr(c.k), *vp = ptr(c.v), *ksp = ptr(c.ks), *vsp = ptr(c.vs), *bp = ptr(c.bt),
         *lp = ptr(c.lens), *op = ptr(o), *qsp = ptr(qs);
    WITHOUT_GIL(g_multi(L->handle, (int32_t)B, (int32_t)c.npages, (int32_t)total, (int32_t)mq, qp, kp, vp,
                        (const float*)ksp, (const float*)vsp, (const int32_t*)bp, (const int32_t*)lp,
                        (const int32_t*)qsp, op, c.ws_ptr, c.ws_room, c.stream, nullptr, nullptr));
    return answer(st, a[9], fresh);
  });
}

// noalloc(q, k, v, block_table, seq_lens, k_scale, v_scale, stream, num_pages, out, flags)
PyObject* layer_noalloc(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n != 11) return PyErr_Format(PyExc_TypeError, "noalloc takes 11 arguments");
  const Layer* L = (const Layer*)self;
  return guarded([&]() -> PyObject* {
    const Tensor* q = tensor(a[0]);
    if (!q || !q->is_cuda() || q->dim() != 3) return nullptr;
    const int dev = q->get_device();
    const int64_t B = q->size(0);
    Call c;
    const Tensor* flags = nullptr;
    if (a[10] != Py_None && !shaped(flags = tensor(a[10]), dev, at::kInt, {1})) return nullptr;
    if (!shaped(q, dev, L->q_dtype, {B, L->hq, L->d}) || !common(L, c, a + 1, dev, B)) return nullptr;
    Tensor fresh;
    const Tensor* o = output(L, a[9], *q, B, fresh);
    if (!o) return nullptr;
    void *qp = ptr(q), *kp = ptr(c.k), *vp = ptr(c.v), *ksp = ptr(c.ks), *vsp = ptr(c.vs), *bp = ptr(c.bt),
         *lp = ptr(c.lens), *op = ptr(o), *fp = ptr(flags);
    WITHOUT_GIL(g_noalloc(L->handle, (int32_t)B, (int32_t)c.npages, qp, kp, vp, (const float*)ksp, (const float*)vsp,
                          (const int32_t*)bp, (const int32_t*)lp, op, (uint32_t*)fp, c.stream));
    return answer(st, a[9], fresh);
  });
}

// append(k_new, k, v, block_table, seq_lens, k_scale, v_scale, stream, num_pages, v_new, workspace):
// the status, or None (not taken).
PyObject* layer_append(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  if (n != 11) return PyErr_Format(PyExc_TypeError, "append takes 11 arguments");
  const Layer* L = (const Layer*)self;
  return guarded([&]() -> PyObject* {
    const Tensor *kn = tensor(a[0]), *vn = tensor(a[9]);
    if (!kn || !kn->is_cuda() || kn->dim() != 3) return nullptr;
    const int dev = kn->get_device();
    const int64_t B = kn->size(0);
    Call c;
    if (!shaped(kn, dev, L->q_dtype, {B, L->hkv, L->d}) || !shaped(vn, dev, L->q_dtype, {B, L->hkv, L->d}) ||
        !common(L, c, a + 1, dev, B) || !workspace(L, c, a[10], false))
      return nullptr;
    void *knp = ptr(kn), *vnp = ptr(vn), *kp = ptr(c.k), *vp = ptr(c.v), *ksp = ptr(c.ks), *vsp = ptr(c.vs),
         *bp = ptr(c.bt), *lp = ptr(c.lens);
    WITHOUT_GIL(g_append(L->handle, (int32_t)B, (int32_t)c.npages, knp, vnp, kp, vp, (float*)ksp, (float*)vsp,
                         (const int32_t*)bp, (const int32_t*)lp, c.ws_ptr, c.ws_room, c.stream));
    return PyLong_FromLong((long)st);
  });
}

PyMethodDef layer_methods[] = {
    {"run", (PyCFunction)(void*)layer_run, METH_FASTCALL, nullptr},
    {"grouped", (PyCFunction)(void*)layer_grouped, METH_FASTCALL, nullptr},
    {"multi", (PyCFunction)(void*)layer_multi, METH_FASTCALL, nullptr},
    {"noalloc", (PyCFunction)(void*)layer_noalloc, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void*)layer_append, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

void layer_dealloc(PyObject* self) {
  Py_XDECREF(((Layer*)self)->workspaces);
  Py_TYPE(self)->tp_free(self);
}

// Layer(handle, workspaces, (Hq, Hkv, d, page, max_batch, max_pages), (q, kv, out dtype codes),
//       (page, head, slot strides), workspace bytes, grouped workspace bytes)
PyObject* layer_new(PyTypeObject* type, PyObject* args, PyObject*) {
  unsigned long long handle = 0;
  PyObject* dict = nullptr;
  long long v[6], s[3], ws = 0, gws = 0;
  int q = 0, kv = 0, out = 0;
  if (!PyArg_ParseTuple(args, "KO!(LLLLLL)(iii)(LLL)LL", &handle, &PyDict_Type, &dict, &v[0], &v[1], &v[2], &v[3], &v[4],
                        &v[5], &q, &kv, &out, &s[0], &s[1], &s[2], &ws, &gws))
    return nullptr;
  Layer* L = (Layer*)type->tp_alloc(type, 0);
  if (!L) return nullptr;
  L->handle = (rl_decode_attn_t)(uintptr_t)handle;
  Py_INCREF(dict);
  L->workspaces = dict;
  L->hq = v[0], L->hkv = v[1], L->d = v[2], L->page = v[3], L->max_batch = v[4], L->max_pages = v[5];
  for (int i = 0; i < 3; ++i) L->stride[i] = s[i];
  L->ws_bytes = ws;
  L->grouped_ws_bytes = gws;
  L->q_dtype = scalar_of(q);
  L->kv_dtype = scalar_of(kv);
  L->out_dtype = scalar_of(out);
  L->fp8 = kv == RLDA_FP8_E4M3FN;
  return (PyObject*)L;
}

PyTypeObject layer_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bind(raw_stream, run, grouped, multi, noalloc, append): the stream lookup and the
// addresses of the loaded library's entry points.
PyObject* bind(PyObject*, PyObject* args) {
  PyObject* raw = nullptr;
  unsigned long long f[5];
  if (!PyArg_ParseTuple(args, "OKKKKK", &raw, &f[0], &f[1], &f[2], &f[3], &f[4])) return nullptr;
  Py_INCREF(raw);
  Py_XDECREF(g_raw_stream);
  g_raw_stream = raw;
  g_run = (decltype(g_run))(uintptr_t)f[0];
  g_grouped = (decltype(g_grouped))(uintptr_t)f[1];
  g_multi = (decltype(g_multi))(uintptr_t)f[2];
  g_noalloc = (decltype(g_noalloc))(uintptr_t)f[3];
  g_append = (decltype(g_append))(uintptr_t)f[4];
  Py_RETURN_NONE;
}

PyMethodDef module_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  layer_type.tp_name = "paper_2607_09207_amd._fastcall.Layer";
  layer_type.tp_basicsize = sizeof(Layer);
  layer_type.tp_flags = Py_TPFLAGS_DEFAULT;
  layer_type.tp_new = layer_new;
  layer_type.tp_dealloc = layer_dealloc;
  layer_type.tp_methods = layer_methods;
  if (PyType_Ready(&layer_type) < 0) return nullptr;
  for (int i = 0; i < kMaxDevices; ++i) {
    g_device_key[i] = PyUnicode_InternFromString(("cuda:" + std::to_string(i)).c_str());
    if (!g_device_key[i]) return nullptr;
  }
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&layer_type);
  if (PyModule_AddObject(m, "Layer", (PyObject*)&layer_type) < 0) return nullptr;
  return m;
}
