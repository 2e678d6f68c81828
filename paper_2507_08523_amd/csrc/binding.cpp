// The device calls of the Python binding that a serving loop issues per layer,
// natively: the same checks as ilpc.py makes before it hands pointers over
// (tensor type, dtype, device, contiguity, shapes), then the library call.  In
// Python, the checks, the ctypes conversions and the launch took about 14 us a
// call, more than the kernels of a small batch run: an append and an attention
// call of 3 requests of 96 rows over a 64-key prefix took 30.0 us back to back,
// 8.8 with these; a host thread that stays ahead of longer kernels gains nothing.
//
// A function returns the library's code, or None with nothing called for
// whatever it does not take as it stands (another type of argument or tensor, a
// failed check, a workspace still to be allocated): ilpc.py then takes its own
// path, which allocates, converts, or raises the error with its text.  Nothing
// is kept from one call to the next but the library's entry points.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <climits>

#include "../../include/ilpc.h"

namespace {

// The entry points of the library that ilpc.py has loaded (bind(), below).
decltype(&ilpc_kv_append) kv_append = nullptr;
decltype(&ilpc_rope_kv_append) rope_kv_append = nullptr;
decltype(&ilpc_attn_workspace_bytes) attn_workspace_bytes = nullptr;
decltype(&ilpc_paged_prefill_attn) prefill_attn = nullptr;
decltype(&ilpc_paged_prefill_attn_cascade) prefill_attn_cascade = nullptr;

constexpr int kNotHere = INT_MIN;  // what a body returns for a call it does not take

// Arguments of one call, in order; ok turns false at the first that does not fit.
struct Args {
  PyObject* const* a;
  Py_ssize_t n, i = 0;
  bool ok = true;

  PyObject* next() {
    if (i >= n) {
      ok = false;
      return Py_None;
    }
    return a[i++];
  }
  // A plain contiguous GPU tensor of this type and rank (nullptr otherwise).
  const at::Tensor* tensor(at::ScalarType type, int64_t dim) {
    PyObject* o = next();
    if (!ok || !THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || t.dim() != dim || !t.is_contiguous()) {
      ok = false;
      return nullptr;
    }
    return &t;
  }
  const at::Tensor* tensor_or_none(at::ScalarType type, int64_t dim) {
    if (i < n && a[i] == Py_None) {
      ++i;
      return nullptr;
    }
    return tensor(type, dim);
  }
  int32_t integer() {
    PyObject* o = next();
    if (!ok || !PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v != int32_t(v)) ok = false;
    return int32_t(v);
  }
  float real() {
    PyObject* o = next();
    if (!ok || !PyFloat_Check(o)) {
      ok = false;
      return 0.f;
    }
    return float(PyFloat_AS_DOUBLE(o));
  }
};

// The stream of a call: a torch stream object, or None for the current
// device's current stream; and its device's index.
bool stream_of(PyObject* o, void** stream, int* device) {
  if (o == Py_None) {
    const auto s = c10::hip::getCurrentHIPStream();
    *stream = s.stream();
    *device = s.device_index();
    return true;
  }
  PyObject* p = PyObject_GetAttrString(o, "cuda_stream");
  PyObject* d = p ? PyObject_GetAttrString(o, "device_index") : nullptr;
  bool ok = p && d && PyLong_Check(p) && PyLong_Check(d);
  if (ok) {
    *stream = PyLong_AsVoidPtr(p);
    *device = int(PyLong_AsLong(d));
    ok = !PyErr_Occurred();
  }
  Py_XDECREF(p);
  Py_XDECREF(d);
  return ok;
}

uint16_t* bf16(const at::Tensor* t) { return static_cast<uint16_t*>(t->data_ptr()); }
int32_t* i32(const at::Tensor* t) { return static_cast<int32_t*>(t->data_ptr()); }

// Pools [NB, Hkv, 16, D] and [NB, Hkv, D, 16] that fit each other.
bool pools_fit(const at::Tensor& k, const at::Tensor& v) {
  return v.size(0) == k.size(0) && v.size(1) == k.size(1) && v.size(2) == k.size(3) && v.size(3) == k.size(2);
}

// Runs a call body: its code, or None.  What it throws (torch's checks do) or
// leaves as a Python error comes before the library call and means None.
template <class F>
PyObject* guarded(F&& body) {
  int rc = kNotHere;
  try {
    rc = body();
  } catch (const std::exception&) {
  }
  PyErr_Clear();
  if (rc == kNotHere) Py_RETURN_NONE;
  return PyLong_FromLong(rc);
}

// The library call, without the interpreter's lock (the arguments are evaluated with it: data_ptr() may throw).
template <class... P, class... A>
int call(int (*fn)(P...), A... args) {
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = fn(args...);
  Py_END_ALLOW_THREADS;
  return rc;
}

// bind(addresses of kv_append, rope_kv_append, attn_workspace_bytes, paged_prefill_attn, paged_prefill_attn_cascade)
PyObject* py_bind(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  void* p[5];
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "bind() takes 5 addresses");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i) p[i] = PyLong_AsVoidPtr(argv[i]);
  if (PyErr_Occurred()) return nullptr;
  kv_append = reinterpret_cast<decltype(kv_append)>(p[0]);
  rope_kv_append = reinterpret_cast<decltype(rope_kv_append)>(p[1]);
  attn_workspace_bytes = reinterpret_cast<decltype(attn_workspace_bytes)>(p[2]);
  prefill_attn = reinterpret_cast<decltype(prefill_attn)>(p[3]);
  prefill_attn_cascade = reinterpret_cast<decltype(prefill_attn_cascade)>(p[4]);
  Py_RETURN_NONE;
}

// kv_append(k_new, v_new, k_pool, v_pool, block_tables, cu_new, start_pos, max_new, stream)
PyObject* py_kv_append(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  return guarded([&]() -> int {
    Args a{argv, n};
    const at::Tensor *k = a.tensor(at::kBFloat16, 3), *v = a.tensor(at::kBFloat16, 3),
                     *kp = a.tensor(at::kBFloat16, 4), *vp = a.tensor(at::kBFloat16, 4), *bt = a.tensor(at::kInt, 2),
                     *cu = a.tensor(at::kInt, 1), *sp = a.tensor(at::kInt, 1);
    const int32_t max_new = a.integer();
    PyObject* so = a.next();
    if (!a.ok) return kNotHere;
    const int64_t NB = kp->size(0), Hkv = kp->size(1), bs = kp->size(2), D = kp->size(3), B = cu->size(0) - 1;
    if (!pools_fit(*kp, *vp) || k->size(1) != Hkv || k->size(2) != D || v->sizes() != k->sizes() ||
        bt->size(0) != B || sp->size(0) != B)
      return kNotHere;
    void* s;
    int dev;
    if (!stream_of(so, &s, &dev)) return kNotHere;
    return call(kv_append, bf16(k), bf16(v), bf16(kp), bf16(vp), int32_t(NB), i32(bt), int32_t(bt->size(1)), i32(cu),
                i32(sp), int32_t(B), max_new, int32_t(Hkv), int32_t(D), int32_t(bs), s);
  });
}

// rope_kv_append(q, q_out, k_new, v_new, k_pool, v_pool, block_tables, cu_new, start_pos, max_new, inv_freq, stream)
PyObject* py_rope_kv_append(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  return guarded([&]() -> int {
    Args a{argv, n};
    const at::Tensor *q = a.tensor_or_none(at::kBFloat16, 3), *qo = a.tensor_or_none(at::kBFloat16, 3),
                     *k = a.tensor(at::kBFloat16, 3), *v = a.tensor(at::kBFloat16, 3),
                     *kp = a.tensor(at::kBFloat16, 4), *vp = a.tensor(at::kBFloat16, 4), *bt = a.tensor(at::kInt, 2),
                     *cu = a.tensor(at::kInt, 1), *sp = a.tensor(at::kInt, 1);
    const int32_t max_new = a.integer();
    const at::Tensor* fr = a.tensor(at::kFloat, 1);
    PyObject* so = a.next();
    if (!a.ok) return kNotHere;
    const int64_t NB = kp->size(0), Hkv = kp->size(1), bs = kp->size(2), D = kp->size(3), B = cu->size(0) - 1;
    if (!pools_fit(*kp, *vp) || k->size(1) != Hkv || k->size(2) != D || v->sizes() != k->sizes() ||
        !q != !qo || (q && (q->size(0) != k->size(0) || q->size(2) != D || qo->sizes() != q->sizes())) ||
        fr->size(0) != D / 2 || bt->size(0) != B || sp->size(0) != B)
      return kNotHere;
    void* s;
    int dev;
    if (!stream_of(so, &s, &dev)) return kNotHere;
    return call(rope_kv_append, q ? bf16(q) : nullptr, q ? bf16(qo) : nullptr, int32_t(q ? q->size(1) : Hkv),
                bf16(k), bf16(v), bf16(kp), bf16(vp), int32_t(NB), i32(bt), int32_t(bt->size(1)), i32(cu), i32(sp),
                int32_t(B), max_new, int32_t(Hkv), int32_t(D), int32_t(bs), static_cast<float*>(fr->data_ptr()), s);
  });
}

struct Attn {
  const at::Tensor *q, *kp, *vp, *bt, *cu, *L;
  int32_t max_q;
  int64_t B;

  bool read(Args& a) {
    q = a.tensor(at::kBFloat16, 3), kp = a.tensor(at::kBFloat16, 4), vp = a.tensor(at::kBFloat16, 4);
    bt = a.tensor(at::kInt, 2), cu = a.tensor(at::kInt, 1), L = a.tensor(at::kInt, 1);
    max_q = a.integer();
    if (!a.ok) return false;
    B = cu->size(0) - 1;
    return q->size(2) == kp->size(3) && pools_fit(*kp, *vp) && bt->size(0) == B && L->size(0) == B;
  }
};

// paged_prefill_attn(q, k_pool, v_pool, block_tables, cu_q, seq_lens, max_q_len, scale, out, workspace, stream,
//                    workspaces kept by (device index, stream))
PyObject* py_prefill_attn(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  return guarded([&]() -> int {
    Args a{argv, n};
    Attn t;
    if (!t.read(a)) return kNotHere;
    const float scale = a.real();
    const at::Tensor* out = a.tensor(at::kBFloat16, 3);
    PyObject *wo = a.next(), *so = a.next(), *kept = a.next();
    if (!a.ok || out->sizes() != t.q->sizes() || !PyDict_CheckExact(kept)) return kNotHere;
    void* s;
    int dev;
    if (!stream_of(so, &s, &dev)) return kNotHere;
    const int32_t Hq = int32_t(t.q->size(1)), Hkv = int32_t(t.kp->size(1)), D = int32_t(t.kp->size(3));
    if (wo == Py_None) {
      // the kept buffer of this stream, where it is there and large enough
      size_t need = 0;
      if (t.q->device().index() != dev || attn_workspace_bytes(int32_t(t.B), t.max_q, Hq, Hkv, D, &need) != ILPC_OK)
        return kNotHere;
      PyObject* key = Py_BuildValue("(iN)", dev, PyLong_FromVoidPtr(s));
      wo = key ? PyDict_GetItemWithError(kept, key) : nullptr;  // (borrowed: the dictionary holds it)
      Py_XDECREF(key);
      if (!wo || !THPVariable_CheckExact(wo) || size_t(THPVariable_Unpack(wo).numel()) < need) return kNotHere;
    }
    PyObject* one[1] = {wo};
    Args w{one, 1};
    const at::Tensor* ws = w.tensor(at::kByte, 1);
    if (!w.ok) return kNotHere;
    const at::Tensor hold = *ws;  // (another thread may replace the kept buffer once the lock is let go)
    return call(prefill_attn, bf16(t.q), bf16(t.kp), bf16(t.vp), int32_t(t.kp->size(0)), i32(t.bt),
                int32_t(t.bt->size(1)), i32(t.cu), i32(t.L), int32_t(t.B), t.max_q, Hq, Hkv, D,
                int32_t(t.kp->size(2)), scale, bf16(out), hold.data_ptr(), size_t(hold.numel()), s);
  });
}

// paged_prefill_attn_cascade(q, k_pool, v_pool, block_tables, cu_q, seq_lens, max_q_len, shared_len, scale, out,
//                            workspace, stream)
PyObject* py_prefill_attn_cascade(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  return guarded([&]() -> int {
    Args a{argv, n};
    Attn t;
    if (!t.read(a)) return kNotHere;
    const int32_t shared = a.integer();
    const float scale = a.real();
    const at::Tensor *out = a.tensor(at::kBFloat16, 3), *ws = a.tensor(at::kByte, 1);
    PyObject* so = a.next();
    if (!a.ok || out->sizes() != t.q->sizes()) return kNotHere;
    void* s;
    int dev;
    if (!stream_of(so, &s, &dev)) return kNotHere;
    return call(prefill_attn_cascade, bf16(t.q), bf16(t.kp), bf16(t.vp), int32_t(t.kp->size(0)), i32(t.bt),
                int32_t(t.bt->size(1)), i32(t.cu), i32(t.L), int32_t(t.B), t.max_q, int32_t(t.q->size(1)),
                int32_t(t.kp->size(1)), int32_t(t.kp->size(3)), int32_t(t.kp->size(2)), shared, scale, bf16(out),
                ws->data_ptr(), size_t(ws->numel()), s);
  });
}

#define FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST("bind", py_bind),
                         FAST("kv_append", py_kv_append), FAST("rope_kv_append", py_rope_kv_append),
                         FAST("paged_prefill_attn", py_prefill_attn),
                         FAST("paged_prefill_attn_cascade", py_prefill_attn_cascade),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
