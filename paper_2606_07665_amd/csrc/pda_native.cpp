// Native argument marshalling of the binding's hot calls (CPython extension).
//
// A small decode call is ~10 us of GPU time; checking its tensors one
// attribute at a time in Python and converting its arguments through ctypes
// took 5-10 us of host time on top of the launches (a prelude with the append
// 14-16 us a call, o_proj 13).  These functions make the same checks on the
// tensors themselves and call the C ABI.
//
// Each returns the library's status code, or kDeclined where anything is not
// the plain accepted case -- another type than a plain torch.Tensor, a wrong
// dtype, shape, device or layout, an argument that is not a number of its
// range.  The caller then takes the Python path, which makes every check
// again in its documented order and raises the specific error, so this file
// decides nothing on its own but the accepted case.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "pda.h"

namespace {

constexpr int kDeclined = -1;

// Entry points of the loaded library, given by address (init).
struct Lib {
  decltype(&paged_decode_attention_ext) attention_ext = nullptr;
  decltype(&paged_decode_attention_noalloc) attention_noalloc = nullptr;
  decltype(&paged_decode_attention_append) attention_append = nullptr;
  decltype(&pda_kv_append_n) kv_append_n = nullptr;
  decltype(&pda_attention_prelude) prelude = nullptr;
  decltype(&pda_attention_prelude_append) prelude_append = nullptr;
  decltype(&pda_o_proj_residual_norm) o_proj = nullptr;
} g_lib;
PyObject* g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream
PyObject* g_device = nullptr;      // torch._C._cuda_getDevice

// One call's accepted tensors: all on one GPU, contiguous.
struct Checker {
  bool ok = true;
  int device = -1;

  // The tensor if it is a plain one of this dtype and rank, else null.
  const at::Tensor* take(PyObject* o, at::ScalarType dt, int64_t ndim) {
    if (!ok || !THPVariable_CheckExact(o)) return reject();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.dim() != ndim || t.scalar_type() != dt || !t.is_cuda() || !t.is_contiguous()) return reject();
    const int d = static_cast<int>(t.get_device());
    if (d < 0 || (device >= 0 && d != device)) return reject();
    device = d;
    return &t;
  }
  const at::Tensor* reject() {
    ok = false;
    return nullptr;
  }
  void same(int64_t a, int64_t b) { ok = ok && a == b; }
  int32_t i32(int64_t v) {
    if (v < INT32_MIN || v > INT32_MAX) ok = false;
    return static_cast<int32_t>(v);
  }
  int32_t integer(PyObject* o) {
    if (!ok || !PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) ok = false;
    return i32(v);
  }
  float number(PyObject* o) {
    if (!ok) return 0.f;
    if (PyFloat_CheckExact(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0.f;
    }
    const double v = PyLong_AsDouble(o);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return static_cast<float>(v);
  }
  // The raw handle of `stream`, or of torch's current stream on the tensors'
  // device.  of_current: the call takes the current device's stream instead,
  // so tensors on another device are left to the Python path.
  void* stream(PyObject* o, bool of_current) {
    if (!ok) return nullptr;
    PyObject* h;
    if (o == Py_None) {
      if (of_current) {
        PyObject* d = PyObject_CallNoArgs(g_device);
        if (!d || PyLong_AsLong(d) != device) ok = false;
        Py_XDECREF(d);
        if (PyErr_Occurred()) PyErr_Clear();
        if (!ok) return nullptr;
      }
      PyObject* d = PyLong_FromLong(device);
      h = d ? PyObject_CallOneArg(g_raw_stream, d) : nullptr;
      Py_XDECREF(d);
    } else {
      h = PyObject_GetAttrString(o, "cuda_stream");
    }
    void* p = h ? PyLong_AsVoidPtr(h) : nullptr;
    Py_XDECREF(h);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return p;
  }
};

const at::ScalarType kBf = at::ScalarType::BFloat16, kI32 = at::ScalarType::Int;

// k_cache, v_cache [N, P, Hkv, D], block_table [B, M], context_lens [B].
struct Cache {
  const at::Tensor *k, *v, *bt, *lens;
  int64_t n = 0, p = 0, hkv = 0, d = 0, m = 0;
  Cache(Checker& c, PyObject* const* a, int64_t batch) {
    k = c.take(a[0], kBf, 4);
    v = c.take(a[1], kBf, 4);
    bt = c.take(a[2], kI32, 2);
    lens = c.take(a[3], kI32, 1);
    if (!c.ok) return;
    n = k->size(0), p = k->size(1), hkv = k->size(2), d = k->size(3), m = bt->size(1);
    c.ok = v->sizes() == k->sizes();
    c.same(bt->size(0), batch);
    c.same(lens->size(0), batch);
  }
};

int32_t* ints(const at::Tensor* t) { return static_cast<int32_t*>(t->data_ptr()); }

// Runs one call's body, which returns the status (or kDeclined); nothing a
// tensor throws (one without storage, say) leaves this file.
template <class F>
PyObject* guarded(Py_ssize_t nargs, Py_ssize_t want, F body) {
  int rc = kDeclined;
  if (nargs == want) {
    try {
      rc = body();
    } catch (...) {
      PyErr_Clear();
      rc = kDeclined;
    }
  }
  return PyLong_FromLong(rc);
}

template <class F>
int released(F call) {  // the library call without the interpreter lock, as ctypes makes it
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return rc;
}

// (q, k, v, bt, lens, out, scale, window, stream, noalloc); q [B, Hq, D], or
// [B, T, Hq, D] with a window argument that is not None
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return guarded(nargs, 10, [&]() -> int {
    Checker c;
    const bool ext = a[7] != Py_None;
    const at::Tensor* q = c.take(a[0], kBf, ext ? 4 : 3);
    if (!c.ok) return kDeclined;
    Cache kv(c, a + 1, q->size(0));
    const at::Tensor* out = c.take(a[5], kBf, ext ? 4 : 3);
    if (!c.ok) return kDeclined;
    c.ok = out->sizes() == q->sizes();
    const int32_t b = c.i32(q->size(0)), t = ext ? c.i32(q->size(1)) : 1, hq = c.i32(q->size(ext ? 2 : 1));
    const int32_t d = c.i32(q->size(ext ? 3 : 2));
    c.same(kv.d, d);
    const int32_t hkv = c.i32(kv.hkv), p = c.i32(kv.p), n = c.i32(kv.n), m = c.i32(kv.m);
    const int32_t window = ext ? c.integer(a[7]) : 0;
    const float scale = c.number(a[6]);
    void* st = c.stream(a[8], /*of_current=*/ext);
    if (!c.ok) return kDeclined;
    void *qp = q->data_ptr(), *kp = kv.k->data_ptr(), *vp = kv.v->data_ptr(), *op = out->data_ptr();
    int32_t *bp = ints(kv.bt), *lp = ints(kv.lens);
    if (a[9] == Py_True)
      return released([&] { return g_lib.attention_noalloc(qp, kp, vp, bp, lp, op, b, hq, hkv, d, p, n, m, scale, st); });
    return released([&] { return g_lib.attention_ext(qp, kp, vp, bp, lp, op, b, hq, hkv, d, p, n, m, t, window, scale, st); });
  });
}

// (k_new, v_new, k, v, bt, lens, several, stream); k_new [B, Hkv, D], or
// [B, T, Hkv, D] where `several` is True
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return guarded(nargs, 8, [&]() -> int {
    Checker c;
    const bool several = a[6] == Py_True;
    const at::Tensor* kn = c.take(a[0], kBf, several ? 4 : 3);
    const at::Tensor* vn = c.take(a[1], kBf, several ? 4 : 3);
    if (!c.ok) return kDeclined;
    Cache kv(c, a + 2, kn->size(0));
    if (!c.ok) return kDeclined;
    c.ok = vn->sizes() == kn->sizes();
    const int32_t b = c.i32(kn->size(0)), t = several ? c.i32(kn->size(1)) : 1;
    c.same(kn->size(several ? 2 : 1), kv.hkv);
    c.same(kn->size(several ? 3 : 2), kv.d);
    const int32_t hkv = c.i32(kv.hkv), d = c.i32(kv.d), p = c.i32(kv.p), n = c.i32(kv.n), m = c.i32(kv.m);
    void* st = c.stream(a[7], /*of_current=*/true);
    if (!c.ok) return kDeclined;
    void *knp = kn->data_ptr(), *vnp = vn->data_ptr(), *kp = kv.k->data_ptr(), *vp = kv.v->data_ptr();
    int32_t *bp = ints(kv.bt), *lp = ints(kv.lens);
    return released([&] { return g_lib.kv_append_n(knp, vnp, kp, vp, bp, lp, b, t, hkv, d, p, n, m, st); });
  });
}

// (q, k_new, v_new, k, v, bt, lens, out, scale, stream)
PyObject* attention_append(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return guarded(nargs, 10, [&]() -> int {
    Checker c;
    const at::Tensor* q = c.take(a[0], kBf, 3);
    const at::Tensor* kn = c.take(a[1], kBf, 3);
    const at::Tensor* vn = c.take(a[2], kBf, 3);
    if (!c.ok) return kDeclined;
    Cache kv(c, a + 3, q->size(0));
    const at::Tensor* out = c.take(a[7], kBf, 3);
    if (!c.ok) return kDeclined;
    c.ok = out->sizes() == q->sizes() && vn->sizes() == kn->sizes();
    c.same(kn->size(0), q->size(0));
    c.same(kn->size(1), kv.hkv);
    c.same(kn->size(2), q->size(2));
    c.same(kv.d, q->size(2));
    const int32_t b = c.i32(q->size(0)), hq = c.i32(q->size(1)), d = c.i32(q->size(2));
    const int32_t hkv = c.i32(kv.hkv), p = c.i32(kv.p), n = c.i32(kv.n), m = c.i32(kv.m);
    const float scale = c.number(a[8]);
    void* st = c.stream(a[9], /*of_current=*/true);
    if (!c.ok) return kDeclined;
    void *qp = q->data_ptr(), *knp = kn->data_ptr(), *vnp = vn->data_ptr();
    void *kp = kv.k->data_ptr(), *vp = kv.v->data_ptr(), *op = out->data_ptr();
    int32_t *bp = ints(kv.bt), *lp = ints(kv.lens);
    return released([&] { return g_lib.attention_append(qp, knp, vnp, kp, vp, bp, lp, op, b, hq, hkv, d, p, n, m, scale, st); });
  });
}

// (x, w_packed, lens, q_out, k, v, block_table or None, num_q_heads,
//  num_kv_heads, head_dim, rope_theta, rotary_dim, interleaved, bias, q_norm,
//  k_norm, eps, stream); k, v are the outputs, or with a block table the caches
PyObject* prelude(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return guarded(nargs, 18, [&]() -> int {
    Checker c;
    const bool append = a[6] != Py_None;
    const at::Tensor* x = c.take(a[0], kBf, 2);
    const at::Tensor* w = c.take(a[1], kBf, 2);
    const at::Tensor* lens = c.take(a[2], kI32, 1);
    const at::Tensor* q = c.take(a[3], kBf, 3);
    const at::Tensor* k = c.take(a[4], kBf, append ? 4 : 3);
    const at::Tensor* v = c.take(a[5], kBf, append ? 4 : 3);
    const at::Tensor* bt = append ? c.take(a[6], kI32, 2) : nullptr;
    const at::Tensor* bias = a[13] != Py_None ? c.take(a[13], kBf, 1) : nullptr;
    const at::Tensor* qn = a[14] != Py_None ? c.take(a[14], kBf, 1) : nullptr;
    const at::Tensor* kn = a[15] != Py_None ? c.take(a[15], kBf, 1) : nullptr;
    pda_prelude_dims dm;
    dm.num_q_heads = c.integer(a[7]);
    dm.num_kv_heads = c.integer(a[8]);
    dm.head_dim = c.integer(a[9]);
    dm.rope_theta = c.number(a[10]);
    dm.rotary_dim = a[11] == Py_None ? dm.head_dim : c.integer(a[11]);
    if (a[12] != Py_True && a[12] != Py_False) c.ok = false;
    dm.interleaved = a[12] == Py_True;
    dm.eps = c.number(a[16]);
    if (!c.ok || (qn == nullptr) != (kn == nullptr)) return kDeclined;
    const int64_t hq = dm.num_q_heads, hkv = dm.num_kv_heads, d = dm.head_dim, rows = (hq + 2 * hkv) * d;
    dm.batch = c.i32(x->size(0));
    dm.hidden = c.i32(x->size(1));
    c.same(w->size(0), rows);
    c.same(w->size(1), x->size(1));
    c.same(lens->size(0), x->size(0));
    c.same(q->size(0), x->size(0));
    c.same(q->size(1), hq);
    c.same(q->size(2), d);
    c.ok = c.ok && k->sizes() == v->sizes();
    c.same(k->size(append ? 2 : 1), hkv);
    c.same(k->size(append ? 3 : 2), d);
    if (append)
      c.same(bt->size(0), x->size(0));
    else
      c.same(k->size(0), x->size(0));
    if (bias) c.same(bias->size(0), rows);
    if (qn) c.same(qn->size(0), d), c.same(kn->size(0), d);
    const int32_t pages = append ? c.i32(k->size(0)) : 0, page = append ? c.i32(k->size(1)) : 0;
    const int32_t m = append ? c.i32(bt->size(1)) : 0;
    void* st = c.stream(a[17], /*of_current=*/true);
    if (!c.ok) return kDeclined;
    auto ptr = [](const at::Tensor* t) -> void* { return t ? t->data_ptr() : nullptr; };
    void *xp = ptr(x), *wp = ptr(w), *bp = ptr(bias), *qnp = ptr(qn), *knp = ptr(kn), *qp = ptr(q), *kp = ptr(k), *vp = ptr(v);
    int32_t *lp = ints(lens), *tp = append ? ints(bt) : nullptr;
    if (append)
      return released([&] { return g_lib.prelude_append(xp, wp, bp, qnp, knp, lp, qp, kp, vp, tp, page, pages, m, &dm, st); });
    return released([&] { return g_lib.prelude(xp, wp, bp, qnp, knp, lp, qp, kp, vp, &dm, st); });
  });
}

// (attn, w_packed, residual, norm_w, residual_out, normed_out, eps, stream)
PyObject* o_proj(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return guarded(nargs, 8, [&]() -> int {
    Checker c;
    const at::Tensor* x = c.take(a[0], kBf, 2);
    const at::Tensor* w = c.take(a[1], kBf, 2);
    const at::Tensor* res = c.take(a[2], kBf, 2);
    const at::Tensor* nw = c.take(a[3], kBf, 1);
    const at::Tensor* z = c.take(a[4], kBf, 2);
    const at::Tensor* h = c.take(a[5], kBf, 2);
    const float eps = c.number(a[6]);
    if (!c.ok) return kDeclined;
    const int32_t b = c.i32(x->size(0)), k = c.i32(x->size(1)), n = c.i32(w->size(0));
    c.same(w->size(1), x->size(1));
    c.same(res->size(0), x->size(0));
    c.same(res->size(1), w->size(0));
    c.same(nw->size(0), w->size(0));
    c.ok = c.ok && z->sizes() == res->sizes() && h->sizes() == res->sizes();
    void* st = c.stream(a[7], /*of_current=*/true);
    if (!c.ok) return kDeclined;
    void *xp = x->data_ptr(), *wp = w->data_ptr(), *rp = res->data_ptr(), *np = nw->data_ptr();
    void *zp = z->data_ptr(), *hp = h->data_ptr();
    return released([&] { return g_lib.o_proj(xp, wp, rp, np, zp, hp, b, k, n, eps, st); });
  });
}

// ({name: address}, raw_stream, device): the loaded library's entry points,
// torch's current raw stream of a device and its current device
PyObject* init(PyObject*, PyObject* args) {
  PyObject *table, *raw, *device;
  if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &table, &raw, &device)) return nullptr;
  auto set = [&](const char* name, auto& fn) {
    PyObject* v = PyDict_GetItemString(table, name);
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
    if (!p) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address for %s", name);
      return false;
    }
    fn = reinterpret_cast<typename std::remove_reference<decltype(fn)>::type>(p);
    return true;
  };
  if (!set("paged_decode_attention_ext", g_lib.attention_ext) ||
      !set("paged_decode_attention_noalloc", g_lib.attention_noalloc) ||
      !set("paged_decode_attention_append", g_lib.attention_append) || !set("pda_kv_append_n", g_lib.kv_append_n) ||
      !set("pda_attention_prelude", g_lib.prelude) ||
      !set("pda_attention_prelude_append", g_lib.prelude_append) ||
      !set("pda_o_proj_residual_norm", g_lib.o_proj))
    return nullptr;
  Py_INCREF(raw);
  Py_XDECREF(g_raw_stream);
  g_raw_stream = raw;
  Py_INCREF(device);
  Py_XDECREF(g_device);
  g_device = device;
  Py_RETURN_NONE;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {FAST(attention), FAST(kv_append), FAST(attention_append), FAST(prelude), FAST(o_proj),
                          {"init", init, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "pda_native", "Native marshalling of the binding's hot calls.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_pda_native() {
  PyObject* m = PyModule_Create(&kModule);
  if (m && PyModule_AddStringConstant(m, "built_for", PDA_BUILT_FOR) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
