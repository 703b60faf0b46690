// Native half of the Python binding: takes a call's arguments straight from
// the interpreter (torch tensors, ints, the ctypes Group and Plan), makes the
// same checks as the Python half and enqueues the call.  A call that fails a
// check, or whose arguments are of any other type, returns None with nothing
// enqueued; the Python half then handles it and raises its errors.
//
// A step is five calls of up to twelve arguments; checked and marshalled in
// Python each takes 5-8 us of host time, which is most of a small step:
// enqueueing the tiny workload's step (8 kernels) takes 53 us through the Python
// half and 25 us through this file.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/ultraep.h"

namespace {

typedef __int128 wide;  // products of caller-given sizes

#define ENTRIES(X)                                                                           \
  X(count) X(plan) X(plan_noalloc) X(plan_replicate) X(plan_reroute) X(dispatch)             \
  X(dispatch_layout) X(dispatch_scatter) X(pack_replicas) X(reroute_and_pack) X(relay_plan)  \
  X(pack_relay) X(combine) X(grad_reduce)

struct Library {
#define FIELD(n) decltype(&ultraep_##n) n = nullptr;
  ENTRIES(FIELD)
#undef FIELD
} lib;
PyObject *t_group, *t_plan, *t_buf;       // Group, Plan, PlanBuf
PyObject *s_c, *s_ws, *s_cuda_stream;     // attribute names

// The arguments of one call, in order; ok turns false at the first one that
// the native half does not take.
struct Args {
  PyObject *const *a;
  bool ok = true;
  // What the call uses beyond its arguments (a Plan's descriptor and its
  // workspace), held until the call has been enqueued: another thread may give
  // the Plan other ones while the interpreter lock is released.
  PyObject *held[2];
  int n_held = 0;

  explicit Args(PyObject *const *argv) : a(argv) {}
  Args(const Args &) = delete;
  Args &operator=(const Args &) = delete;
  ~Args() {
    for (int i = 0; i < n_held; ++i) Py_DECREF(held[i]);
  }
  // takes over a new reference
  PyObject *hold(PyObject *o) { return held[n_held++] = o; }

  PyObject *fail() {
    ok = false;
    return nullptr;
  }
  // an int (exactly) within [lo, hi]
  int64_t integer(int i, int64_t lo, int64_t hi) {
    if (!ok || !PyLong_CheckExact(a[i])) return fail(), 0;
    int over = 0;
    const int64_t v = PyLong_AsLongLongAndOverflow(a[i], &over);
    if (over || v < lo || v > hi) return fail(), 0;
    return v;
  }
  int32_t i32(int i) { return static_cast<int32_t>(integer(i, INT32_MIN, INT32_MAX)); }
  int64_t i64(int i) { return integer(i, INT64_MIN, INT64_MAX); }

  // a contiguous device tensor of at least n elements of esize bytes (any, or
  // None, if n <= 0); null for an empty one
  template <class T = void>
  T *tensor(PyObject *o, wide n, int64_t esize) {
    if (!ok) return nullptr;
    if (o == Py_None) return n > 0 ? (fail(), nullptr) : nullptr;
    if (!THPVariable_CheckExact(o)) return fail(), nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || !t.is_cuda() || !t.is_contiguous()) return fail(), nullptr;
    if (n > 0 && (static_cast<int64_t>(t.element_size()) != esize || t.numel() < n))
      return fail(), nullptr;
    return t.numel() ? static_cast<T *>(t.mutable_data_ptr()) : nullptr;
  }
  template <class T = void>
  T *tensor(int i, wide n) {
    return tensor<T>(ok ? a[i] : Py_None, n, sizeof(T));
  }

  // the memory of a ctypes structure of exactly type `type`
  void *structure(PyObject *o, PyObject *type, Py_ssize_t size) {
    if (!ok || reinterpret_cast<PyObject *>(Py_TYPE(o)) != type) return fail();
    Py_buffer v;
    if (PyObject_GetBuffer(o, &v, PyBUF_SIMPLE) != 0) return PyErr_Clear(), fail();
    void *p = v.len == size ? v.buf : nullptr;
    PyBuffer_Release(&v);
    return p ? p : fail();
  }
  const ultraep_group *group(int i) {
    auto *g = static_cast<const ultraep_group *>(structure(a[i], t_group, sizeof(ultraep_group)));
    if (g && (g->R < 1 || g->E < 1 || g->n_slot < 0)) return fail(), nullptr;
    return g;
  }
  PyObject *attr(PyObject *o, PyObject *name) {
    PyObject *v = ok ? PyObject_GetAttr(o, name) : nullptr;
    if (!v) return PyErr_Clear(), fail();
    return v;
  }
  const ultraep_plan_buf *plan(int i) {
    if (!ok || reinterpret_cast<PyObject *>(Py_TYPE(a[i])) != t_plan) return fail(), nullptr;
    PyObject *c = attr(a[i], s_c);
    if (!c) return nullptr;
    return static_cast<const ultraep_plan_buf *>(
        structure(hold(c), t_buf, sizeof(ultraep_plan_buf)));
  }
  // a workspace tensor (None: the plan's own) and its bytes
  void *workspace(int i, int plan_arg, size_t &bytes) {
    bytes = 0;
    if (!ok) return nullptr;
    PyObject *o = a[i];
    if (o == Py_None) {
      if (plan_arg < 0 || !(o = attr(a[plan_arg], s_ws))) return fail();
      if (hold(o) == Py_None) return fail();
    }
    void *p = tensor(o, 0, 0);
    if (ok) {
      const at::Tensor &t = THPVariable_Unpack(o);
      bytes = static_cast<size_t>(t.numel()) * t.element_size();
    }
    return p;
  }
  // torch's current stream for None, a torch stream, or an address
  hipStream_t stream(int i) {
    if (!ok) return nullptr;
    if (a[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *v = a[i];
    Py_INCREF(v);
    if (!PyLong_CheckExact(v)) {
      Py_DECREF(v);
      if (!(v = attr(a[i], s_cuda_stream))) return nullptr;
    }
    void *p = PyLong_CheckExact(v) ? PyLong_AsVoidPtr(v) : fail();
    if (PyErr_Occurred()) PyErr_Clear(), fail();
    Py_DECREF(v);
    return static_cast<hipStream_t>(p);
  }
};

int64_t slots(const ultraep_group *g) { return static_cast<int64_t>(g->R) * g->n_slot; }
int64_t blocks(const ultraep_group *g) {
  return static_cast<int64_t>(g->R) * (g->E / g->R + static_cast<int64_t>(g->n_slot)) + 1;
}
wide loads(const ultraep_group *g) { return wide(g->R) * g->E; }
wide mains(const ultraep_group *g) { return g->E / g->R; }

// None if an argument was not taken, else the entry point's return value
template <class F>
PyObject *finish(const Args &v, F call) {
  if (!v.ok) Py_RETURN_NONE;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

#define ENTRY(name, n_args, ...)                                                           \
  PyObject *py_##name(PyObject *, PyObject *const *argv, Py_ssize_t argc) {                \
    if (argc != n_args || !lib.name) Py_RETURN_NONE;                                       \
    try {                                                                                  \
      Args v{argv};                                                                        \
      __VA_ARGS__                                                                          \
    } catch (const std::exception &) {                                                     \
      Py_RETURN_NONE;                                                                      \
    }                                                                                      \
  }

// topk, T, k, E, n_groups, counts, status, stream
ENTRY(count, 8, {
  const int64_t T = v.i64(1);
  const int32_t k = v.i32(2), E = v.i32(3), n = v.i32(4);
  auto *topk = v.tensor<int32_t>(0, wide(n) * T * k);
  auto *counts = v.tensor<int32_t>(5, wide(n) * E);
  auto *status = v.tensor<int32_t>(6, 1);
  hipStream_t s = v.stream(7);
  return finish(v, [&] { return lib.count(topk, T, k, E, n, counts, status, s); });
})

// load, g, plan, ws, stream
ENTRY(plan, 5, {
  auto *g = v.group(1);
  auto *load = v.tensor<int32_t>(0, g ? loads(g) : 0);
  auto *p = v.plan(2);
  size_t bytes;
  void *ws = v.workspace(3, 2, bytes);
  hipStream_t s = v.stream(4);
  return finish(v, [&] { return lib.plan(load, g, p, ws, bytes, s); });
})
ENTRY(plan_replicate, 5, {
  auto *g = v.group(1);
  auto *load = v.tensor<int32_t>(0, g ? loads(g) : 0);
  auto *p = v.plan(2);
  size_t bytes;
  void *ws = v.workspace(3, 2, bytes);
  hipStream_t s = v.stream(4);
  return finish(v, [&] { return lib.plan_replicate(load, g, p, ws, bytes, s); });
})

// load, g, plan, stream
ENTRY(plan_noalloc, 4, {
  auto *g = v.group(1);
  auto *load = v.tensor<int32_t>(0, g ? loads(g) : 0);
  auto *p = v.plan(2);
  hipStream_t s = v.stream(3);
  return finish(v, [&] { return lib.plan_noalloc(load, g, p, s); });
})
ENTRY(plan_reroute, 4, {
  auto *g = v.group(1);
  auto *load = v.tensor<int32_t>(0, g ? loads(g) : 0);
  auto *p = v.plan(2);
  hipStream_t s = v.stream(3);
  return finish(v, [&] { return lib.plan_reroute(load, g, p, s); });
})

// x, topk, T, k, H, rank, g, plan, send, row_of_slot, block_off, ws, status, stream
ENTRY(dispatch, 14, {
  const int64_t T = v.i64(2);
  const int32_t k = v.i32(3), H = v.i32(4), rank = v.i32(5);
  auto *g = v.group(6);
  auto *p = v.plan(7);
  auto *x = v.tensor<uint16_t>(0, wide(T) * H);
  auto *send = v.tensor<uint16_t>(8, wide(T) * k * H);
  auto *topk = v.tensor<int32_t>(1, wide(T) * k);
  auto *ros = v.tensor<int32_t>(9, wide(T) * k);
  auto *off = v.tensor<int64_t>(10, g ? blocks(g) : 0);
  size_t bytes;
  void *ws = v.workspace(11, -1, bytes);
  auto *status = v.tensor<int32_t>(12, 1);
  hipStream_t s = v.stream(13);
  return finish(v, [&] {
    return lib.dispatch(x, topk, T, k, H, rank, g, p, send, ros, off, ws, bytes, status, s);
  });
})

// topk, T, k, rank, g, plan, row_of_slot, block_off, ws, status, stream
ENTRY(dispatch_layout, 11, {
  const int64_t T = v.i64(1);
  const int32_t k = v.i32(2), rank = v.i32(3);
  auto *g = v.group(4);
  auto *p = v.plan(5);
  auto *topk = v.tensor<int32_t>(0, wide(T) * k);
  auto *ros = v.tensor<int32_t>(6, wide(T) * k);
  auto *off = v.tensor<int64_t>(7, g ? blocks(g) : 0);
  size_t bytes;
  void *ws = v.workspace(8, -1, bytes);
  auto *status = v.tensor<int32_t>(9, 1);
  hipStream_t s = v.stream(10);
  return finish(v, [&] {
    return lib.dispatch_layout(topk, T, k, rank, g, p, ros, off, ws, bytes, status, s);
  });
})

// x, T, k, H, row_of_slot, n_routed, send, stream
ENTRY(dispatch_scatter, 8, {
  const int64_t T = v.i64(1);
  const int32_t k = v.i32(2), H = v.i32(3);
  auto *x = v.tensor<uint16_t>(0, wide(T) * H);
  auto *ros = v.tensor<int32_t>(4, wide(T) * k);
  auto *nr = v.tensor<int64_t>(5, T > 0 ? 1 : 0);
  auto *send = v.tensor<uint16_t>(6, wide(T) * k * H);
  hipStream_t s = v.stream(7);
  return finish(v, [&] { return lib.dispatch_scatter(x, T, k, H, ros, nr, send, s); });
})

// w_main, W, rank, g, plan, staging, cap, dest_off, status, stream
ENTRY(pack_replicas, 10, {
  const int64_t W = v.i64(1), cap = v.i64(6);
  const int32_t rank = v.i32(2);
  auto *g = v.group(3);
  auto *p = v.plan(4);
  auto *w = v.tensor<uint16_t>(0, g ? mains(g) * W : 0);
  auto *st = v.tensor<uint16_t>(5, wide(cap) * W);
  auto *off = v.tensor<int64_t>(7, g ? wide(g->R) + 1 : 0);
  auto *status = v.tensor<int32_t>(8, 1);
  hipStream_t s = v.stream(9);
  return finish(v, [&] { return lib.pack_replicas(w, W, rank, g, p, st, cap, off, status, s); });
})

// load, g, plan, w_main, W, rank, staging, cap, dest_off, status, stream
ENTRY(reroute_and_pack, 11, {
  const int64_t W = v.i64(4), cap = v.i64(7);
  const int32_t rank = v.i32(5);
  auto *g = v.group(1);
  auto *p = v.plan(2);
  auto *load = v.tensor<int32_t>(0, g ? loads(g) : 0);
  auto *w = v.tensor<uint16_t>(3, g ? mains(g) * W : 0);
  auto *st = v.tensor<uint16_t>(6, wide(cap) * W);
  auto *off = v.tensor<int64_t>(8, g ? wide(g->R) + 1 : 0);
  auto *status = v.tensor<int32_t>(9, 1);
  hipStream_t s = v.stream(10);
  return finish(v, [&] {
    return lib.reroute_and_pack(load, g, p, w, W, rank, st, cap, off, status, s);
  });
})

// g, plan, threshold, slot_src, send_vol, relay_stats, status, stream
ENTRY(relay_plan, 8, {
  auto *g = v.group(0);
  auto *p = v.plan(1);
  const int32_t threshold = v.i32(2);
  auto *src = v.tensor<int32_t>(3, g ? slots(g) : 0);
  auto *vol = v.tensor<int32_t>(4, g ? g->R : 0);
  auto *stats = v.tensor<int64_t>(5, 4);
  auto *status = v.tensor<int32_t>(6, 1);
  hipStream_t s = v.stream(7);
  return finish(v, [&] { return lib.relay_plan(g, p, threshold, src, vol, stats, status, s); });
})

// w_main, relay_src, W, rank, g, plan, slot_src, staging, cap, dest_off, status, stream
ENTRY(pack_relay, 12, {
  const int64_t W = v.i64(2), cap = v.i64(8);
  const int32_t rank = v.i32(3);
  auto *g = v.group(4);
  auto *p = v.plan(5);
  auto *w = v.tensor<uint16_t>(0, g ? mains(g) * W : 0);
  auto *st = v.tensor<uint16_t>(7, wide(cap) * W);
  auto *off = v.tensor<int64_t>(9, g ? wide(g->R) + 1 : 0);
  auto *status = v.tensor<int32_t>(10, 1);
  auto *rs = v.tensor<uint16_t>(1, g ? wide(g->n_slot) * W : 0);
  auto *src = v.tensor<int32_t>(6, g ? slots(g) : 0);
  hipStream_t s = v.stream(11);
  return finish(v, [&] {
    return lib.pack_relay(w, rs, W, rank, g, p, src, st, cap, off, status, s);
  });
})

// y, n_rows, gate, row_of_slot, T, k, H, out, status, stream
ENTRY(combine, 10, {
  const int64_t n_rows = v.i64(1), T = v.i64(4);
  const int32_t k = v.i32(5), H = v.i32(6);
  auto *y = v.tensor<uint16_t>(0, wide(n_rows) * H);
  auto *gate = v.tensor<float>(2, wide(T) * k);
  auto *ros = v.tensor<int32_t>(3, wide(T) * k);
  auto *out = v.tensor<uint16_t>(7, wide(T) * H);
  auto *status = v.tensor<int32_t>(8, 1);
  hipStream_t s = v.stream(9);
  return finish(v, [&] { return lib.combine(y, n_rows, gate, ros, T, k, H, out, status, s); });
})

// main_grad, rgrad, W, rank, g, plan, cap, status, stream
ENTRY(grad_reduce, 9, {
  const int64_t W = v.i64(2), cap = v.i64(6);
  const int32_t rank = v.i32(3);
  auto *g = v.group(4);
  auto *p = v.plan(5);
  auto *mg = v.tensor<float>(0, g ? mains(g) * W : 0);
  auto *rg = v.tensor<float>(1, wide(cap) * W);
  auto *status = v.tensor<int32_t>(7, 1);
  hipStream_t s = v.stream(8);
  return finish(v, [&] { return lib.grad_reduce(mg, rg, W, rank, g, p, cap, status, s); });
})

// bind({entry point: address}, Group, Plan, PlanBuf)
PyObject *py_bind(PyObject *, PyObject *args) {
  PyObject *d, *g, *p, *b;
  if (!PyArg_ParseTuple(args, "O!OOO", &PyDict_Type, &d, &g, &p, &b)) return nullptr;
#define SET(n)                                                                        \
  {                                                                                   \
    PyObject *v = PyDict_GetItemString(d, "ultraep_" #n);                             \
    lib.n = v ? reinterpret_cast<decltype(lib.n)>(PyLong_AsVoidPtr(v)) : nullptr;     \
    if (PyErr_Occurred()) return nullptr;                                             \
  }
  ENTRIES(SET)
#undef SET
  Py_INCREF(g);
  Py_INCREF(p);
  Py_INCREF(b);
  Py_XDECREF(t_group);
  Py_XDECREF(t_plan);
  Py_XDECREF(t_buf);
  t_group = g;
  t_plan = p;
  t_buf = b;
  Py_RETURN_NONE;
}

#define FAST(n)                                                                         \
  {                                                                                     \
    #n, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##n)),        \
        METH_FASTCALL, nullptr                                                          \
  }
PyMethodDef methods[] = {FAST(count), FAST(plan), FAST(plan_noalloc), FAST(plan_replicate),
                         FAST(plan_reroute), FAST(dispatch), FAST(dispatch_layout),
                         FAST(dispatch_scatter), FAST(pack_replicas), FAST(reroute_and_pack),
                         FAST(relay_plan), FAST(pack_relay), FAST(combine), FAST(grad_reduce),
                         {"bind", py_bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  s_c = PyUnicode_InternFromString("c");
  s_ws = PyUnicode_InternFromString("ws");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!s_c || !s_ws || !s_cuda_stream) return nullptr;
  PyObject *m = PyModule_Create(&module);
  // torch's C++ interface differs between versions: the Python half checks this
  if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_BUILD) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
