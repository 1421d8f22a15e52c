// Argument marshalling of binding.py's calls in native code: a call of the Python layer checks up to fifteen tensors (device,
// contiguous, type, shape) and takes their addresses, which at 0.5 us a tensor was two thirds of the host time of a small pass.  Host
// time of a pass, Python / this: forward of six calls 57 / 21 us, training step of eleven 118 / 43 us, of which 20 and 38 are the launches
// (on another host 62 / 28 and 129 / 61).
//
// Only calls that pass every check are made here.  Whatever is unusual -- another type of argument, a tensor subclass, a wrapped tensor, a
// shape that does not fit -- returns NOT_TAKEN before anything is enqueued, and binding.py's own checks say what is wrong, or accept it.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>

#include <cstring>
#include <initializer_list>
#include <optional>
#include <utility>

#include "../../include/moe.h"

namespace {

constexpr int NOT_TAKEN = -1;

// the library's entry points, by address: whichever library binding.py has loaded
struct Entry {
  decltype(&moe_route) route;
  decltype(&moe_dispatch) dispatch;
  decltype(&moe_dispatch_static) dispatch_static;
  decltype(&moe_expert_fwd) expert_fwd;
  decltype(&moe_expert_bwd) expert_bwd;
  decltype(&moe_combine) combine;
  decltype(&moe_router_fwd) router_fwd;
  decltype(&moe_combine_bwd) combine_bwd;
  decltype(&moe_gate_bwd) gate_bwd;
  decltype(&moe_router_bwd) router_bwd;
} entry;
constexpr int N_ENTRIES = sizeof(Entry) / sizeof(void*);

struct NotTaken {};
[[noreturn]] void refuse() { throw NotTaken(); }

// Arguments in order.
struct Args {
  PyObject* const* v;
  Py_ssize_t n, at = 0;
  PyObject* next() {
    if (at >= n) refuse();
    return v[at++];
  }
  int integer() {
    PyObject* o = next();
    if (!PyLong_Check(o)) refuse();
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over || x < INT32_MIN || x > INT32_MAX) refuse();
    return (int)x;
  }
  int flag() {
    PyObject* o = next();
    if (o == Py_True) return 1;
    if (o == Py_False) return 0;
    --at;
    return integer();
  }
};

struct Buf {                               // a tensor, or nothing
  const at::Tensor* t = nullptr;
  void* ptr = nullptr;
  int64_t size(int i) const { return t->size(i); }
  int64_t bytes() const { return t ? t->numel() * (int64_t)t->element_size() : 0; }
};

Buf any(Args& a, bool optional = false) {
  PyObject* o = a.next();
  if (o == Py_None && optional) return {};
  if (!THPVariable_CheckExact(o)) refuse();
  Buf b;
  b.t = &THPVariable_Unpack(o);
  if (!b.t->is_cuda() || !b.t->is_contiguous()) refuse();
  b.ptr = b.t->data_ptr();                 // (throws for a tensor without storage)
  return b;
}
Buf typed(Args& a, at::ScalarType type, bool optional = false) {
  const Buf b = any(a, optional);
  if (b.t && b.t->scalar_type() != type) refuse();
  return b;
}
const Buf& shaped(const Buf& b, std::initializer_list<int64_t> shape) {
  if (b.t && b.t->sizes() != at::IntArrayRef(shape)) refuse();
  return b;
}
void dims(const Buf& b, int64_t n) {
  if (b.t->dim() != n) refuse();
}
int small(int64_t v) {
  if (v < 0 || v > INT32_MAX) refuse();
  return (int)v;
}
int dtype_code(const Buf& b) {
  if (b.t->scalar_type() == at::kFloat) return MOE_F32;
  if (b.t->scalar_type() == at::kBFloat16) return MOE_BF16;
  refuse();
}
moe_stream_t stream() { return (moe_stream_t)c10::hip::getCurrentHIPStream().stream(); }

constexpr auto F32 = at::kFloat;
constexpr auto I32 = at::kInt;

// f(args) marshals and returns the call to make; the interpreter's lock is not held while it enqueues.  Only marshalling may end in "not
// taken": the call itself is made once, and what it might throw leaves as it would leave ctypes.
template <typename F>
PyObject* take(PyObject* const* v, Py_ssize_t n, F f) {
  std::optional<decltype(f(std::declval<Args&>()))> call;
  try {
    Args a{v, n};
    auto made = f(a);
    if (a.at != n) refuse();
    call.emplace(std::move(made));
  } catch (...) {
    PyErr_Clear();
    return PyLong_FromLong(NOT_TAKEN);
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = (*call)();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

PyObject* route(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf logits = typed(a, F32);
    dims(logits, 2);
    const int k = a.integer(), mode = a.integer(), e_lo = a.integer(), e_cnt = a.integer();
    const Buf idx = typed(a, I32), w = typed(a, F32), counts = typed(a, I32);
    const int T = small(logits.size(0)), E = small(logits.size(1));
    shaped(idx, {T, k});
    shaped(w, {T, k});
    shaped(counts, {e_cnt});
    return [=, s = stream()] {
      return entry.route((const float*)logits.ptr, T, E, k, mode, e_lo, e_cnt, (int32_t*)idx.ptr, (float*)w.ptr, (int32_t*)counts.ptr, s);
    };
  });
}

struct Plan {
  Buf x, idx, scale, offsets, perm, inv, xp;
  int T, d, k, e_lo, e_cnt, cap, dt;
  Plan(Args& a) {
    x = any(a);
    dims(x, 2);
    k = a.integer();
    idx = typed(a, I32, true);
    scale = typed(a, F32, true);
    e_lo = a.integer();
    e_cnt = a.integer();
    offsets = typed(a, I32);
    perm = typed(a, I32);
    inv = typed(a, I32);
    T = small(x.size(0));
    d = small(x.size(1));
    dt = dtype_code(x);
    shaped(idx, {T, k});
    shaped(scale, {T, k});
    shaped(offsets, {(int64_t)e_cnt + 1});
    shaped(inv, {T, k});
  }
  void rows(Args& a) {
    xp = typed(a, x.t->scalar_type());
    dims(xp, 2);
    cap = small(xp.size(0));
    shaped(xp, {cap, d});
    shaped(perm, {cap});
  }
};

PyObject* dispatch(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    Plan p(a);
    const int reuse = a.flag();
    p.rows(a);
    const Buf ws = any(a, true);
    const size_t ws_bytes = (size_t)ws.bytes();
    return [=, s = stream()] {
      return entry.dispatch(p.x.ptr, p.dt, p.T, p.d, p.k, (const int32_t*)p.idx.ptr, (const float*)p.scale.ptr, p.e_lo, p.e_cnt,
                            (int32_t*)p.offsets.ptr, (int32_t*)p.perm.ptr, (int32_t*)p.inv.ptr, reuse, p.xp.ptr, p.cap, ws.ptr, ws_bytes, s);
    };
  });
}

PyObject* dispatch_static(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    Plan p(a);
    p.rows(a);
    const Buf status = typed(a, I32, true);
    return [=, s = stream()] {
      return entry.dispatch_static(p.x.ptr, p.dt, p.T, p.d, p.k, (const int32_t*)p.idx.ptr, (const float*)p.scale.ptr, p.e_lo, p.e_cnt,
                                   (int32_t*)p.offsets.ptr, (int32_t*)p.perm.ptr, (int32_t*)p.inv.ptr, p.xp.ptr, p.cap, (int32_t*)status.ptr, s);
    };
  });
}

PyObject* expert_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf xp = any(a), off = typed(a, I32);
    const auto t = xp.t->scalar_type();
    const Buf w1 = typed(a, t), w3 = typed(a, t), w2 = typed(a, t), h1 = typed(a, t, true), h3 = typed(a, t, true), o = typed(a, t), ws = any(a),
              act = typed(a, t, true);
    dims(xp, 2);
    dims(w1, 3);
    const int cap = small(xp.size(0)), d = small(xp.size(1)), e = small(w1.size(0)), f = small(w1.size(2)), dt = dtype_code(xp);
    shaped(o, {cap, d});
    shaped(w1, {e, d, f});
    shaped(w3, {e, d, f});
    shaped(w2, {e, f, d});
    shaped(h1, {cap, f});
    shaped(h3, {cap, f});
    shaped(act, {cap, f});
    shaped(off, {(int64_t)e + 1});
    const size_t ws_bytes = (size_t)ws.bytes();
    return [=, s = stream()] {
      return entry.expert_fwd(xp.ptr, dt, cap, d, f, e, (const int32_t*)off.ptr, w1.ptr, w3.ptr, w2.ptr, h1.ptr, h3.ptr, act.ptr, o.ptr, ws.ptr,
                              ws_bytes, s);
    };
  });
}

PyObject* expert_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf xp = any(a);
    const auto t = xp.t->scalar_type();
    const Buf h1 = typed(a, t), h3 = typed(a, t), d_o = typed(a, t), off = typed(a, I32), w1 = typed(a, t), w3 = typed(a, t), w2 = typed(a, t),
              dxp = typed(a, t), dw1 = typed(a, t), dw3 = typed(a, t), dw2 = typed(a, t);
    const int accumulate = a.flag();
    const Buf ws = any(a), act = typed(a, t, true);
    dims(xp, 2);
    dims(w1, 3);
    const int cap = small(xp.size(0)), d = small(xp.size(1)), e = small(w1.size(0)), f = small(w1.size(2)), dt = dtype_code(xp);
    for (const Buf* b : {&h1, &h3, &act}) shaped(*b, {cap, f});
    for (const Buf* b : {&d_o, &dxp}) shaped(*b, {cap, d});
    for (const Buf* b : {&w1, &w3, &dw1, &dw3}) shaped(*b, {e, d, f});
    for (const Buf* b : {&w2, &dw2}) shaped(*b, {e, f, d});
    shaped(off, {(int64_t)e + 1});
    const size_t ws_bytes = (size_t)ws.bytes();
    return [=, s = stream()] {
      return entry.expert_bwd(xp.ptr, h1.ptr, h3.ptr, act.ptr, d_o.ptr, dt, cap, d, f, e, (const int32_t*)off.ptr, w1.ptr, w3.ptr, w2.ptr, dxp.ptr,
                              dw1.ptr, dw3.ptr, dw2.ptr, accumulate, ws.ptr, ws_bytes, s);
    };
  });
}

PyObject* combine(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf o = any(a), inv = typed(a, I32), w = typed(a, F32, true), y = typed(a, o.t->scalar_type());
    dims(o, 2);
    dims(inv, 2);
    const int T = small(inv.size(0)), k = small(inv.size(1)), d = small(o.size(1)), dt = dtype_code(o);
    shaped(y, {T, d});
    shaped(w, {T, k});
    return [=, s = stream()] { return entry.combine(o.ptr, dt, T, d, k, (const int32_t*)inv.ptr, (const float*)w.ptr, y.ptr, s); };
  });
}

PyObject* router_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf x = any(a), wr = typed(a, x.t->scalar_type()), logits = typed(a, F32), ws = any(a);
    dims(x, 2);
    dims(wr, 2);
    const int T = small(x.size(0)), d = small(x.size(1)), E = small(wr.size(1)), dt = dtype_code(x);
    shaped(wr, {d, E});
    shaped(logits, {T, E});
    const size_t ws_bytes = (size_t)ws.bytes();
    return [=, s = stream()] { return entry.router_fwd(x.ptr, wr.ptr, dt, T, d, E, (float*)logits.ptr, ws.ptr, ws_bytes, s); };
  });
}

PyObject* combine_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf dy = any(a);
    const auto t = dy.t->scalar_type();
    const Buf o = typed(a, t), inv = typed(a, I32), w = typed(a, F32), d_o = typed(a, t), dgate = typed(a, F32);
    dims(dy, 2);
    dims(o, 2);
    dims(inv, 2);
    const int T = small(inv.size(0)), k = small(inv.size(1)), d = small(dy.size(1)), dt = dtype_code(dy);
    shaped(dy, {T, d});
    shaped(o, {o.size(0), d});
    shaped(d_o, {o.size(0), d});
    shaped(w, {T, k});
    shaped(dgate, {T, k});
    return [=, s = stream()] {
      return entry.combine_bwd(dy.ptr, o.ptr, dt, T, d, k, (const int32_t*)inv.ptr, (const float*)w.ptr, d_o.ptr, (float*)dgate.ptr, s);
    };
  });
}

PyObject* gate_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf logits = typed(a, F32), idx = typed(a, I32), dgate = typed(a, F32);
    const int mode = a.integer();
    const Buf dl = typed(a, F32);
    dims(logits, 2);
    dims(idx, 2);
    const int T = small(logits.size(0)), E = small(logits.size(1)), k = small(idx.size(1));
    shaped(idx, {T, k});
    shaped(dgate, {T, k});
    shaped(dl, {T, E});
    return [=, s = stream()] {
      return entry.gate_bwd((const float*)logits.ptr, (const int32_t*)idx.ptr, (const float*)dgate.ptr, T, E, k, mode, (float*)dl.ptr, s);
    };
  });
}

PyObject* router_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return take(v, n, [](Args& a) {
    const Buf x = any(a);
    const auto t = x.t->scalar_type();
    const Buf wr = typed(a, t), dl = typed(a, F32), dwr = typed(a, t, true);
    const int dwr_acc = a.flag();
    const Buf dx = typed(a, t, true);
    const int dx_acc = a.flag();
    const Buf ws = any(a);
    dims(x, 2);
    dims(wr, 2);
    const int T = small(x.size(0)), d = small(x.size(1)), E = small(wr.size(1)), dt = dtype_code(x);
    shaped(wr, {d, E});
    shaped(dl, {T, E});
    shaped(dwr, {d, E});
    shaped(dx, {T, d});
    const size_t ws_bytes = (size_t)ws.bytes();
    return [=, s = stream()] {
      return entry.router_bwd(x.ptr, wr.ptr, (const float*)dl.ptr, dt, T, d, E, dwr.ptr, dwr_acc, dx.ptr, dx_acc, ws.ptr, ws_bytes, s);
    };
  });
}

// bind(addresses): the entry points in the order of Entry
PyObject* bind(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != N_ENTRIES) {
    PyErr_SetString(PyExc_TypeError, "one address per entry point");
    return nullptr;
  }
  void* at[N_ENTRIES];
  for (int i = 0; i < N_ENTRIES; ++i) {
    at[i] = PyLong_AsVoidPtr(v[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  static_assert(sizeof(at) == sizeof(entry), "");
  memcpy(&entry, at, sizeof(at));
  Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(route),    METHOD(dispatch),   METHOD(dispatch_static), METHOD(expert_fwd), METHOD(expert_bwd), METHOD(combine),
                         METHOD(router_fwd), METHOD(combine_bwd), METHOD(gate_bwd),      METHOD(router_bwd), METHOD(bind),       {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
