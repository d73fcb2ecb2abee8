// CPython entry points of the three calls of a decode step: the argument
// marshalling of _lib.py in native code for the ordinary case.
//
// What bounds a small call is the host: checking 14 tensors, allocating the
// outputs and a 25-argument ctypes call took ~16 us in Python (attention and
// the LM head of the tiny workload, 5 to 10 us of GPU time each).  Each
// function here returns None without having enqueued anything when an
// argument is not exactly what the call takes (another type, shape, layout or
// device, a tensor subclass, a sequence that is no int list or array); the
// caller then goes through the Python checks, which convert it or raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <cstdint>

#include "../../include/asynclane.h"

namespace {

// The library's entry points and the binding's Python helpers (set by init).
decltype(&::lane_attn_workspace_size) f_attn_ws;
decltype(&::lane_attn_forward) f_attn;
decltype(&::lmhead_confidence_workspace_size) f_lm_ws;
decltype(&::lmhead_packed_weight_size) f_lm_packed_size;
decltype(&::lmhead_confidence) f_lm;
decltype(&::lmhead_confidence_packed) f_lm_packed;
decltype(&::select_unmask) f_select;
PyObject *py_check, *py_workspace, *py_raw_stream;   // _check, _workspace, current raw stream

// Arguments as the library takes them.  What is not exactly that clears ok: the
// Python path takes the call.  (Not an exception: one costs ~2 us, and calls
// that always decline, such as those with an int64 parent array, pay it each time.)
struct Args {
  bool ok = true;
  template <class T>
  T no(T v) {
    ok = false;
    return v;
  }

  const at::Tensor* tensor(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) return no<const at::Tensor*>(nullptr);
    return &THPVariable_Unpack(o);
  }
  void* data(const at::Tensor* t, at::ScalarType dtype, int dev) {
    if (!t) return nullptr;
    if (!t->is_cuda() || t->get_device() != dev || t->layout() != at::kStrided || t->scalar_type() != dtype ||
        !t->is_contiguous())
      return no<void*>(nullptr);
    return t->data_ptr();
  }
  void* data3(const at::Tensor* t, at::ScalarType dtype, int dev, int64_t a, int64_t b, int64_t c) {
    if (!t || t->dim() != 3 || t->size(0) != a || t->size(1) != b || t->size(2) != c) return no<void*>(nullptr);
    return data(t, dtype, dev);
  }
  void* data2(const at::Tensor* t, at::ScalarType dtype, int dev, int64_t a, int64_t b) {
    if (t && (t->dim() != 2 || t->size(0) != a || t->size(1) != b)) return no<void*>(nullptr);
    return data(t, dtype, dev);
  }
  void* data_n(const at::Tensor* t, at::ScalarType dtype, int dev, int64_t least) {
    if (t && t->numel() < least) return no<void*>(nullptr);
    return data(t, dtype, dev);
  }

  int to_int(PyObject* o) {
    if (!PyLong_Check(o)) return no(0);
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) return no(0);
    return (int)v;
  }
  float to_float(PyObject* o) {
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return no(0.f);
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
      PyErr_Clear();
      return no(0.f);
    }
    return (float)v;
  }
  bool to_bool(PyObject* o) {
    if (!PyBool_Check(o)) return no(false);
    return o == Py_True;
  }

  // A host array of n entries of T: a contiguous one-dimensional buffer of that
  // type, or a list or tuple of ints (T = int32_t), copied to out.  (bytes have a
  // buffer too, but numpy takes them for text and refuses them.)
  template <class T>
  void host_array(PyObject* o, T* out, Py_ssize_t n) {
    if (sizeof(T) == 4 && (PyList_CheckExact(o) || PyTuple_CheckExact(o))) {
      if (PySequence_Fast_GET_SIZE(o) != n) ok = false;
      for (Py_ssize_t i = 0; ok && i < n; ++i) out[i] = (T)to_int(PySequence_Fast_GET_ITEM(o, i));
      return;
    }
    if (!PyObject_CheckBuffer(o) || PyBytes_Check(o) || THPVariable_Check(o)) {
      ok = false;
      return;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_FORMAT | PyBUF_ND | PyBUF_C_CONTIGUOUS) != 0) {
      PyErr_Clear();
      ok = false;
      return;
    }
    const char want = sizeof(T) == 4 ? 'i' : 'B';
    if (b.ndim == 1 && b.itemsize == (Py_ssize_t)sizeof(T) && b.format && b.format[0] == want && b.format[1] == 0 &&
        b.shape[0] == n)
      memcpy(out, b.buf, n * sizeof(T));
    else
      ok = false;
    PyBuffer_Release(&b);
  }
  // Token ids: a tuple or list of ints; returns the count.
  int id_set(PyObject* o, int32_t* out, int most) {
    if (!PyTuple_CheckExact(o) && !PyList_CheckExact(o)) return no(0);
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    if (n > most) return no(0);
    host_array(o, out, n);
    return (int)n;
  }

  void* stream_of(int dev) {
    PyObject* i = PyLong_FromLong(dev);
    PyObject* r = i ? PyObject_CallOneArg(py_raw_stream, i) : nullptr;
    Py_XDECREF(i);
    void* s = r ? PyLong_AsVoidPtr(r) : nullptr;
    Py_XDECREF(r);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return s;
  }
};

// Current device index; every tensor must be on it.
int current_device() { return c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice().index(); }

struct Error {};   // a Python exception is set

// The workspace of a call: the caller's tensor, or the binding's own buffer.
// *keep holds a reference for the duration of the call.
void* workspace(Args& g, PyObject* ws, const char* kind, size_t need, const at::Tensor& like, int dev, void* stream,
                size_t* bytes, PyObject** keep) {
  *keep = nullptr;
  *bytes = 0;
  const at::Tensor* t;
  if (ws != Py_None) {
    t = g.tensor(ws);
  } else {
    if (need == 0) return nullptr;
    PyObject* d = THPVariable_Wrap(like);
    PyObject* device = d ? PyObject_GetAttrString(d, "device") : nullptr;
    Py_XDECREF(d);
    PyObject* r = device ? PyObject_CallFunction(py_workspace, "snOn", kind, (Py_ssize_t)need, device,
                                                 (Py_ssize_t)(intptr_t)stream)
                         : nullptr;
    Py_XDECREF(device);
    if (!r) throw Error{};
    *keep = r;
    t = g.tensor(PyTuple_GET_ITEM(r, 0));
  }
  if (!t || !t->is_cuda() || t->get_device() != dev || !t->is_contiguous()) return g.no<void*>(nullptr);
  *bytes = t->nbytes();
  return t->data_ptr();
}

PyObject* wrap(const at::Tensor* given, PyObject* obj, const at::Tensor& made) {
  if (given) {
    Py_INCREF(obj);
    return obj;
  }
  if (made.defined()) return THPVariable_Wrap(made);
  Py_RETURN_NONE;
}

bool status_ok(int st, const char* what) {
  if (st == AL_OK) return true;
  PyObject* r = PyObject_CallFunction(py_check, "is", st, what);   // raises
  Py_XDECREF(r);
  return false;
}

PyObject* decline() { Py_RETURN_NONE; }

template <class F>
PyObject* guarded(F&& f) {
  PyObject* keep = nullptr;
  PyObject* r = nullptr;
  try {
    r = f(&keep);
  } catch (const Error&) {
  } catch (...) {   // a C++ error of torch: the Python path meets it again
    PyErr_Clear();
    r = decline();
  }
  Py_XDECREF(keep);
  return r;
}

// attn(q, k_lane, v_lane, k_prefix, v_prefix, parent, B, scale, refresh_idx,
//      q_ref, k_ref, v_ref, o, lse, o_ref, lse_ref, want_lse, workspace)
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&](PyObject** keep) -> PyObject* {
    if (na != 18) return decline();
    const auto bf16 = at::kBFloat16, f32 = at::kFloat;
    Args g;
    const at::Tensor *q = g.tensor(a[0]), *kl = g.tensor(a[1]), *vl = g.tensor(a[2]), *kp = g.tensor(a[3]),
                     *vp = g.tensor(a[4]), *ri = g.tensor(a[8]), *qr = g.tensor(a[9]), *kr = g.tensor(a[10]),
                     *vr = g.tensor(a[11]), *o = g.tensor(a[12]), *lse = g.tensor(a[13]), *o_r = g.tensor(a[14]),
                     *lse_r = g.tensor(a[15]);
    const bool want = g.to_bool(a[16]);
    const float scale = g.to_float(a[7]);
    if (!g.ok || !kp || kp->dim() != 3 || !kp->is_cuda()) return decline();
    int32_t parent[AL_MAX_LANES];
    const Py_ssize_t L = PyObject_Length(a[5]);
    if (L < 0) PyErr_Clear();
    if (L < 0 || L > AL_MAX_LANES) return decline();
    g.host_array(a[5], parent, L);
    if (!g.ok) return decline();
    const int dev = current_device();
    const int64_t P = kp->size(0), Hkv = kp->size(1), D = kp->size(2);
    void* kpp = g.data(kp, bf16, dev);
    void* vpp = g.data3(vp, bf16, dev, P, Hkv, D);
    int64_t n_ref = 0, Hq = 0;
    int B = 16;
    void *qp = nullptr, *klp = nullptr, *vlp = nullptr;
    at::Tensor mo, ml, mor, mlr;
    void *op = nullptr, *lp = nullptr, *orp = nullptr, *lrp = nullptr;
    if (ri) {
      if (ri->dim() != 1 || ri->size(0) == 0) return decline();
      n_ref = ri->size(0);
    }
    if (L > 0) {
      B = g.to_int(a[6]);
      if (!g.ok || !q || q->dim() != 3) return decline();
      const int64_t LB = (int64_t)L * B;
      Hq = q->size(1);
      qp = g.data3(q, bf16, dev, LB, Hq, D);
      klp = g.data3(kl, bf16, dev, LB, Hkv, D);
      vlp = g.data3(vl, bf16, dev, LB, Hkv, D);
      if (o) op = g.data3(o, bf16, dev, LB, Hq, D);
      lp = g.data2(lse, f32, dev, LB, Hq);
    } else {
      if (n_ref == 0 || !qr || qr->dim() != 3 || q || kl || vl || o || lse) return decline();
      Hq = qr->size(1);
    }
    void *rip = nullptr, *qrp = nullptr, *krp = nullptr, *vrp = nullptr;
    if (n_ref) {
      rip = g.data(ri, at::kInt, dev);
      qrp = g.data3(qr, bf16, dev, n_ref, Hq, D);
      krp = g.data3(kr, bf16, dev, n_ref, Hkv, D);
      vrp = g.data3(vr, bf16, dev, n_ref, Hkv, D);
      if (o_r) orp = g.data3(o_r, bf16, dev, n_ref, Hq, D);
      lrp = g.data2(lse_r, f32, dev, n_ref, Hq);
    } else if (qr || kr || vr || o_r || lse_r) {
      return decline();
    }
    if (P > INT32_MAX || Hkv > INT32_MAX || Hq > INT32_MAX || D > INT32_MAX || n_ref > INT32_MAX) return decline();
    if (!g.ok) return decline();
    void* stream = g.stream_of(dev);
    size_t bytes = 0;
    const size_t need = f_attn_ws((int)L, B, (int)P, (int)Hq, (int)Hkv, (int)D, (int)n_ref);
    void* ws = g.ok ? workspace(g, a[17], "attn", need, *kp, dev, stream, &bytes, keep) : nullptr;
    if (!g.ok) return decline();
    if (L > 0 && !o) {
      mo = at::empty({L * B, Hq, D}, q->options());
      op = mo.data_ptr();
    }
    if (L > 0 && !lse && want) {
      ml = at::empty({L * B, Hq}, kp->options().dtype(f32));
      lp = ml.data_ptr();
    }
    if (n_ref && !o_r) {
      mor = at::empty({n_ref, Hq, D}, qr->options());
      orp = mor.data_ptr();
    }
    if (n_ref && !lse_r && want) {
      mlr = at::empty({n_ref, Hq}, kp->options().dtype(f32));
      lrp = mlr.data_ptr();
    }
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f_attn((al_bf16*)qp, (al_bf16*)klp, (al_bf16*)vlp, (al_bf16*)kpp, (al_bf16*)vpp, L ? parent : nullptr, (int)L,
                B, (int)P, (int)Hq, (int)Hkv, (int)D, scale, (int32_t*)rip, (int)n_ref, (al_bf16*)qrp, (al_bf16*)krp,
                (al_bf16*)vrp, (al_bf16*)orp, (float*)lrp, (al_bf16*)op, (float*)lp, ws, bytes, stream);
    Py_END_ALLOW_THREADS
    if (!status_ok(st, "lane_attn_forward")) return nullptr;
    PyObject* t = PyTuple_New(4);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, wrap(o, a[12], mo));
    PyTuple_SET_ITEM(t, 1, wrap(lse, a[13], ml));
    PyTuple_SET_ITEM(t, 2, wrap(o_r, a[14], mor));
    PyTuple_SET_ITEM(t, 3, wrap(lse_r, a[15], mlr));
    return t;
  });
}

// lmhead(hidden, W, V or None, row_idx, suppress_eos, eos_id, conf, argmax,
//        lse, want_lse, workspace): V given = W is the packed copy.
PyObject* lmhead(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&](PyObject** keep) -> PyObject* {
    if (na != 11) return decline();
    Args g;
    const at::Tensor *h = g.tensor(a[0]), *W = g.tensor(a[1]), *ri = g.tensor(a[3]), *sup = g.tensor(a[4]),
                     *conf = g.tensor(a[6]), *arg = g.tensor(a[7]), *lse = g.tensor(a[8]);
    const int eos = g.to_int(a[5]);
    const bool want = g.to_bool(a[9]), packed = a[2] != Py_None;
    if (!g.ok || !h || !W || h->dim() != 2 || !h->is_cuda()) return decline();
    const int64_t n_rows = h->size(0), d = h->size(1);
    if (n_rows > INT32_MAX || d > INT32_MAX) return decline();
    int64_t V;
    if (packed) {
      V = g.to_int(a[2]);
      const size_t nb = g.ok ? f_lm_packed_size((int)d, (int)V) : 0;
      if (nb == 0 || W->numel() < (int64_t)(nb / 2)) return decline();
    } else {
      if (W->dim() != 2 || W->size(1) != d || W->size(0) > INT32_MAX) return decline();
      V = W->size(0);
    }
    int64_t N = n_rows;
    if (ri) {
      if (ri->dim() != 1) return decline();
      N = ri->size(0);
    }
    if (N == 0 || N > INT32_MAX) return decline();
    const int dev = current_device();
    void* hp = g.data(h, at::kBFloat16, dev);
    void* Wp = g.data(W, at::kBFloat16, dev);
    void* rp = g.data(ri, at::kInt, dev);
    void* sp = g.data_n(sup, at::kByte, dev, N);
    void* cp = g.data_n(conf, at::kFloat, dev, N);
    void* ap = g.data_n(arg, at::kInt, dev, N);
    void* lp = g.data_n(lse, at::kFloat, dev, N);
    if (!g.ok) return decline();
    void* stream = g.stream_of(dev);
    size_t bytes = 0;
    void* ws = g.ok ? workspace(g, a[10], "lmhead", f_lm_ws((int)N, (int)d, (int)V), *h, dev, stream, &bytes, keep) : nullptr;
    if (!g.ok) return decline();
    at::Tensor mc, ma, ml;
    const auto f32 = h->options().dtype(at::kFloat);
    if (!conf) {
      mc = at::empty({N}, f32);
      cp = mc.data_ptr();
    }
    if (!arg) {
      ma = at::empty({N}, h->options().dtype(at::kInt));
      ap = ma.data_ptr();
    }
    if (!lse && want) {
      ml = at::empty({N}, f32);
      lp = ml.data_ptr();
    }
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = (packed ? f_lm_packed : f_lm)((al_bf16*)hp, (int)n_rows, (int32_t*)rp, (int)N, (al_bf16*)Wp, (int)d, (int)V,
                                       (uint8_t*)sp, eos, (float*)cp, (int32_t*)ap, (float*)lp, ws, bytes, stream);
    Py_END_ALLOW_THREADS
    if (!status_ok(st, packed ? "lmhead_confidence_packed" : "lmhead_confidence")) return nullptr;
    PyObject* t = PyTuple_New(3);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, wrap(conf, a[6], mc));
    PyTuple_SET_ITEM(t, 1, wrap(arg, a[7], ma));
    PyTuple_SET_ITEM(t, 2, wrap(lse, a[8], ml));
    return t;
  });
}

const at::Tensor* item(Args& g, PyObject* dict, const char* key) {
  PyObject* o = PyDict_GetItemString(dict, key);
  return o ? g.tensor(o) : g.no<const at::Tensor*>(nullptr);
}

// select(conf, argmax, row_pos, tokens, is_masked, L, B, role, b_len, t_lane,
//        mode, tau, fallback_k, k_lane, delim_ids, eos_id, rho_min, t_min,
//        tau_future, out, digit_ids, open_ids, close_ids): True once enqueued
// (with the result buffers in the dict `out`).
PyObject* select(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&](PyObject**) -> PyObject* {
    if (na != 23 || !PyDict_CheckExact(a[19])) return decline();
    Args g;
    const at::Tensor *conf = g.tensor(a[0]), *arg = g.tensor(a[1]), *rp = g.tensor(a[2]), *tok = g.tensor(a[3]),
                     *msk = g.tensor(a[4]);
    const int L = g.to_int(a[5]), B = g.to_int(a[6]);
    if (!g.ok || !conf || !arg || !rp || !tok || !msk || rp->dim() != 1 || !tok->is_cuda()) return decline();
    if (L < 1 || L > AL_MAX_LANES || B < 1 || (int64_t)L * B > AL_MAX_SELECT_POSITIONS) return decline();
    const int64_t LB = (int64_t)L * B, N = rp->size(0);
    if (tok->numel() != LB || msk->numel() != LB || N > LB) return decline();
    uint8_t role[AL_MAX_LANES];
    int32_t b_len[AL_MAX_LANES], t_lane[AL_MAX_LANES], k_lane[AL_MAX_LANES];
    g.host_array(a[7], role, L);
    if (a[8] != Py_None) g.host_array(a[8], b_len, L);
    if (a[9] != Py_None) g.host_array(a[9], t_lane, L);
    if (a[13] != Py_None) g.host_array(a[13], k_lane, L);
    int32_t delim[AL_MAX_DELIMS], digit[AL_MAX_BOUNDARY_IDS], open[AL_MAX_BOUNDARY_IDS], close[AL_MAX_BOUNDARY_IDS];
    const int n_delim = g.id_set(a[14], delim, AL_MAX_DELIMS);
    const int n_digit = g.id_set(a[20], digit, AL_MAX_BOUNDARY_IDS);
    const int n_open = g.id_set(a[21], open, AL_MAX_BOUNDARY_IDS);
    const int n_close = g.id_set(a[22], close, AL_MAX_BOUNDARY_IDS);
    const int mode = g.to_int(a[10]), fallback_k = g.to_int(a[12]), eos = g.to_int(a[15]), t_min = g.to_int(a[17]);
    const float tau = g.to_float(a[11]), rho = g.to_float(a[16]);
    const float tau_f = a[18] == Py_None ? INFINITY : g.to_float(a[18]);
    PyObject* out = a[19];
    const at::Tensor *uf = item(g, out, "unmask_flag"), *up = item(g, out, "unmasked_pos"),
                     *sp = item(g, out, "still_masked_pos"), *cn = item(g, out, "counts"),
                     *ls = item(g, out, "lane_stats");
    PyObject* dfo = PyDict_GetItemString(out, "delim_flag");
    const at::Tensor* df = dfo ? g.tensor(dfo) : nullptr;
    if (!g.ok || !uf || !up || !sp || !cn || !ls || PyDict_GET_SIZE(out) > 6 || (PyDict_GET_SIZE(out) == 6 && !dfo))
      return decline();
    const int dev = current_device();
    void* cp = g.data_n(conf, at::kFloat, dev, N);
    void* ap = g.data_n(arg, at::kInt, dev, N);
    void* rpp = g.data(rp, at::kInt, dev);
    void* tp = g.data(tok, at::kInt, dev);
    void* mp = g.data(msk, at::kByte, dev);
    void* ufp = g.data_n(uf, at::kByte, dev, N);
    void* upp = g.data_n(up, at::kInt, dev, N);
    void* spp = g.data_n(sp, at::kInt, dev, N);
    void* cnp = g.data_n(cn, at::kInt, dev, 2);
    void* lsp = g.data_n(ls, at::kInt, dev, (int64_t)L * AL_LANE_STATS);
    void* dfp = g.data_n(df, at::kByte, dev, LB);
    if (!g.ok) return decline();
    void* stream = g.stream_of(dev);
    if (!g.ok) return decline();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f_select(N ? (float*)cp : nullptr, N ? (int32_t*)ap : nullptr, N ? (int32_t*)rpp : nullptr, (int)N,
                  (int32_t*)tp, (uint8_t*)mp, L, B, role, a[8] == Py_None ? nullptr : b_len,
                  a[9] == Py_None ? nullptr : t_lane, mode, tau, fallback_k, a[13] == Py_None ? nullptr : k_lane,
                  n_delim ? delim : nullptr, n_delim, n_digit ? digit : nullptr, n_digit, n_open ? open : nullptr,
                  n_open, n_close ? close : nullptr, n_close, eos, rho, t_min, tau_f, (uint8_t*)ufp, (int32_t*)upp,
                  (int32_t*)spp, (int32_t*)cnp, (int32_t*)lsp, (uint8_t*)dfp, stream);
    Py_END_ALLOW_THREADS
    if (!status_ok(st, "select_unmask")) return nullptr;
    Py_RETURN_TRUE;
  });
}

// init(addresses, check, workspace, raw_stream): addresses maps the C ABI's
// names to their addresses in the loaded library.
PyObject* init(PyObject*, PyObject* args) {
  PyObject *addr, *check, *ws, *rs;
  if (!PyArg_ParseTuple(args, "O!OOO", &PyDict_Type, &addr, &check, &ws, &rs)) return nullptr;
  auto get = [&](const char* name) -> void* {
    PyObject* o = PyDict_GetItemString(addr, name);
    return o ? PyLong_AsVoidPtr(o) : nullptr;
  };
#define AL_GET(var, name)                                       \
  var = reinterpret_cast<decltype(var)>(get(name));             \
  if (!var) return PyErr_Format(PyExc_ValueError, "no %s", name);
  AL_GET(f_attn_ws, "lane_attn_workspace_size")
  AL_GET(f_attn, "lane_attn_forward")
  AL_GET(f_lm_ws, "lmhead_confidence_workspace_size")
  AL_GET(f_lm_packed_size, "lmhead_packed_weight_size")
  AL_GET(f_lm, "lmhead_confidence")
  AL_GET(f_lm_packed, "lmhead_confidence_packed")
  AL_GET(f_select, "select_unmask")
#undef AL_GET
  Py_XINCREF(check);
  Py_XINCREF(ws);
  Py_XINCREF(rs);
  py_check = check;
  py_workspace = ws;
  py_raw_stream = rs;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)init, METH_VARARGS, nullptr},
    {"attn", (PyCFunction)(void (*)())attn, METH_FASTCALL, nullptr},
    {"lmhead", (PyCFunction)(void (*)())lmhead, METH_FASTCALL, nullptr},
    {"select", (PyCFunction)(void (*)())select, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast() { return PyModule_Create(&module); }
