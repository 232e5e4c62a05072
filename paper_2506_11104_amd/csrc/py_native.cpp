// The hot entry points of libdam.so for Python, without ctypes: a decode step of one sequence from a plan is one launch of
// about 3 us of host time, and filling a parameter structure through ctypes, taking six tensors' addresses and asking
// torch for its stream cost another 9 us (while a step was two launches, 14.4 us per call, host bound). Reading shapes,
// strides and addresses from the tensor objects here costs about 1 us.
//
// Argument marshalling only, as in binding.py: every function takes tensors (or None) and numbers, enqueues on torch's
// current stream and returns the dam_status, or one of the codes below for what the wrappers in binding.py report as a
// Python error of their own.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "dam.h"

namespace {

constexpr int kBadDtype = -1000;    // a query tensor that is neither fp32 nor bf16
constexpr int kBadLayout = -1001;   // strides or shapes the wrappers rule out by assertion

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// A tensor argument. None is allowed where `maybe` says so and leaves `defined` false.
struct Arg {
  const at::Tensor *t = nullptr;
  bool ok = true;
  Arg(PyObject *o, bool maybe = false) {
    if (THPVariable_Check(o)) {
      t = &THPVariable_Unpack(o);
    } else if (!(maybe && o == Py_None)) {
      ok = false;
      PyErr_Format(PyExc_TypeError, "a tensor%s is wanted, got %s", maybe ? " or None" : "", Py_TYPE(o)->tp_name);
    }
  }
  void *ptr() const { return t ? t->data_ptr() : nullptr; }
  size_t bytes() const { return t ? (size_t)t->numel() : 0; }  // of a workspace: a byte tensor
  int64_t dim() const { return t->dim(); }
  int64_t size(int i) const { return t->sizes()[i]; }
  int64_t stride(int i) const { return t->strides()[i]; }
};

bool number(PyObject *o, int64_t *v) {
  *v = PyLong_AsLongLong(o);
  return !(*v == -1 && PyErr_Occurred());
}
bool number(PyObject *o, float *v) {
  const double d = PyFloat_AsDouble(o);
  *v = (float)d;
  return !(d == -1.0 && PyErr_Occurred());
}

// The memory of a ctypes structure of at least n bytes.
struct Struct {
  Py_buffer b{};
  bool ok;
  Struct(PyObject *o, size_t n) {
    ok = PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) == 0;
    if (ok && (size_t)b.len < n) {
      PyErr_SetString(PyExc_ValueError, "parameter structure too small");
      PyBuffer_Release(&b);
      ok = false;
    }
  }
  ~Struct() {
    if (ok) PyBuffer_Release(&b);
  }
  template <typename T>
  T *as() const { return static_cast<T *>(b.buf); }
};

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) PyErr_Format(PyExc_TypeError, "%zd arguments are wanted, got %zd", want, n);
  return n == want;
}

int dtype_code(const Arg &q) {
  return q.t->scalar_type() == at::kFloat ? DAM_F32 : q.t->scalar_type() == at::kBFloat16 ? DAM_BF16 : -1;
}

PyObject *status(int st) { return PyLong_FromLong(st); }

// A call of the library, with the interpreter's lock given back: a launch may have to wait for room in the stream's queue.
template <typename F, typename... A>
PyObject *call(F f, A... args) {
  PyThreadState *const saved = PyEval_SaveThread();
  const int st = f(args...);
  PyEval_RestoreThread(saved);
  return status(st);
}

// An entry as Python sees it: what torch throws (a tensor without memory or strides: fake, sparse) becomes a Python error.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n) {
  try {
    return F(a, n);
  } catch (const std::exception &e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// (params, attn_sum, attn_cnt, diag_in, vert_in, out, ws)
PyObject *mask_build(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 7)) return nullptr;
  const Struct p(a[0], sizeof(dam_mask_params)), o(a[5], sizeof(dam_mask_out));
  const Arg as(a[1], true), ac(a[2], true), di(a[3], true), vi(a[4], true), ws(a[6], true);
  if (!p.ok || !o.ok || !as.ok || !ac.ok || !di.ok || !vi.ok || !ws.ok) return nullptr;
  return call(dam_mask_build, p.as<dam_mask_params>(), (const float *)as.ptr(), (const float *)ac.ptr(), (const uint8_t *)di.ptr(),
              (const uint8_t *)vi.ptr(), o.as<dam_mask_out>(), ws.ptr(), ws.bytes(), stream());
}

// (params, capture params, q, k, out, ws)
PyObject *mask_build_from_qk(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 6)) return nullptr;
  const Struct p(a[0], sizeof(dam_mask_params)), cp(a[1], sizeof(dam_capture_params)), o(a[4], sizeof(dam_mask_out));
  const Arg q(a[2]), k(a[3]), ws(a[5], true);
  if (!p.ok || !cp.ok || !o.ok || !q.ok || !k.ok || !ws.ok) return nullptr;
  return call(dam_mask_build_from_qk, p.as<dam_mask_params>(), cp.as<dam_capture_params>(), q.ptr(), k.ptr(), o.as<dam_mask_out>(),
              ws.ptr(), ws.bytes(), stream());
}

// (q, k, attn_sum, attn_cnt, L, scale, ws)
PyObject *capture_accumulate(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 7)) return nullptr;
  const Arg q(a[0]), k(a[1]), as(a[2]), ac(a[3], true), ws(a[6], true);
  int64_t L;
  float scale;
  if (!q.ok || !k.ok || !as.ok || !ac.ok || !ws.ok || !number(a[4], &L) || !number(a[5], &scale)) return nullptr;
  if (q.dim() != 3 || k.dim() < 3 || k.size(1) != q.size(1) || k.size(2) != q.size(2) || q.stride(2) != 1 || k.stride(2) != 1)
    return status(kBadLayout);
  dam_capture_params p{};
  p.hq = (int32_t)q.size(0);
  p.hkv = (int32_t)k.size(0);
  p.len = (int32_t)q.size(1);
  p.pcl = (int32_t)L;
  p.head_dim = (int32_t)q.size(2);
  p.dtype = dtype_code(q);
  if (p.dtype < 0) return status(kBadDtype);
  p.scale = scale;
  for (int i = 0; i < 2; ++i) p.q_stride[i] = q.stride(i), p.k_stride[i] = k.stride(i);
  return call(dam_capture_accumulate, &p, q.ptr(), k.ptr(), (float *)as.ptr(), (float *)ac.ptr(), ws.ptr(), ws.bytes(), stream());
}

// (q, k, v, blk_row_ptr, blk_col, blk_kind, tile_bits, gather_idx, gather_cnt, tile_m, tile_n, gather_rows, flags, scale, out, lse, ws)
PyObject *prefill(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 17)) return nullptr;
  const Arg q(a[0]), k(a[1]), v(a[2]), row(a[3], true), col(a[4], true), kind(a[5], true), bits(a[6], true), gi(a[7], true), gc(a[8], true),
      out(a[14]), lse(a[15], true), ws(a[16], true);
  int64_t tm, tn, gr, flags;
  float scale;
  if (!q.ok || !k.ok || !v.ok || !row.ok || !col.ok || !kind.ok || !bits.ok || !gi.ok || !gc.ok || !out.ok || !lse.ok || !ws.ok ||
      !number(a[9], &tm) || !number(a[10], &tn) || !number(a[11], &gr) || !number(a[12], &flags) || !number(a[13], &scale))
    return nullptr;
  for (const Arg *t : {&q, &k, &v, &out})
    if (t->dim() < 4 || t->stride(3) != 1) return status(kBadLayout);
  if (q.dim() != 4 || (gi.t && gi.dim() < 2)) return status(kBadLayout);
  dam_attn_params p{};
  p.batch = (int32_t)q.size(0);
  p.hq = (int32_t)q.size(1);
  p.hkv = (int32_t)k.size(1);
  p.seq = (int32_t)q.size(2);
  p.head_dim = (int32_t)q.size(3);
  p.dtype = dtype_code(q);
  if (p.dtype < 0) return status(kBadDtype);
  p.scale = scale;
  for (int i = 0; i < 3; ++i)
    p.q_stride[i] = q.stride(i), p.k_stride[i] = k.stride(i), p.v_stride[i] = v.stride(i), p.o_stride[i] = out.stride(i);
  p.tile_m = (int32_t)tm;
  p.tile_n = (int32_t)tn;
  p.gather_rows = (int32_t)gr;
  p.flags = (int32_t)flags;
  const dam_mask_view mv{(const int32_t *)row.ptr(),   (const int32_t *)col.ptr(), (const uint8_t *)kind.ptr(),
                         (const uint64_t *)bits.ptr(), (const int32_t *)gi.ptr(),  (const int32_t *)gc.ptr(),
                         gi.t ? (int32_t)gi.size(1) : 0};
  return call(dam_sparse_attn_prefill, &p, q.ptr(), k.ptr(), v.ptr(), &mv, out.ptr(), (float *)lse.ptr(), ws.ptr(), ws.bytes(), stream());
}

// The tensors and numbers every decode form shares.
struct Decode {
  Arg q, kc, vc, out, lse, ws;
  dam_decode_params p{};
  int bad = 0;  // a code from above
  bool ok;
  Decode(PyObject *q_, PyObject *kc_, PyObject *vc_, PyObject *out_, PyObject *lse_, PyObject *ws_, PyObject *scale_, bool shared)
      : q(q_), kc(kc_), vc(vc_), out(out_), lse(lse_, true), ws(ws_, true) {
    float scale;
    ok = q.ok && kc.ok && vc.ok && out.ok && lse.ok && ws.ok && number(scale_, &scale);
    if (!ok) return;
    if (q.dim() != 3 || kc.dim() < 3 || out.dim() < 2 || kc.t->strides() != vc.t->strides()) {
      bad = kBadLayout;
      return;
    }
    p.batch = (int32_t)q.size(0);
    p.hq = (int32_t)q.size(1);
    p.hkv = (int32_t)kc.size(1);
    p.kv_capacity = (int32_t)kc.size(2);
    p.head_dim = (int32_t)q.size(2);
    p.dtype = dtype_code(q);
    if (p.dtype < 0) bad = kBadDtype;
    p.scale = scale;
    for (int i = 0; i < 2; ++i) p.q_stride[i] = q.stride(i), p.o_stride[i] = out.stride(i);
    for (int i = 0; i < 3; ++i) p.kv_stride[i] = kc.stride(i);
    p.shared_lists = shared ? 1 : 0;
  }
};

// (q, kcache, vcache, kept_ptr, kept_idx, kept_member, max_kept, out, lse, scale, shared, ws, form)
// form 0: a list per query head; 1: merged lists per KV head; 2: the same with the library's fixed scratch array.
PyObject *decode(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 13)) return nullptr;
  const Arg ptr(a[3]), idx(a[4], true), mem(a[5], true);
  int64_t max_kept;
  int64_t form;
  const int shared = PyObject_IsTrue(a[10]);
  if (!ptr.ok || !idx.ok || !mem.ok || shared < 0 || !number(a[6], &max_kept) || !number(a[12], &form)) return nullptr;
  const Decode d(a[0], a[1], a[2], a[7], a[8], a[11], a[9], shared != 0);
  if (!d.ok) return nullptr;
  if (d.bad) return status(d.bad);
  const int32_t *kp = (const int32_t *)ptr.ptr(), *ki = (const int32_t *)idx.ptr();
  const uint8_t *km = (const uint8_t *)mem.ptr();
  if (form == 2)
    return call(dam_sparse_attn_decode_grouped_static, &d.p, d.q.ptr(), d.kc.ptr(), d.vc.ptr(), kp, ki, km, max_kept, d.out.ptr(),
                (float *)d.lse.ptr(), stream());
  if (form == 0)
    return call(dam_sparse_attn_decode, &d.p, d.q.ptr(), d.kc.ptr(), d.vc.ptr(), kp, ki, max_kept, d.out.ptr(), (float *)d.lse.ptr(),
                d.ws.ptr(), d.ws.bytes(), stream());
  return call(dam_sparse_attn_decode_grouped, &d.p, d.q.ptr(), d.kc.ptr(), d.vc.ptr(), kp, ki, km, max_kept, d.out.ptr(),
              (float *)d.lse.ptr(), d.ws.ptr(), d.ws.bytes(), stream());
}

// (q, kcache, vcache, plan_ptr, plan_val, plan_member, plan_table, pos, max_entries, out, lse, scale, ws)
PyObject *decode_patterns(PyObject *const *a, Py_ssize_t n) {
  if (!arity(n, 13)) return nullptr;
  const Arg ptr(a[3]), val(a[4], true), mem(a[5], true), tab(a[6]);
  int64_t pos, most;
  if (!ptr.ok || !val.ok || !mem.ok || !tab.ok || !number(a[7], &pos) || !number(a[8], &most)) return nullptr;
  const Decode d(a[0], a[1], a[2], a[9], a[10], a[12], a[11], true);
  if (!d.ok) return nullptr;
  if (d.bad || tab.dim() != 2) return status(d.bad ? d.bad : kBadLayout);
  return call(dam_sparse_attn_decode_patterns, &d.p, d.q.ptr(), d.kc.ptr(), d.vc.ptr(), (const int32_t *)ptr.ptr(),
              (const int32_t *)val.ptr(), (const uint8_t *)mem.ptr(), (const uint8_t *)tab.ptr(),
              (int32_t)tab.size(1), (int32_t)pos, most, d.out.ptr(), (float *)d.lse.ptr(), d.ws.ptr(),
                                                d.ws.bytes(), stream());
}

#define DAM_FN(name) {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DAM_FN(mask_build), DAM_FN(mask_build_from_qk), DAM_FN(capture_accumulate), DAM_FN(prefill), DAM_FN(decode),
                         DAM_FN(decode_patterns), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dam_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dam_native(void) { return PyModule_Create(&module); }
