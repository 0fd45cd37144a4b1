// The Python calls of a serving loop without ctypes: parameters read from the tensors, outputs allocated and the C
// function called in one step.  A call costs what its launch costs, and ctypes, the attribute reads and four
// torch.empty cost more than that: 14.8 us for a compress call whose kernel takes 9 us, 6.2 us for a token in
// decode whose kernel takes 3 us.
//
// It takes the plain forms only (exact tensors of one device, four dimensions, integers and floats as such).  Anything
// else - and what lagkv_plan refuses or an allocator throws - it leaves alone and says so (None, or -1): lagkv.py
// then goes through its own steps, which raise what they raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include "compress_ws.h"
#include "lagkv.h"

namespace {

decltype(&lagkv_plan) plan_fn;
decltype(&lagkv_workspace_bytes) workspace_fn;
decltype(&lagkv_compress) compress_fn;
decltype(&lagkv_append_and_compress) append_fn;
PyObject* raw_stream_fn;  // device index -> handle of the current stream

bool to_int(PyObject* o, int32_t* v) {
  if (!PyLong_Check(o)) return false;
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  if (over || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

bool to_double(PyObject* o, double* v) {
  if (!PyFloat_CheckExact(o)) return false;
  *v = PyFloat_AS_DOUBLE(o);
  return true;
}

// A [B,H,T,D] device tensor of one of the element types.
const at::Tensor* rows_of(PyObject* o, int32_t* dtype) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || t.dim() != 4 || t.stride(3) != 1) return nullptr;
  switch (t.scalar_type()) {
    case at::kFloat: *dtype = LAGKV_F32; break;
    case at::kBFloat16: *dtype = LAGKV_BF16; break;
    case at::kHalf: *dtype = LAGKV_F16; break;
    default: return nullptr;
  }
  return &t;
}

bool alike(const at::Tensor& a, const at::Tensor& b) {
  return a.sizes() == b.sizes() && a.strides() == b.strides() && a.device() == b.device();
}

// S, L, r, variant, std_ddof, launch from args[0 .. 6)
bool params_of(PyObject* const* args, const at::Tensor& K, int32_t dtype, lagkv_params* p) {
  if (K.size(0) > INT32_MAX || K.size(1) > INT32_MAX || K.size(3) > INT32_MAX) return false;
  p->B = (int32_t)K.size(0);
  p->H = (int32_t)K.size(1);
  p->D = (int32_t)K.size(3);
  p->dtype = dtype;
  p->stride_b = K.stride(0);
  p->stride_h = K.stride(1);
  p->stride_t = K.stride(2);
  return to_int(args[0], &p->S) && to_int(args[1], &p->L) && to_double(args[2], &p->r) && to_int(args[3], &p->variant) &&
         to_int(args[4], &p->std_ddof) && to_int(args[5], &p->launch);
}

bool stream_of(const at::Tensor& t, void** s) {
  PyObject* i = PyLong_FromLong(t.device().index());
  PyObject* h = i ? PyObject_CallFunctionObjArgs(raw_stream_fn, i, nullptr) : nullptr;
  Py_XDECREF(i);
  if (!h) return false;
  *s = (void*)PyLong_AsSize_t(h);
  Py_DECREF(h);
  return !PyErr_Occurred();
}

PyObject* none() {
  PyErr_Clear();
  Py_RETURN_NONE;
}

// compress(K, V, S, L, r, variant, std_ddof, launch, want_idx, want_scores)
//   -> (K_out, V_out, idx or None, scores or None, bytes of the plan), the status that lagkv_compress refused with (it is
//      not called a second time), or None: not called
PyObject* compress(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 10 || !PyBool_Check(args[8]) || !PyBool_Check(args[9])) return none();
  try {
    int32_t dt, dv;
    const at::Tensor *K = rows_of(args[0], &dt), *V = rows_of(args[1], &dv);
    lagkv_params p;
    void* stream;
    if (!K || !V || dt != dv || !alike(*K, *V) || !params_of(args + 2, *K, dt, &p)) return none();
    const int64_t T = K->size(2);
    lagkv_plan_t pl;
    if (plan_fn(&p, T, -1, &pl) != LAGKV_OK || !stream_of(*K, &stream)) return none();
    const auto opt = K->options().requires_grad(false);
    const int64_t B = p.B, H = p.H, D = p.D;
    at::Tensor Ko = at::empty({B, H, pl.T_out, D}, opt), Vo = at::empty({B, H, pl.T_out, D}, opt), idx, scores, ws;
    if (args[8] == Py_True) idx = at::empty({B, H, pl.T_out}, opt.dtype(at::kInt));
    if (args[9] == Py_True) scores = at::empty({B, H, pl.n_scored * p.L}, opt.dtype(at::kFloat));
    size_t need = 0;
    if (workspace_fn(&p, T)) {
      need = lagkv::compress_ws(B * H, pl.n_scored, p.L, pl.k, true).total;
      ws = at::empty({(int64_t)need}, opt.dtype(at::kByte));
    }
    const void *k = K->data_ptr(), *v = V->data_ptr();
    void *ko = Ko.data_ptr(), *vo = Vo.data_ptr(), *w = need ? ws.data_ptr() : nullptr;
    int32_t* ip = idx.defined() ? (int32_t*)idx.data_ptr() : nullptr;
    float* sp = scores.defined() ? (float*)scores.data_ptr() : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = compress_fn(&p, k, v, T, ko, vo, ip, sp, w, need, stream);
    Py_END_ALLOW_THREADS
    if (rc != LAGKV_OK) return PyLong_FromLong(rc);
    PyObject* out = PyTuple_New(5);
    if (!out) return nullptr;
    auto put = [&](int i, const at::Tensor& t) {
      PyObject* o = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
      PyTuple_SET_ITEM(out, i, o);
      return o != nullptr;
    };
    bool ok = put(0, Ko);
    ok = put(1, Vo) && ok;
    ok = put(2, idx) && ok;
    ok = put(3, scores) && ok;
    PyObject* b = PyBytes_FromStringAndSize((const char*)&pl, sizeof(pl));
    PyTuple_SET_ITEM(out, 4, b);
    if (ok && b) return out;
    Py_DECREF(out);
    return nullptr;
  } catch (...) {
    return none();
  }
}

// append(counters, K of the cache, S, L, r, variant, std_ddof, launch, workspace or None, K_new, V_new)
//   -> the status of lagkv_append_and_compress, or -1: not called
PyObject* append(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  auto status = [](long v) {
    PyErr_Clear();
    return PyLong_FromLong(v);
  };
  if (nargs != 11) return status(-1);
  try {
    int32_t dc, dk, dv;
    const at::Tensor *C = rows_of(args[1], &dc), *K = rows_of(args[9], &dk), *V = rows_of(args[10], &dv);
    lagkv_params p;
    void* stream;
    if (!C || !K || !V || dk != dc || dv != dc || !alike(*K, *V) || K->device() != C->device() ||
        K->size(0) != C->size(0) || K->size(1) != C->size(1) || K->size(3) != C->size(3) ||
        !params_of(args + 2, *K, dk, &p))
      return status(-1);
    const size_t need = workspace_fn(&p, C->size(2));
    void* w = nullptr;
    size_t ws_bytes = 0;
    if (args[8] != Py_None) {
      if (!THPVariable_CheckExact(args[8])) return status(-1);
      const at::Tensor& ws = THPVariable_Unpack(args[8]);
      w = ws.data_ptr();
      ws_bytes = (size_t)ws.numel();
    }
    if (ws_bytes < need || !stream_of(*C, &stream)) return status(-1);
    const void *k = K->data_ptr(), *v = V->data_ptr();
    const int64_t n_new = K->size(2);
    Py_buffer view;
    if (PyObject_GetBuffer(args[0], &view, PyBUF_WRITABLE) != 0) return status(-1);
    int rc = -1;
    if (view.len == (Py_ssize_t)sizeof(lagkv_cache)) {
      Py_BEGIN_ALLOW_THREADS
      rc = append_fn(&p, (lagkv_cache*)view.buf, k, v, n_new, w, ws_bytes, stream);
      Py_END_ALLOW_THREADS
    }
    PyBuffer_Release(&view);
    return status(rc);
  } catch (...) {
    return status(-1);
  }
}

// init(plan, workspace_bytes, compress, append_and_compress: addresses; raw stream function)
PyObject* init(PyObject*, PyObject* args) {
  size_t a[4];
  PyObject* f;
  static_assert(sizeof(size_t) == sizeof(unsigned long), "");
  if (!PyArg_ParseTuple(args, "kkkkO", &a[0], &a[1], &a[2], &a[3], &f)) return nullptr;
  plan_fn = (decltype(plan_fn))a[0];
  workspace_fn = (decltype(workspace_fn))a[1];
  compress_fn = (decltype(compress_fn))a[2];
  append_fn = (decltype(append_fn))a[3];
  Py_INCREF(f);
  Py_XSETREF(raw_stream_fn, f);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"compress", (PyCFunction)(void (*)(void))compress, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)(void))append, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lagkv_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lagkv_native(void) { return PyModule_Create(&module); }
