// The argument checks of a decoding step in native code, for the binding.  A step of a short cache is two kernels of
// 8.6 us together, and the checks of its twelve tensors took 5 us of interpreter time per call, so that the host and
// not the GPU decided how long it took: 11.3 us to issue one, now 6.6, and a step over 8 KV heads of 512 rows at
// d = 64 took 11.0 us, now 9.1.  Only the case in which everything is as it has to be is handled here: whatever is
// not comes back as None, and the checks in binding.py look again and report it.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <limits>

#include "adakv.h"

namespace {

typedef int (*StepFn)(const adakv_layer *, const void *, const void *, const void *, const int32_t *, int32_t, void *, void *,
                      int32_t *, int32_t *, float *, float *, void *, size_t, void *);

// A plain tensor on the GPU of the given type, else nullptr (subclasses are the interpreter's business).
const at::Tensor *device_tensor(PyObject *o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  return t.is_cuda() && t.scalar_type() == type ? &t : nullptr;
}
bool is_rows(const at::Tensor *t, int64_t batch, int64_t h, int64_t d) {
  return t && t->dim() == 3 && t->size(0) == batch && t->size(1) == h && t->size(2) == d && t->is_contiguous();
}
bool is_cache(const at::Tensor *t, int64_t rows, int64_t d) {
  return t && t->dim() >= 1 && t->size(0) >= rows && t->size(-1) == d && t->numel() >= rows * d && t->is_contiguous();
}
bool holds(const at::Tensor *t, int64_t numel) { return t && t->numel() >= numel && t->is_contiguous(); }

// decode_step(function, layer, q, k, v, cu_seqlens, headroom, K_cache, V_cache, seg_len, overflow, out, lse, ws, stream)
// -> the library's status, or None where the arguments are for binding.py to look at
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 15) {
    PyErr_SetString(PyExc_TypeError, "decode_step takes 15 arguments");
    return nullptr;
  }
  const StepFn fn = reinterpret_cast<StepFn>(PyLong_AsVoidPtr(a[0]));
  const adakv_layer *L = static_cast<const adakv_layer *>(PyLong_AsVoidPtr(a[1]));
  void *stream = PyLong_AsVoidPtr(a[14]);
  const long headroom = PyLong_Check(a[6]) ? PyLong_AsLong(a[6]) : -1;
  if (PyErr_Occurred()) {                      // an address, a stream or a head-room that is no whole number
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (!fn || !L || headroom < 0 || headroom > std::numeric_limits<int32_t>::max()) Py_RETURN_NONE;
  try {
    const at::ScalarType type = L->dtype == ADAKV_BF16 ? at::kBFloat16 : L->dtype == ADAKV_FP16 ? at::kHalf : at::kFloat;
    if ((L->dtype != ADAKV_FP32 && type == at::kFloat) || L->batch < 1 || L->batch > ADAKV_MAX_BATCH) Py_RETURN_NONE;
    const int64_t nseg = (int64_t)L->batch * L->h_kv;
    int64_t rows = nseg * headroom;
    for (int b = 0; b < L->batch; ++b) rows += L->B[b];
    const at::Tensor *q = device_tensor(a[2], type), *k = device_tensor(a[3], type), *v = device_tensor(a[4], type);
    const at::Tensor *cu = device_tensor(a[5], at::kInt), *Kc = device_tensor(a[7], type), *Vc = device_tensor(a[8], type);
    const at::Tensor *len = device_tensor(a[9], at::kInt), *over = a[10] == Py_None ? nullptr : device_tensor(a[10], at::kInt);
    const at::Tensor *out = device_tensor(a[11], at::kFloat), *lse = a[12] == Py_None ? nullptr : device_tensor(a[12], at::kFloat);
    const at::Tensor *ws = device_tensor(a[13], at::kByte);
    if (!is_rows(q, L->batch, L->h_q, L->d) || !is_rows(k, L->batch, L->h_kv, L->d) || !is_rows(v, L->batch, L->h_kv, L->d) ||
        !is_cache(Kc, rows, L->d) || !is_cache(Vc, rows, L->d) || !holds(cu, nseg + 1) || !holds(len, nseg) ||
        (a[10] != Py_None && !holds(over, 1)) || !holds(out, (int64_t)L->batch * L->h_q * L->d) ||
        (a[12] != Py_None && !holds(lse, (int64_t)L->batch * L->h_q)) || !holds(ws, 0))
      Py_RETURN_NONE;
    void *p[12] = {q->data_ptr(), k->data_ptr(), v->data_ptr(), cu->data_ptr(), Kc->data_ptr(), Vc->data_ptr(), len->data_ptr(),
                   over ? over->data_ptr() : nullptr, out->data_ptr(), lse ? lse->data_ptr() : nullptr, ws->data_ptr(), stream};
    const size_t ws_bytes = (size_t)ws->numel();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(L, p[0], p[1], p[2], (const int32_t *)p[3], (int32_t)headroom, p[4], p[5], (int32_t *)p[6], (int32_t *)p[7],
            (float *)p[8], (float *)p[9], p[10], ws_bytes, p[11]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (...) {                              // a tensor without memory of its own, for instance
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL,
     "decode_step(function, layer, q, k, v, cu_seqlens, headroom, K_cache, V_cache, seg_len, overflow, out, lse, ws, stream)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// TORCH_VERSION: a tensor's layout is that of the headers compiled against, which binding.py compares with torch itself.
PyMODINIT_FUNC PyInit__marshal() {
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "TORCH_VERSION", TORCH_VERSION) < 0) Py_CLEAR(m);
  return m;
}
