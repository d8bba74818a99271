// The calls that a program makes per product, from Python without ctypes: checks of the tensors, the current
// stream and the call into libspmm_brick.so.  A function here takes the plain case only -- tensors of the exact
// class on a device, of the right type, contiguous, with the right sizes and not empty -- and returns None for
// every other, which binding.py's own code then serves or refuses with its message.
//
// A product of a small matrix was bound by the host: 8.5 us a call through ctypes and torch.cuda.current_stream()
// (2.7 us alone), of which the library's launch is 3.4.  3.7 so, which is what the device takes for a product of
// 4096 rows behind another.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

typedef int (*ExecFn)(void* plan, const float* B, int64_t N, float* C, void* stream);
typedef int (*UpdateFn)(void* plan, const float* vals, void* stream);
typedef int (*PlanFn)(int64_t M, int64_t K, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                      const float* vals, void* stream, void** out);
ExecFn g_exec = nullptr, g_exec_noalloc = nullptr;
UpdateFn g_update = nullptr;
PlanFn g_plan = nullptr;

// a contiguous, non-empty tensor of `type` on a device, or null
const at::TensorBase* plain(PyObject* o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::TensorBase& t = THPVariable_Unpack(o);
  return t.defined() && t.is_cuda() && t.scalar_type() == type && t.is_contiguous() && t.numel() > 0 ? &t : nullptr;
}

bool integer(PyObject* o, int64_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  *out = PyLong_AsLongLong(o);
  if (*out == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// What a function does in the plain case, or None: nothing that torch throws (a tensor without storage, say)
// leaves here, the general code meets it again.
template <typename F> PyObject* none_unless(F f) {
  try {
    if (PyObject* r = f()) return r;
  } catch (...) {
  }
  if (PyErr_Occurred()) PyErr_Clear();
  Py_RETURN_NONE;
}

// (noalloc, plan, M, K, B, C) -> status
PyObject* product(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return none_unless([&]() -> PyObject* {
    int64_t plan, M, K;
    if (n != 6 || !integer(a[1], &plan) || !integer(a[2], &M) || !integer(a[3], &K)) return nullptr;
    const at::TensorBase *B = plain(a[4], at::kFloat), *C = plain(a[5], at::kFloat);
    if (!plan || !B || !C || B->dim() != 2 || C->dim() != 2) return nullptr;
    const int64_t N = B->size(1);
    if (B->size(0) != K || C->size(0) != M || C->size(1) != N) return nullptr;
    const float* b = static_cast<const float*>(B->data_ptr());
    float* c = static_cast<float*>(C->data_ptr());
    void* stream = current_stream();
    const ExecFn f = a[0] == Py_True ? g_exec_noalloc : g_exec;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f(reinterpret_cast<void*>(plan), b, N, c, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  });
}

// (plan, nnz, vals) -> status
PyObject* update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return none_unless([&]() -> PyObject* {
    int64_t plan, nnz;
    if (n != 3 || !integer(a[0], &plan) || !integer(a[1], &nnz)) return nullptr;
    const at::TensorBase* v = plain(a[2], at::kFloat);
    if (!plan || !v || v->numel() != nnz) return nullptr;
    const float* vals = static_cast<const float*>(v->data_ptr());
    void* stream = current_stream();
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = g_update(reinterpret_cast<void*>(plan), vals, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
  });
}

// (M, K, rowptr, colind, vals) -> (status, plan)
PyObject* plan(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return none_unless([&]() -> PyObject* {
    int64_t M, K;
    if (n != 5 || !integer(a[0], &M) || !integer(a[1], &K)) return nullptr;
    const at::TensorBase *r = plain(a[2], at::kInt), *c = plain(a[3], at::kInt), *v = plain(a[4], at::kFloat);
    if (!r || !c || !v || M < 0 || r->numel() != M + 1 || v->numel() != c->numel()) return nullptr;
    const int64_t nnz = c->numel();
    const int32_t *rowptr = static_cast<const int32_t*>(r->data_ptr()), *colind = static_cast<const int32_t*>(c->data_ptr());
    const float* vals = static_cast<const float*>(v->data_ptr());
    void *stream = current_stream(), *out = nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = g_plan(M, K, nnz, rowptr, colind, vals, stream, &out);
    Py_END_ALLOW_THREADS
    return Py_BuildValue("(iL)", status, (long long)reinterpret_cast<intptr_t>(out));
  });
}

// (addresses of spmm_exec, spmm_exec_noalloc, spmm_plan_update_values, spmm_plan)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t at[4];
  if (n != 4) { PyErr_SetString(PyExc_TypeError, "four addresses"); return nullptr; }
  for (int i = 0; i < 4; ++i)
    if (!integer(a[i], &at[i]) || !at[i]) { PyErr_SetString(PyExc_TypeError, "four addresses"); return nullptr; }
  g_exec = reinterpret_cast<ExecFn>(at[0]);
  g_exec_noalloc = reinterpret_cast<ExecFn>(at[1]);
  g_update = reinterpret_cast<UpdateFn>(at[2]);
  g_plan = reinterpret_cast<PlanFn>(at[3]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {"product", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(product)), METH_FASTCALL, nullptr},
    {"update", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(update)), METH_FASTCALL, nullptr},
    {"plan", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(plan)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", SPMM_BUILT_FOR) < 0) Py_CLEAR(m);
  return m;
}
