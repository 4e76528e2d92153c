// The four attention calls on torch tensors as the Python wrappers make them: checks, outputs, workspace, current
// stream and the call itself, without the interpreter between them.
//
// The smallest calls are bound by the host.  Host time of a call on a tree of 256 tokens, with the same steps in Python
// and here: forward 13.0 -> 5.9 us, backward 18.5 -> 10.6 (its launches are most of what is left), a segment's forward
// 10.3 -> 6.9, its backward 14.9 -> 7.3; forward and backward of a tiny fp32 tree 34.3 -> 28.2 us, now what the GPU takes.
//
// Every function returns None, having done nothing, where it does not know its arguments (another kind of tensor, a
// shape, type, device or layout that does not fit, an integer that is none): the wrapper in Python then makes the call or
// raises the error.  Otherwise it returns the library's status if that is not 0, or its outputs.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cxxabi.h>

#include <algorithm>

#include "dta.h"

namespace {

// What the arguments of one call have in common.
struct Call {
  dta_tree_t* tree;
  const dta_attn_params_t* params;
  int64_t n_tokens;
  at::ScalarType dtype;

  // handle, address of the parameters, tokens of the tree
  bool read(PyObject* const* args) {
    if (at::impl::torch_function_mode_enabled()) return false;   // (it is to see the allocations)
    if (!PyLong_CheckExact(args[0]) || !PyLong_CheckExact(args[1]) || !PyLong_CheckExact(args[2])) return false;
    tree = static_cast<dta_tree_t*>(PyLong_AsVoidPtr(args[0]));
    params = static_cast<const dta_attn_params_t*>(PyLong_AsVoidPtr(args[1]));
    n_tokens = PyLong_AsLongLong(args[2]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    if (!tree || !params) return false;
    dtype = params->dtype == DTA_F32 ? at::kFloat : at::kBFloat16;
    return true;
  }
  // a plain contiguous device tensor of `dims` dimensions: [n_tokens, heads(, head_dim)]
  bool fits(PyObject* obj, size_t dims, int64_t heads, at::ScalarType type) const {
    if (!THPVariable_CheckExact(obj)) return false;
    const at::Tensor& t = THPVariable_Unpack(obj);
    const auto size = t.sizes();
    return t.is_cuda() && t.scalar_type() == type && size.size() == dims && size[0] == n_tokens &&
           size[1] == heads && (dims == 2 || size[2] == params->head_dim) && t.is_contiguous();
  }
  bool q_like(PyObject* obj) const { return fits(obj, 3, params->n_q_heads, dtype); }
  bool k_like(PyObject* obj) const { return fits(obj, 3, params->n_kv_heads, dtype); }
  bool k_sum(PyObject* obj) const { return fits(obj, 3, params->n_kv_heads, at::kFloat); }
  bool row(PyObject* obj) const { return fits(obj, 2, params->n_q_heads, at::kFloat); }
};

void* data(PyObject* obj) { return THPVariable_Unpack(obj).data_ptr(); }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the caller's workspace: any contiguous device tensor, or an empty one
bool workspace_of(PyObject* obj, void** ptr, size_t* bytes) {
  if (!THPVariable_CheckExact(obj)) return false;
  const at::Tensor& t = THPVariable_Unpack(obj);
  if (t.numel() && !(t.is_cuda() && t.is_contiguous())) return false;
  *ptr = t.data_ptr();
  *bytes = (size_t)t.numel() * t.element_size();
  return true;
}

// The interpreter's lock is given up for the allocations and the call, as torch and ctypes do.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  Unlocked() = default;
  Unlocked(const Unlocked&) = delete;
  // (a thread that asks for the lock after the interpreter has ended is unwound from here)
  ~Unlocked() noexcept(false) { PyEval_RestoreThread(state); }
};

// The caller's output (its object is returned), or a new tensor.
struct Output {
  PyObject* given = nullptr;
  at::Tensor made;
  void* ptr(PyObject* obj, const at::Tensor& like) {
    if (obj != Py_None) {
      given = obj;
      return data(obj);
    }
    made = at::empty_like(like);
    return made.data_ptr();
  }
  PyObject* result() {
    if (given) {
      Py_INCREF(given);
      return given;
    }
    return THPVariable_Wrap(std::move(made));
  }
};

// No C++ exception leaves a function: what torch throws (a tensor without memory, no memory left) is met again, as the
// Python exception it is, by the wrapper that makes the call itself.
template <class Body>
PyObject* guarded(Body body) {
  try {
    return body();
  } catch (abi::__forced_unwind&) {
    throw;
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyObject* tuple_of(Output* outputs, int n) {
  PyObject* res = PyTuple_New(n);
  for (int i = 0; res && i < n; ++i) {
    PyObject* item = outputs[i].result();
    if (!item) {
      Py_DECREF(res);
      return nullptr;
    }
    PyTuple_SET_ITEM(res, i, item);
  }
  return res;
}

// handle, params, n_tokens, q, k, v, o | None, lse | None, workspace | None -> (o, lse)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    if (n != 9 || !c.read(a) || !c.q_like(a[3]) || !c.k_like(a[4]) || !c.k_like(a[5]) ||
        (a[6] != Py_None && !c.q_like(a[6])) || (a[7] != Py_None && !c.row(a[7])))
      Py_RETURN_NONE;
    const at::Tensor& q = THPVariable_Unpack(a[3]);
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (a[8] != Py_None && !workspace_of(a[8], &ws, &ws_bytes)) Py_RETURN_NONE;
    void *qp = data(a[3]), *kp = data(a[4]), *vp = data(a[5]), *st = stream();
    Output out[2];
    at::Tensor own;
    int status;
    {
      Unlocked unlocked;
      void* op = out[0].ptr(a[6], q);
      if (a[7] != Py_None) {
        out[1].given = a[7];
      } else {
        out[1].made = at::empty({c.n_tokens, c.params->n_q_heads}, q.options().dtype(at::kFloat));
      }
      float* lp = static_cast<float*>(out[1].given ? data(a[7]) : out[1].made.data_ptr());
      if (a[8] == Py_None && (ws_bytes = dta_tree_attn_workspace_bytes(c.tree, c.params, 0))) {
        own = at::empty({(int64_t)ws_bytes}, q.options().dtype(at::kByte));
        ws = own.data_ptr();
      }
      status = dta_tree_attn_fwd(c.tree, c.params, qp, kp, vp, op, lp, ws, ws_bytes, st);
    }
    return status ? PyLong_FromLong(status) : tuple_of(out, 2);
  });
}

// handle, params, n_tokens, q, k, v, o, lse, d_o, dq | None, dk | None, dv | None, workspace | None -> (dq, dk, dv)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    if (n != 13 || !c.read(a) || !c.q_like(a[3]) || !c.k_like(a[4]) || !c.k_like(a[5]) || !c.q_like(a[6]) ||
        !c.row(a[7]) || !c.q_like(a[8]) || (a[9] != Py_None && !c.q_like(a[9])) ||
        (a[10] != Py_None && !c.k_like(a[10])) || (a[11] != Py_None && !c.k_like(a[11])))
      Py_RETURN_NONE;
    const at::Tensor& q = THPVariable_Unpack(a[3]);
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (a[12] != Py_None && !workspace_of(a[12], &ws, &ws_bytes)) Py_RETURN_NONE;
    void *qp = data(a[3]), *kp = data(a[4]), *vp = data(a[5]), *op = data(a[6]), *dop = data(a[8]), *st = stream();
    float* lp = static_cast<float*>(data(a[7]));
    Output out[3];
    at::Tensor own;
    int status;
    {
      Unlocked unlocked;
      void* dqp = out[0].ptr(a[9], q);
      void* dkp = out[1].ptr(a[10], THPVariable_Unpack(a[4]));
      void* dvp = out[2].ptr(a[11], THPVariable_Unpack(a[5]));
      if (a[12] == Py_None) {
        ws_bytes = std::max<size_t>(dta_tree_attn_workspace_bytes(c.tree, c.params, 1), 256);
        own = at::empty({(int64_t)ws_bytes}, q.options().dtype(at::kByte));
        ws = own.data_ptr();
      }
      status = dta_tree_attn_bwd(c.tree, c.params, qp, kp, vp, op, lp, dop, dqp, dkp, dvp, ws, ws_bytes, st);
    }
    return status ? PyLong_FromLong(status) : tuple_of(out, 3);
  });
}

bool rows_of(PyObject* const* a, int64_t* begin, int64_t* end) {
  if (!PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[1])) return false;
  *begin = PyLong_AsLongLong(a[0]);
  *end = PyLong_AsLongLong(a[1]);
  if (!PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

// handle, params, n_tokens, t_begin, t_end, q, k, v, o, lse -> status
PyObject* fwd_segment(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    int64_t t0, t1;
    if (n != 10 || !c.read(a) || !rows_of(a + 3, &t0, &t1) || !c.q_like(a[5]) || !c.k_like(a[6]) || !c.k_like(a[7]) ||
        !c.q_like(a[8]) || !c.row(a[9]))
      Py_RETURN_NONE;
    void *qp = data(a[5]), *kp = data(a[6]), *vp = data(a[7]), *op = data(a[8]), *st = stream();
    float* lp = static_cast<float*>(data(a[9]));
    int status;
    {
      Unlocked unlocked;
      status = dta_tree_attn_fwd_segment(c.tree, c.params, t0, t1, qp, kp, vp, op, lp, nullptr, 0, st);
    }
    return PyLong_FromLong(status);
  });
}

// handle, params, n_tokens, t_begin, t_end, q, k, v, o, lse, d_o, dq, dk_acc, dv_acc, workspace -> status
PyObject* bwd_segment(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    int64_t t0, t1;
    void* ws;
    size_t ws_bytes;
    if (n != 15 || !c.read(a) || !rows_of(a + 3, &t0, &t1) || !c.q_like(a[5]) || !c.k_like(a[6]) || !c.k_like(a[7]) ||
        !c.q_like(a[8]) || !c.row(a[9]) || !c.q_like(a[10]) || !c.q_like(a[11]) || !c.k_sum(a[12]) ||
        !c.k_sum(a[13]) || !workspace_of(a[14], &ws, &ws_bytes))
      Py_RETURN_NONE;
    void *qp = data(a[5]), *kp = data(a[6]), *vp = data(a[7]), *op = data(a[8]), *dop = data(a[10]), *dqp = data(a[11]);
    float *lp = static_cast<float*>(data(a[9])), *dkp = static_cast<float*>(data(a[12])),
          *dvp = static_cast<float*>(data(a[13]));
    void* st = stream();
    int status;
    {
      Unlocked unlocked;
      status = dta_tree_attn_bwd_segment(c.tree, c.params, t0, t1, qp, kp, vp, op, lp, dop, dqp, dkp, dvp, ws, ws_bytes, st);
    }
    return PyLong_FromLong(status);
  });
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<fwd>("fwd"), method<bwd>("bwd"), method<fwd_segment>("fwd_segment"),
                         method<bwd_segment>("bwd_segment"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "dta_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_dta_torch() {
  PyObject* module = PyModule_Create(&module_def);
  // the torch and Python it was compiled against: with others its tensors may be laid out otherwise
  if (module && PyModule_AddStringConstant(module, "built_for", DTA_TORCH_BUILT_FOR) < 0) Py_CLEAR(module);
  return module;
}
