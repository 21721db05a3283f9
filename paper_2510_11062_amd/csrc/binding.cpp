// The grouping call as Python makes it: checks its tensors, makes the outputs and enqueues the kernels.
//
// A grouping call of a training step is 7 to 17 us of kernels, so what the host does around it is what a program waits for: of 16.3
// us for 64 responses, seven outputs made one by one from Python were 9, the checks and pointers of the arguments 3.  Everything else in
// api.py stays Python: those calls' kernels are longer than what the host does in front of them.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "at_grpo.h"

namespace {

using GroupFn = decltype(&at_grpo_group_advantage);
using MixedFn = decltype(&at_grpo_group_advantage_mixed);

enum Key { REWARD, GROUP_ID, N_GROUPS, SEG_OFFSETS, PERM, ADV, MEAN, STD, BEST, KEYS };
const char* const kKeyNames[KEYS] = {"reward", "group_id", "n_groups", "seg_offsets", "perm", "adv", "group_mean", "group_std", "best"};
PyObject* g_keys[KEYS];

// a contiguous tensor of the dtype on a GPU, or null
const at::Tensor* tensor(PyObject* o, at::ScalarType dtype) {
  if (!THPVariable_Check(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous() ? &t : nullptr;
}

// Other Python threads run while it lives, as they do during torch.empty: an allocation may have to wait for the driver, or for a thread
// that holds the allocator's lock and waits for Python's.
struct WithoutPythonLock {
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutPythonLock() { PyEval_RestoreThread(state); }
};

// group_advantage(function's address, env_id, agent_id, turn_id, reward or r_team, r_loc or None, alpha, n_env, n_agent, n_turn,
//                 eps_std, ddof, norm, want_stats, want_best, workspace, its bytes, stream)
// Returns the outputs, or the call's status, or None where an argument is no contiguous GPU tensor of its dtype (the caller says which).
// With r_loc the function is at_grpo_group_advantage_mixed, else at_grpo_group_advantage.
PyObject* group_advantage(PyObject*, PyObject* const* v, Py_ssize_t n_args) {
  // From the first look at a tensor on: some cannot say whether they are contiguous, and what they throw must not leave C.  An
  // allocator's error keeps the Python type that torch.empty raises it with (torch.OutOfMemoryError).
  HANDLE_TH_ERRORS
  if (n_args != 18) {
    PyErr_SetString(PyExc_TypeError, "group_advantage takes 18 arguments");
    return nullptr;
  }
  const bool mixed = v[5] != Py_None;
  const at::Tensor* ids[3];
  for (int k = 0; k < 3; ++k)
    if (!(ids[k] = tensor(v[1 + k], at::kInt))) Py_RETURN_NONE;
  const at::Tensor* reward = tensor(v[4], at::kFloat);
  const at::Tensor* loc = mixed ? tensor(v[5], at::kFloat) : nullptr;
  if (!reward || (mixed && !loc)) Py_RETURN_NONE;
  void* fn = PyLong_AsVoidPtr(v[0]);
  const double alpha = PyFloat_AsDouble(v[6]), eps_std = PyFloat_AsDouble(v[10]);
  const int64_t n_env = PyLong_AsLongLong(v[7]), n_agent = PyLong_AsLongLong(v[8]), n_turn = PyLong_AsLongLong(v[9]);
  const int64_t ddof = PyLong_AsLongLong(v[11]), norm = PyLong_AsLongLong(v[12]);
  const bool want_stats = PyObject_IsTrue(v[13]) == 1, want_best = PyObject_IsTrue(v[14]) == 1;
  void* ws = PyLong_AsVoidPtr(v[15]);
  const size_t ws_bytes = PyLong_AsSize_t(v[16]);
  void* stream = PyLong_AsVoidPtr(v[17]);
  if (PyErr_Occurred()) return nullptr;

  const int64_t R = reward->numel(), keys = n_env * n_agent * n_turn, groups = R < keys ? R : keys;
  const at::TensorOptions f32 = reward->options(), i32 = f32.dtype(at::kInt);
  at::Tensor out[KEYS];
  int status;
  {
    const WithoutPythonLock others_run;
    auto make_f = [&](Key key, int64_t n) { return static_cast<float*>((out[key] = at::empty({n}, f32)).data_ptr()); };
    auto make_i = [&](Key key, int64_t n) { return static_cast<int32_t*>((out[key] = at::empty({n}, i32)).data_ptr()); };
    float* mix = mixed ? make_f(REWARD, R) : nullptr;
    int32_t* group_id = make_i(GROUP_ID, R);
    int32_t* n_groups = make_i(N_GROUPS, 1);
    int32_t* seg = make_i(SEG_OFFSETS, groups + 1);
    int32_t* perm = make_i(PERM, R);
    float* adv = make_f(ADV, R);
    float* mean = want_stats ? make_f(MEAN, groups) : nullptr;
    float* std = want_stats ? make_f(STD, groups) : nullptr;
    int32_t* best = mixed && want_best ? make_i(BEST, groups) : nullptr;
    const int32_t *env = static_cast<const int32_t*>(ids[0]->data_ptr()), *agent = static_cast<const int32_t*>(ids[1]->data_ptr()),
                  *turn = static_cast<const int32_t*>(ids[2]->data_ptr());
    const float *r = static_cast<const float*>(reward->data_ptr()), *l = loc ? static_cast<const float*>(loc->data_ptr()) : nullptr;
    const int32_t nR = static_cast<int32_t>(R), nE = static_cast<int32_t>(n_env), nA = static_cast<int32_t>(n_agent),
                  nT = static_cast<int32_t>(n_turn), dd = static_cast<int32_t>(ddof), nm = static_cast<int32_t>(norm);
    status = mixed ? reinterpret_cast<MixedFn>(fn)(nR, nE, nA, nT, env, agent, turn, r, l, static_cast<float>(alpha),
                                                   static_cast<float>(eps_std), dd, nm, mix, group_id, n_groups, seg, perm, adv, mean,
                                                   std, best, ws, ws_bytes, stream)
                   : reinterpret_cast<GroupFn>(fn)(nR, nE, nA, nT, env, agent, turn, r, static_cast<float>(eps_std), dd, nm, group_id,
                                                   n_groups, seg, perm, adv, mean, std, ws, ws_bytes, stream);
  }
  if (status != AT_GRPO_OK) return PyLong_FromLong(status);
  THPObjectPtr dict(PyDict_New());
  if (!dict) return nullptr;
  for (int k = mixed ? REWARD : GROUP_ID; k < (mixed ? KEYS : BEST); ++k) {
    THPObjectPtr o(THPVariable_Wrap(std::move(out[k])));      // None where there is no tensor
    if (!o || PyDict_SetItem(dict.get(), g_keys[k], o.get()) != 0) return nullptr;
  }
  return dict.release();
  END_HANDLE_TH_ERRORS
}

PyMethodDef g_methods[] = {
    {"group_advantage", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(group_advantage)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  for (int k = 0; k < KEYS; ++k)
    if (!(g_keys[k] = PyUnicode_InternFromString(kKeyNames[k]))) return nullptr;
  return PyModule_Create(&g_module);
}
