// The host side of the calls that a decoding step makes several times and whose kernels are short (draft layers and the forest
// layout): checks, output tensors and the call into libdsbd.so without the interpreter in between.  From Python a draft layer
// took 17.5 us of host time, 6 of them its two launches, which is longer than its kernels.
//
// A module of its own: libdsbd.so knows nothing of torch.  binding.py holds the public functions, with their defaults, the
// fault words and the error codes' exceptions; these take every argument by position.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include "dsbd.h"

namespace {

// A tensor argument; `optional`: None stands for none.
const at::Tensor* tensor(PyObject* o, bool optional = false) {
  if (optional && o == Py_None) return nullptr;
  TORCH_CHECK_TYPE(THPVariable_Check(o), "expected a tensor");
  return &THPVariable_Unpack(o);
}
long long integer(PyObject* o) {
  PyObject* const n = PyNumber_Long(o);
  if (!n) throw python_error();
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}
int32_t int32(PyObject* o) {
  const long long v = integer(o);
  TORCH_CHECK_VALUE(v >= INT32_MIN && v <= INT32_MAX, "integer argument out of range");
  return (int32_t)v;
}
double number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw python_error();
  return v;
}
void* stream(PyObject* o) {
  void* const p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw python_error();
  return p;
}
// What the binding asserts of its arguments.
#define EXPECT(x)                                              \
  do {                                                         \
    if (!(x)) {                                                \
      PyErr_SetString(PyExc_AssertionError, #x);               \
      throw python_error();                                    \
    }                                                          \
  } while (0)

PyObject* wrap(const at::Tensor& t) {
  PyObject* const o = THPVariable_Wrap(t);
  if (!o) throw python_error();
  return o;
}

// draft_layer(beam_off, logits, logp, u, W_S, max_prompt_beams, top_k, top_p, workspace, fault, stream): the outputs (parent,
// token, logp), or an error code of the library; a workspace query that fails is the code -2 as an empty tuple.
PyObject* draft_layer(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 11, "draft_layer takes 11 arguments");
  const at::Tensor &beam_off = *tensor(args[0]), &z = *tensor(args[1]), &cum = *tensor(args[2]), &u = *tensor(args[3]);
  const int32_t W_S = int32(args[4]), top_k = int32(args[6]);
  const float top_p = (float)number(args[7]);
  const at::Tensor* const given = tensor(args[8], true);
  const at::Tensor& fault = *tensor(args[9]);
  void* const s = stream(args[10]);
  TORCH_CHECK_VALUE(z.dim() == 2, "logits_draft is [n_beams, V]");
  const int64_t P = beam_off.numel() - 1;
  EXPECT(beam_off.scalar_type() == at::kInt && z.scalar_type() == at::kFloat && z.is_contiguous());
  EXPECT(cum.scalar_type() == at::kDouble && u.scalar_type() == at::kFloat && u.is_contiguous());
  EXPECT(u.numel() == P * W_S && cum.numel() == z.size(0));
  dsbd_draft_in in;
  in.n_prompts = (int32_t)P; in.n_beams = (int32_t)z.size(0); in.max_prompt_beams = int32(args[5]); in.V = (int32_t)z.size(1);
  in.beam_off = (const int32_t*)beam_off.data_ptr(); in.logits_draft = (const float*)z.data_ptr();
  in.beam_logp_draft = (const double*)cum.data_ptr(); in.u = (const float*)u.data_ptr();
  const auto on = z.options();
  const at::Tensor parent = at::empty({P, W_S}, on.dtype(at::kInt)), token = at::empty({P, W_S}, on.dtype(at::kInt));
  const at::Tensor logp = at::empty({P, W_S}, on.dtype(at::kDouble));
  dsbd_draft_out out;
  out.parent = (int32_t*)parent.data_ptr(); out.token = (int32_t*)token.data_ptr(); out.logp_draft = (double*)logp.data_ptr();
  at::Tensor workspace;
  if (given) workspace = *given;
  else {
    const size_t bytes = dsbd_draft_layer_workspace_bytes(&in, W_S, top_k, top_p);
    if (bytes == 0) return PyTuple_New(0);
    workspace = at::empty({(int64_t)(bytes > 256 ? bytes : 256)}, on.dtype(at::kByte));
  }
  void* const ws = workspace.data_ptr();
  const size_t ws_bytes = (size_t)workspace.numel();
  int32_t* const fw = (int32_t*)fault.data_ptr();
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = dsbd_draft_layer(&in, W_S, top_k, top_p, &out, ws, ws_bytes, fw, s);
  Py_END_ALLOW_THREADS
  if (rc != DSBD_OK) return PyLong_FromLong(rc);
  PyObject* const r = PyTuple_New(3);
  if (!r) throw python_error();
  PyTuple_SET_ITEM(r, 0, wrap(parent));
  PyTuple_SET_ITEM(r, 1, wrap(token));
  PyTuple_SET_ITEM(r, 2, wrap(logp));
  return r;
  END_HANDLE_TH_ERRORS
}

// build_forest(root_off, layer_parent, layer_token, root_token, n_roots, fault, stream): (gamma, tree_prompt, tree_off,
// parent, token, draft_rank, node_of_root, node_of, max_tree_nodes), or an error code.
PyObject* build_forest(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 7, "build_forest takes 7 arguments");
  const at::Tensor& root_off = *tensor(args[0]);
  const at::Tensor *layer_parent = tensor(args[1], true), *layer_token = tensor(args[2], true), *root_token = tensor(args[3], true);
  const int64_t n_roots = integer(args[4]);
  const at::Tensor& fault = *tensor(args[5]);
  void* const s = stream(args[6]);
  const int64_t P = root_off.numel() - 1;
  const int64_t gamma = layer_parent && layer_parent->numel() > 0 ? layer_parent->size(0) : 0;
  if (gamma && P == 0) {
    PyErr_SetString(PyExc_ZeroDivisionError, "layers without prompts");
    throw python_error();
  }
  const int64_t W_S = gamma ? layer_parent->size(1) / P : 0;
  const int64_t D = gamma * P * W_S, N = n_roots + D;
  const at::Tensor* const all[4] = {&root_off, layer_parent, layer_token, root_token};
  for (const at::Tensor* t : all) EXPECT(t == nullptr || (t->scalar_type() == at::kInt && t->is_contiguous()));
  // one allocation, cut into the arrays (an array of no entries has no pointer of its own)
  const int64_t sizes[8] = {n_roots, n_roots + 1, N, N, N, n_roots, D, 1};
  int64_t total = 0;
  for (int64_t k : sizes) total += k;
  const at::Tensor buf = at::empty({total}, root_off.options().dtype(at::kInt));
  int32_t* at_ = (int32_t*)buf.data_ptr();
  at::Tensor part[8];
  int32_t* place[8];
  int64_t off = 0;
  for (int k = 0; k < 8; ++k) {
    place[k] = at_ + off;
    part[k] = k == 6 && gamma ? buf.as_strided({gamma, P * W_S}, {P * W_S, 1}, off) : buf.as_strided({sizes[k]}, {1}, off);
    off += sizes[k];
  }
  dsbd_forest_out out;
  out.tree_prompt = place[0]; out.tree_off = place[1]; out.parent = place[2]; out.token = place[3]; out.draft_rank = place[4];
  out.node_of_root = place[5]; out.node_of = place[6]; out.max_tree_nodes = place[7];
  const int32_t* const ro = (const int32_t*)root_off.data_ptr();
  const int32_t* const rt = root_token ? (const int32_t*)root_token->data_ptr() : nullptr;
  const int32_t* const lp = gamma ? (const int32_t*)layer_parent->data_ptr() : nullptr;
  const int32_t* const lt = gamma && layer_token ? (const int32_t*)layer_token->data_ptr() : nullptr;
  int32_t* const fw = (int32_t*)fault.data_ptr();
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS
  rc = dsbd_build_forest((int32_t)P, (int32_t)n_roots, (int32_t)gamma, (int32_t)W_S, ro, rt, lp, lt, &out, fw, s);
  Py_END_ALLOW_THREADS
  if (rc != DSBD_OK) return PyLong_FromLong(rc);
  PyObject* const r = PyTuple_New(9);
  if (!r) throw python_error();
  PyTuple_SET_ITEM(r, 0, PyLong_FromLongLong(gamma));
  for (int k = 0; k < 8; ++k) PyTuple_SET_ITEM(r, k + 1, wrap(part[k]));
  return r;
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"draft_layer", (PyCFunction)(void (*)(void))draft_layer, METH_FASTCALL, nullptr},
    {"build_forest", (PyCFunction)(void (*)(void))build_forest, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_dsbd_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dsbd_host(void) { return PyModule_Create(&module); }
