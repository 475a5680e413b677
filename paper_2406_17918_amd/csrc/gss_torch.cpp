// CPython module of the binding's hot calls (enqueue, collect, step, gather): argument marshalling in C++.
//
// A minibatch of a 3-hop sampler returns nine tensors, and making them in Python (a slice and a view of the allocation
// each) took 16 us per step - as long as the whole step on the GPU (17 us on the 1,024-seed workload of the 169k-node
// graph, 3 us of which were the call itself).  Here a tensor is a TensorImpl on the allocation's storage: 0.3 us.
// The library is called through the function addresses of the ctypes handle, so that there is one copy of it in the
// process, and without the GIL, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "gss.h"

namespace {

struct Lib {
  decltype(&gss_step) step = nullptr;
  decltype(&gss_step_async) step_async = nullptr;
  decltype(&gss_step_wait) step_wait = nullptr;
  decltype(&gss_gather_rows) gather_rows = nullptr;
} lib;

// seeds, fanouts, step, seed_type of a call
struct StepArgs {
  gss_sampler* handle;
  const int32_t* seeds;
  int32_t num_seeds, seed_type, num_layers;
  int32_t fanouts[GSS_MAX_LAYERS + 1];
  int64_t step;
};

bool as_i32(PyObject* o, int32_t* out) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) return false;
  if (v < INT32_MIN || v > INT32_MAX) { PyErr_SetString(PyExc_OverflowError, "a 32-bit integer is expected"); return false; }
  *out = (int32_t)v;
  return true;
}

// (handle, seeds, fanouts, step, seed_type)
bool parse_step(PyObject* const* a, StepArgs* s) {
  s->handle = static_cast<gss_sampler*>(PyLong_AsVoidPtr(a[0]));
  if (PyErr_Occurred()) return false;
  if (!THPVariable_Check(a[1])) { PyErr_SetString(PyExc_TypeError, "seeds: a torch tensor is expected"); return false; }
  const at::Tensor& t = THPVariable_Unpack(a[1]);
  s->num_seeds = (int32_t)t.numel();
  s->seeds = s->num_seeds ? static_cast<const int32_t*>(t.data_ptr()) : nullptr;
  PyObject* fast = PySequence_Fast(a[2], "fanouts: a sequence of integers is expected");
  if (!fast) return false;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(fast);
  s->num_layers = (int32_t)(n <= GSS_MAX_LAYERS ? n : GSS_MAX_LAYERS + 1);   // (one more than the library takes: it refuses)
  bool ok = true;
  for (int32_t i = 0; i < s->num_layers && ok; ++i) ok = as_i32(PySequence_Fast_GET_ITEM(fast, i), &s->fanouts[i]);
  Py_DECREF(fast);
  if (!ok) return false;
  s->step = PyLong_AsLongLong(a[3]);
  if (s->step == -1 && PyErr_Occurred()) return false;
  return as_i32(a[4], &s->seed_type);
}

bool nargs_are(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected", want);
  return false;
}

// int32 tensor of n elements at `ptr`, sharing the storage of the allocation live[ptr] (any tensor that covers it).
PyObject* view_i32(PyObject* live, const void* ptr, int64_t n, const at::Tensor& empty) {
  if (!ptr || n == 0) return THPVariable_Wrap(empty.alias());
  PyObject* key = PyLong_FromVoidPtr(const_cast<void*>(ptr));
  PyObject* owner = key ? PyDict_GetItemWithError(live, key) : nullptr;    // borrowed
  if (!owner || !THPVariable_Check(owner)) {
    if (key && !PyErr_Occurred()) PyErr_SetObject(PyExc_KeyError, key);
    Py_XDECREF(key);
    return nullptr;
  }
  Py_DECREF(key);
  const at::Tensor& base = THPVariable_Unpack(owner);
  const int64_t have = (int64_t)base.nbytes();
  if (have < 4 * n) {                          // (the library reported more elements than the buffer it asked for holds)
    PyErr_Format(PyExc_ValueError, "output of %lld int32 in an allocation of %lld bytes", (long long)n, (long long)have);
    return nullptr;
  }
  const int64_t offset = (int64_t)base.storage_offset() * (int64_t)base.itemsize();
  if (offset % 4 != 0) { PyErr_SetString(PyExc_ValueError, "an allocation is not aligned to int32"); return nullptr; }
  at::Tensor t = at::detail::make_tensor<c10::TensorImpl>(c10::Storage(base.storage()), base.key_set(),
                                                          caffe2::TypeMeta::Make<int32_t>());
  t.unsafeGetTensorImpl()->set_storage_offset(offset / 4);
  t.unsafeGetTensorImpl()->set_sizes_contiguous({n});
  return THPVariable_Wrap(std::move(t));
}

bool put(PyObject* list, Py_ssize_t i, PyObject* item) {     // steals the item
  if (!item) return false;
  PyList_SET_ITEM(list, i, item);
  return true;
}

// The Block of one layer: block_type(num_dst, num_src, src_nodes, num_edges, src_local, dst_local), lists per node type
// and per relation.
PyObject* make_block(const gss_blocks& b, int l, PyObject* live, PyObject* block_type, const at::Tensor& empty) {
  const int T = b.num_node_types, R = b.num_relations;
  PyObject* f[6];
  for (int i = 0; i < 6; ++i) f[i] = PyList_New(i < 3 ? T : R);
  bool ok = f[0] && f[1] && f[2] && f[3] && f[4] && f[5];
  for (int t = 0; t < T && ok; ++t) {
    const gss_block_nodes& n = b.nodes[l * T + t];
    ok = put(f[0], t, PyLong_FromLong(n.num_dst)) && put(f[1], t, PyLong_FromLong(n.num_src)) &&
         put(f[2], t, view_i32(live, n.src_nodes, n.num_src, empty));
  }
  for (int r = 0; r < R && ok; ++r) {
    const gss_block_edges& e = b.edges[l * R + r];
    ok = put(f[3], r, PyLong_FromLong(e.num_edges)) && put(f[4], r, view_i32(live, e.src_local, e.num_edges, empty)) &&
         put(f[5], r, view_i32(live, e.dst_local, e.num_edges, empty));
  }
  PyObject* block = ok ? PyObject_Vectorcall(block_type, f, 6, nullptr) : nullptr;
  for (PyObject* o : f) Py_XDECREF(o);
  return block;
}

PyObject* make_blocks(const gss_blocks& b, PyObject* live, PyObject* block_type, PyObject* empty) {
  if (!PyDict_Check(live) || !THPVariable_Check(empty)) { PyErr_SetString(PyExc_TypeError, "live: dict, empty: tensor"); return nullptr; }
  const at::Tensor& e = THPVariable_Unpack(empty);
  PyObject* out = PyList_New(b.num_layers);
  if (!out) return nullptr;
  for (int l = 0; l < b.num_layers; ++l)
    if (!put(out, l, make_block(b, l, live, block_type, e))) { Py_DECREF(out); return nullptr; }
  return out;
}

// step_async(handle, seeds, fanouts, step, seed_type) -> status
PyObject* py_step_async(PyObject*, PyObject* const* a, Py_ssize_t n) {
  StepArgs s;
  if (!nargs_are(n, 5) || !parse_step(a, &s)) return nullptr;
  gss_status st;
  Py_BEGIN_ALLOW_THREADS
  st = lib.step_async(s.handle, s.seeds, s.num_seeds, s.seed_type, s.fanouts, s.num_layers, s.step);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// step_wait(handle, live, block_type, empty) -> list of blocks, or a status other than GSS_OK
PyObject* py_step_wait(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!nargs_are(n, 4)) return nullptr;
  gss_sampler* h = static_cast<gss_sampler*>(PyLong_AsVoidPtr(a[0]));
  if (PyErr_Occurred()) return nullptr;
  gss_blocks b;
  gss_status st;
  Py_BEGIN_ALLOW_THREADS
  st = lib.step_wait(h, &b);
  Py_END_ALLOW_THREADS
  return st == GSS_OK ? make_blocks(b, a[1], a[2], a[3]) : PyLong_FromLong(st);
}

// step(handle, seeds, fanouts, step, seed_type, live, block_type, empty) -> as step_wait
PyObject* py_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  StepArgs s;
  if (!nargs_are(n, 8) || !parse_step(a, &s)) return nullptr;
  gss_blocks b;
  gss_status st;
  Py_BEGIN_ALLOW_THREADS
  st = lib.step(s.handle, s.seeds, s.num_seeds, s.seed_type, s.fanouts, s.num_layers, s.step, &b);
  Py_END_ALLOW_THREADS
  return st == GSS_OK ? make_blocks(b, a[5], a[6], a[7]) : PyLong_FromLong(st);
}

// gather_rows(table, ids, out) -> status, on the current stream of the table's device; the tensors' devices, types and sizes
// are checked here
PyObject* py_gather_rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!nargs_are(n, 3)) return nullptr;
  for (int i = 0; i < 3; ++i)
    if (!THPVariable_Check(a[i])) { PyErr_SetString(PyExc_TypeError, "gather_rows: torch tensors are expected"); return nullptr; }
  const at::Tensor &table = THPVariable_Unpack(a[0]), &ids = THPVariable_Unpack(a[1]), &out = THPVariable_Unpack(a[2]);
  const int64_t count = ids.numel(), values = table.numel();
  if (!(table.is_cuda() && ids.is_cuda() && ids.scalar_type() == at::kInt && table.is_contiguous() && ids.is_contiguous() &&
        table.dim() >= 1 && out.is_contiguous() && out.scalar_type() == table.scalar_type() &&
        out.numel() * table.size(0) == count * values)) {
    PyErr_SetString(PyExc_AssertionError, "gather_rows: table [N, ...], int32 ids and out, contiguous, on the GPU");
    return nullptr;
  }
  int64_t row_bytes = (int64_t)table.itemsize();
  for (int64_t d = 1; d < table.dim(); ++d) row_bytes *= table.size(d);
  void* const stream = c10::hip::getCurrentHIPStream(table.device().index()).stream();
  gss_status st;
  Py_BEGIN_ALLOW_THREADS
  st = lib.gather_rows(values ? table.data_ptr() : nullptr, table.size(0), row_bytes,
                       count ? static_cast<const int32_t*>(ids.data_ptr()) : nullptr, count, count ? out.data_ptr() : nullptr, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// bind(step, step_async, step_wait, gather_rows): addresses of the library's functions
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!nargs_are(n, 4)) return nullptr;
  void* p[4];
  for (int i = 0; i < 4; ++i) p[i] = PyLong_AsVoidPtr(a[i]);
  if (PyErr_Occurred()) return nullptr;
  lib.step = reinterpret_cast<decltype(lib.step)>(p[0]);
  lib.step_async = reinterpret_cast<decltype(lib.step_async)>(p[1]);
  lib.step_wait = reinterpret_cast<decltype(lib.step_wait)>(p[2]);
  lib.gather_rows = reinterpret_cast<decltype(lib.gather_rows)>(p[3]);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind), FAST(step), FAST(step_async), FAST(step_wait), FAST(gather_rows), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "gss_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_gss_torch(void) { return PyModule_Create(&module); }
