// Native half of the Python binding (CPython module _isp_torch): argument marshalling between torch tensors and
// the C ABI (include/isp.h), and the autograd nodes.  No arithmetic here.
//
// Why it is not Python: on small graphs a call costs more on the host than on the GPU.  Marshalled through ctypes a
// SpMM of 4,096 rows took 8.8 us of host time for 5 us of kernel, and a forward + backward through a Python
// autograd.Function 48 - 115 us: the engine runs the backward on a thread of its own, and every Python statement
// there competes for the interpreter.  Measured after the move: see the comments at spmm() and at the nodes.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/utils/pybind.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <atomic>
#include <memory>
#include <mutex>
#include <vector>
#include "isp.h"

namespace {

using at::Tensor;
using torch::autograd::variable_list;

PyObject* g_check = nullptr;      // binding._check: raises IspError for a status
PyObject* g_transpose = nullptr;  // binding.csr_transpose_cached

// The stream of a call.  own: one of torch's, which live as long as the process; a stream that somebody else made may be gone when
// a handle is dropped.
struct Where {
  void* s;
  bool own;
};

// A handle as the Python object CSR owns it; destroy() on that object clears h for everybody who shares the cell.
struct Cell {
  std::atomic<isp_csr_t*> h{nullptr};
  int64_t n_rows = 0, n_cols = 0, nnz = 0;

  // The streams that calls on the handle have been put on.
  struct Use {
    void* s;
    int device;
  };
  void ran_on(Where w) {
    if (!w.own) {
      foreign.store(true, std::memory_order_relaxed);
      return;
    }
    if (w.s == last.load(std::memory_order_relaxed)) return;
    std::lock_guard<std::mutex> lock(m);
    last.store(w.s, std::memory_order_relaxed);
    for (const Use& u : uses)
      if (u.s == w.s) return;
    hipDevice_t device = 0;
    if (w.s ? hipStreamGetDevice((hipStream_t)w.s, &device) != hipSuccess : hipGetDevice(&device) != hipSuccess) {
      foreign.store(true, std::memory_order_relaxed);
      return;
    }
    uses.push_back({w.s, device});
  }
  std::atomic<bool> foreign{false};  // a call ran on a stream that is not one of torch's
  std::mutex m;
  std::vector<Use> uses;

 private:
  static inline char none;  // (the default stream is a null pointer)
  std::atomic<void*> last{&none};
};
using CellPtr = std::shared_ptr<Cell>;

// What autograd.SparseGraph keeps on this side.
struct Graph {
  CellPtr A, At;          // At: the cached transpose, once it has been built
  Tensor values;          // undefined when all entries are 1
  uint32_t version = 0;   // of `values` when the handle last read them
  PyObject* csr = nullptr;  // the CSR object (keeps the handle and every tensor it borrows alive)
  ~Graph() {
    if (csr && Py_IsInitialized()) {
      pybind11::gil_scoped_acquire gil;  // (an autograd node may be the last owner, on a thread of the engine)
      Py_DECREF(csr);
    }
  }
};
using GraphPtr = std::shared_ptr<Graph>;

const char* const CELL = "isp.cell";
const char* const GRAPH = "isp.graph";

template <class T>
void drop(PyObject* c) {
  delete static_cast<std::shared_ptr<T>*>(PyCapsule_GetPointer(c, PyCapsule_GetName(c)));
}
template <class T>
PyObject* wrap(std::shared_ptr<T> p, const char* name) {
  auto* box = new std::shared_ptr<T>(std::move(p));
  PyObject* c = PyCapsule_New(box, name, drop<T>);
  if (!c) delete box;
  return c;
}
Cell* cell_of(PyObject* c) {
  auto* p = static_cast<CellPtr*>(PyCapsule_GetPointer(c, CELL));
  return p ? p->get() : nullptr;
}

PyObject* fail(const char* what) {
  PyErr_SetString(PyExc_AssertionError, what);
  return nullptr;
}

// One dense operand: fp32 rows on the GPU, contiguous within a row.
struct Dense {
  float* p;
  int64_t rows, d, ld;
};
const char* dense_of(const Tensor& t, Dense& o) {
  if (t.dim() != 2) return "a dense operand has two dimensions";
  if (!t.is_cuda()) return "a dense operand lives on the GPU";
  if (t.scalar_type() != at::kFloat) return "a dense operand is float32";
  if (t.stride(1) != 1) return "the rows of a dense operand are contiguous";
  o.p = static_cast<float*>(t.data_ptr());
  o.rows = t.size(0);
  o.d = t.size(1);
  o.ld = o.rows > 1 ? t.stride(0) : std::max<int64_t>(t.stride(0), o.d);
  return nullptr;
}
// (THPVariable_Unpack trusts its argument: whatever comes from a caller is looked at first)
bool is_tensor(PyObject* o) {
  if (THPVariable_Check(o)) return true;
  PyErr_SetString(PyExc_TypeError, "a torch tensor is expected");
  return false;
}
bool dense_of(PyObject* o, Dense& out) {
  if (!is_tensor(o)) return false;
  const char* bad = dense_of(THPVariable_Unpack(o), out);
  if (bad) fail(bad);
  return !bad;
}

Where here() {  // the current stream of the current device
  const auto s = c10::hip::getCurrentHIPStream();
  void* const p = s.stream();
  return {p, !p || s.id() != reinterpret_cast<intptr_t>(p)};  // (the id of a stream that torch has not made is its address)
}
Where stream_of(PyObject* o) {  // None: the current one; else its address, negative if it is not one of torch's
  if (o == Py_None) return here();
  const long long p = PyLong_AsLongLong(o);
  return {reinterpret_cast<void*>(p < 0 ? -p : p), p >= 0};
}

#define ISP_ARGS(n)                                                                            \
  if (nargs != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }

template <class F>
PyObject* call(Cell* c, Where w, F&& f) {  // the library call on c's handle with the interpreter released, its status as a Python int
  isp_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f(c->h.load(), w.s);
  if (st == ISP_OK || st == ISP_EHIP) c->ran_on(w);  // (else nothing has been launched)
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// (h as a ctypes integer, n_rows, n_cols, nnz) -> cell
PyObject* py_cell(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(4)
  auto c = std::make_shared<Cell>();
  c->h = static_cast<isp_csr_t*>(PyLong_AsVoidPtr(a[0]));
  c->n_rows = PyLong_AsLongLong(a[1]);
  c->n_cols = PyLong_AsLongLong(a[2]);
  c->nnz = PyLong_AsLongLong(a[3]);
  if (PyErr_Occurred()) return nullptr;
  return wrap(std::move(c), CELL);
}
// (cell, stream): a call through ctypes on that stream has used the handle
PyObject* py_cell_ran(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(2)
  Cell* c = cell_of(a[0]);
  if (!c) return nullptr;
  const Where w = stream_of(a[1]);
  if (PyErr_Occurred()) return nullptr;
  c->ran_on(w);
  Py_RETURN_NONE;
}
// (cell) -> has a call run on a stream that is not one of torch's?
PyObject* py_cell_foreign(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(1)
  Cell* c = cell_of(a[0]);
  if (!c) return nullptr;
  return PyBool_FromLong(c->foreign.load());
}
// (cells, list, cell or None): before the list's tensors are let go.  The allocator hears of every stream that calls on the cells' handles
// ran on, and reuses the memory once those are through; the other cell (an alias's source, whose arrays the calls read) takes the
// streams over.
PyObject* py_cells_release(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(3)
  Cell* heir = nullptr;
  if (a[2] != Py_None && !(heir = cell_of(a[2]))) return nullptr;
  if (!PyList_Check(a[0]) || !PyList_Check(a[1])) return fail("lists of cells and of what they borrow");
  std::vector<Cell::Use> uses;
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(a[0]); ++i) {
    Cell* c = cell_of(PyList_GET_ITEM(a[0], i));
    if (!c) return nullptr;
    std::lock_guard<std::mutex> lock(c->m);
    uses.insert(uses.end(), c->uses.begin(), c->uses.end());
    if (heir && c->foreign.load()) heir->foreign.store(true);
  }
  for (size_t u = 0; u < uses.size(); ++u) {
    bool again = false;
    for (size_t v = 0; v < u; ++v) again |= uses[v].s == uses[u].s;
    if (again) continue;
    if (heir) heir->ran_on({uses[u].s, true});
    const auto dev = static_cast<c10::DeviceIndex>(uses[u].device);
    const auto s = uses[u].s ? c10::hip::getStreamFromExternal((hipStream_t)uses[u].s, dev) : c10::hip::getDefaultHIPStream(dev);
    for (Py_ssize_t i = 0; i < PyList_GET_SIZE(a[1]); ++i) {
      PyObject* o = PyList_GET_ITEM(a[1], i);
      // (Tensor.record_stream without the dispatcher: a mode that is active where a handle happens to go has no part in this)
      if (THPVariable_Check(o)) c10::hip::HIPCachingAllocator::recordStream(THPVariable_Unpack(o).storage().data_ptr(), s);
    }
  }
  Py_RETURN_NONE;
}
PyObject* py_cell_clear(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(1)
  Cell* c = cell_of(a[0]);
  if (!c) return nullptr;
  c->h = nullptr;
  Py_RETURN_NONE;
}

// (cell, X, Y, stream): a 4,096-row call 8.8 -> 3.3 us of host time (most of it the kernel launch)
template <isp_status (*FN)(const isp_csr_t*, const float*, int64_t, int32_t, float*, int64_t, void*)>
PyObject* py_spmm(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(4)
  Cell* c = cell_of(a[0]);
  Dense X, Y;
  if (!c || !dense_of(a[1], X) || !dense_of(a[2], Y)) return nullptr;
  if (X.rows != c->n_cols || Y.rows != c->n_rows || Y.d != X.d) return fail("X has A's columns as rows, Y its rows, both the same width");
  const Where w = stream_of(a[3]);
  if (PyErr_Occurred()) return nullptr;
  return call(c, w, [&](isp_csr_t* h, void* s) { return FN(h, X.p, X.ld, (int32_t)X.d, Y.p, Y.ld, s); });
}

// (cell, U, V, out, flags, stream)
PyObject* py_sddmm(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(6)
  Cell* c = cell_of(a[0]);
  Dense U, V;
  if (!c || !dense_of(a[1], U) || !dense_of(a[2], V)) return nullptr;
  if (!THPVariable_Check(a[3])) return fail("out is a tensor");
  const Tensor& out = THPVariable_Unpack(a[3]);
  if (U.rows != c->n_rows || V.rows != c->n_cols || V.d != U.d || out.numel() != c->nnz) return fail("U has A's rows, V its columns as rows, out one value per entry");
  const unsigned flags = (unsigned)PyLong_AsUnsignedLong(a[4]);
  const Where w = stream_of(a[5]);
  if (PyErr_Occurred()) return nullptr;
  float* o = static_cast<float*>(out.data_ptr());
  return call(c, w, [&](isp_csr_t* h, void* s) { return isp_sddmm(h, U.p, U.ld, V.p, V.ld, (int32_t)U.d, flags, o, s); });
}

// (cell, X, Y, op, stream)
PyObject* py_fusedmm(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(5)
  Cell* c = cell_of(a[0]);
  Dense X, Y;
  if (!c || !dense_of(a[1], X) || !dense_of(a[2], Y)) return nullptr;
  if (X.rows != c->n_rows || Y.rows != X.rows || Y.d != X.d) return fail("X and Y have A's rows and one width");
  const int op = (int)PyLong_AsLong(a[3]);
  const Where w = stream_of(a[4]);
  if (PyErr_Occurred()) return nullptr;
  return call(c, w, [&](isp_csr_t* h, void* s) { return isp_fusedmm(h, X.p, X.ld, (int32_t)X.d, op, Y.p, Y.ld, s); });
}

// (cell, X, dY, dX, op, stream)
PyObject* py_fusedmm_backward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(6)
  Cell* c = cell_of(a[0]);
  Dense X, G, O;
  if (!c || !dense_of(a[1], X) || !dense_of(a[2], G) || !dense_of(a[3], O)) return nullptr;
  if (G.rows != X.rows || G.d != X.d || O.rows != X.rows || O.d != X.d) return fail("X, dY and dX have one shape");
  const int op = (int)PyLong_AsLong(a[4]);
  const Where w = stream_of(a[5]);
  if (PyErr_Occurred()) return nullptr;
  return call(c, w, [&](isp_csr_t* h, void* s) { return isp_fusedmm_backward(h, X.p, X.ld, G.p, G.ld, (int32_t)X.d, op, O.p, O.ld, s); });
}

// The arg array of min / max (None: absent).
bool arg_of(PyObject* o, const Cell* c, int64_t d, bool check, int32_t** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) { fail("arg is a tensor"); return false; }
  const Tensor& t = THPVariable_Unpack(o);
  if (check && (t.scalar_type() != at::kInt || !t.is_contiguous() || t.dim() != 2 || t.size(0) != c->n_rows || t.size(1) != d)) {
    fail("arg is int32, contiguous, one row per row of A");
    return false;
  }
  *out = static_cast<int32_t*>(t.data_ptr());
  return true;
}

// (cell, X, Y, reduce, arg, stream)
PyObject* py_spmm_reduce(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(6)
  Cell* c = cell_of(a[0]);
  Dense X, Y;
  int32_t* arg;
  if (!c || !dense_of(a[1], X) || !dense_of(a[2], Y)) return nullptr;
  if (X.rows != c->n_cols || Y.rows != c->n_rows || Y.d != X.d) return fail("X has A's columns as rows, Y its rows, both the same width");
  if (!arg_of(a[4], c, X.d, true, &arg)) return nullptr;
  const int red = (int)PyLong_AsLong(a[3]);
  const Where w = stream_of(a[5]);
  if (PyErr_Occurred()) return nullptr;
  return call(c, w, [&](isp_csr_t* h, void* s) { return isp_spmm_reduce(h, X.p, X.ld, (int32_t)X.d, red, Y.p, Y.ld, arg, s); });
}

// (cell, dY, dX, reduce, arg, stream)
PyObject* py_spmm_reduce_backward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(6)
  Cell* c = cell_of(a[0]);
  Dense G, O;
  int32_t* arg;
  if (!c || !dense_of(a[1], G) || !dense_of(a[2], O)) return nullptr;
  if (G.rows != c->n_rows || O.rows != c->n_cols || O.d != G.d) return fail("dY has A's rows, dX its columns as rows, both the same width");
  if (!arg_of(a[4], c, G.d, false, &arg)) return nullptr;
  const int red = (int)PyLong_AsLong(a[3]);
  const Where w = stream_of(a[5]);
  if (PyErr_Occurred()) return nullptr;
  return call(c, w, [&](isp_csr_t* h, void* s) { return isp_spmm_reduce_backward(h, G.p, G.ld, (int32_t)G.d, red, arg, O.p, O.ld, s); });
}

// ---- autograd -------------------------------------------------------------------------------------------------
// The same operations as nodes of torch's graph.  The backward touches the interpreter only when a transpose has to
// be built or a call fails.  (4,096 rows, 32 columns, forward + backward: 112 -> 44 us of host time; a multiplication by
// a scalar takes 43 us in the same process: the rest is the engine's hand-over to its thread.)

// Raises binding.IspError for a status other than ISP_OK.
void check(isp_status st) {
  if (st == ISP_OK) return;
  pybind11::gil_scoped_acquire gil;
  PyObject* r = PyObject_CallFunction(g_check, "i", (int)st);
  Py_XDECREF(r);
  python_error e;
  e.persist();
  throw python_error(std::move(e));
}
// AssertionError, as the wrappers' own checks raise.
[[noreturn]] void assertion(const char* what) {
  pybind11::gil_scoped_acquire gil;
  PyErr_SetString(PyExc_AssertionError, what);
  python_error e;
  e.persist();
  throw python_error(std::move(e));
}
Dense dense(const Tensor& t) {
  Dense o;
  if (const char* bad = dense_of(t, o)) assertion(bad);
  return o;
}
// A library call on a cell's handle and the current stream.
template <class F>
void run(Cell& c, F&& f) {
  const Where w = here();
  const isp_status st = f(c.h.load(), w.s);
  if (st == ISP_OK || st == ISP_EHIP) c.ran_on(w);
  check(st);
}

// Everything the handle keeps of the values follows an in-place change of the tensor.
void sync_values(Graph& g) {
  if (!g.values.defined()) return;
  const uint32_t v = g.values._version();
  if (v == g.version) return;
  run(*g.A, [](isp_csr_t* h, void* s) { return isp_csr_values_changed(h, s); });
  g.version = v;
}

Cell& transpose(Graph& g) {
  sync_values(g);
  if (!g.At || !g.At->h.load()) {
    pybind11::gil_scoped_acquire gil;
    PyObject* r = PyObject_CallFunctionObjArgs(g_transpose, g.csr, nullptr);  // (At, was_cached)
    PyObject* cell = r ? PyObject_GetAttrString(PyTuple_GET_ITEM(r, 0), "_cell") : nullptr;
    if (cell) {
      if (auto* p = static_cast<CellPtr*>(PyCapsule_GetPointer(cell, CELL))) g.At = *p;
      Py_DECREF(cell);
    }
    Py_XDECREF(r);
    if (PyErr_Occurred()) {
      python_error e;
      e.persist();
      throw python_error(std::move(e));
    }
  }
  return *g.At;
}

Tensor new_like(const Tensor& t, int64_t rows, int64_t d) { return at::empty({rows, d}, t.options().requires_grad(false)); }

struct SpmmBackward : torch::autograd::Node {
  GraphPtr graph;
  torch::autograd::SavedVariable X;  // only where the values have a gradient
  bool need_dA = false;
  std::string name() const override { return "IspSpmmBackward"; }
  void release_variables() override { X.reset_data(); }
  variable_list apply(variable_list&& grads) override {
    variable_list out(2);
    if (!grads[0].defined()) return out;
    at::NoGradGuard no_grad;
    const Tensor dY = grads[0].contiguous();
    const Dense G = dense(dY);
    if (task_should_compute_output(1)) {
      out[1] = new_like(dY, graph->A->n_cols, G.d);
      const Dense O = dense(out[1]);
      run(transpose(*graph), [&](isp_csr_t* h, void* s) { return isp_spmm(h, G.p, G.ld, (int32_t)G.d, O.p, O.ld, s); });
    }
    if (need_dA && task_should_compute_output(0)) {
      const Tensor x = X.unpack();
      const Dense V = dense(x);
      out[0] = at::empty({graph->A->nnz}, dY.options());
      run(*graph->A, [&](isp_csr_t* h, void* s) { return isp_sddmm(h, G.p, G.ld, V.p, V.ld, (int32_t)G.d, 0, static_cast<float*>(out[0].data_ptr()), s); });
    }
    return out;
  }
};

struct ReduceBackward : torch::autograd::Node {
  GraphPtr graph;
  int reduce = 0;
  Tensor arg;
  std::string name() const override { return "IspSpmmReduceBackward"; }
  variable_list apply(variable_list&& grads) override {
    variable_list out(1);
    if (!grads[0].defined()) return out;
    at::NoGradGuard no_grad;
    transpose(*graph);  // built on the first backward, cached afterwards
    const Tensor dY = grads[0].contiguous();
    const Dense G = dense(dY);
    out[0] = new_like(dY, graph->A->n_cols, G.d);
    const Dense O = dense(out[0]);
    run(*graph->A, [&](isp_csr_t* h, void* s) {
      return isp_spmm_reduce_backward(h, G.p, G.ld, (int32_t)G.d, reduce, arg.defined() ? static_cast<const int32_t*>(arg.data_ptr()) : nullptr, O.p, O.ld, s);
    });
    return out;
  }
};

struct FusedBackward : torch::autograd::Node {
  GraphPtr graph;
  torch::autograd::SavedVariable X;
  std::string name() const override { return "IspFusedmmBackward"; }
  void release_variables() override { X.reset_data(); }
  variable_list apply(variable_list&& grads) override {
    variable_list out(1);
    if (!grads[0].defined()) return out;
    at::NoGradGuard no_grad;
    transpose(*graph);
    const Tensor x = X.unpack(), dY = grads[0].contiguous();
    const Dense V = dense(x), G = dense(dY);
    out[0] = new_like(x, V.rows, V.d);
    const Dense O = dense(out[0]);
    run(*graph->A, [&](isp_csr_t* h, void* s) { return isp_fusedmm_backward(h, V.p, V.ld, G.p, G.ld, (int32_t)V.d, ISP_OP_SIGMOID, O.p, O.ld, s); });
    return out;
  }
};

// The nodes have no forward-mode rule: a tangent would be lost without a word.
bool no_tangent(const Tensor& t) {
  if (!t.defined() || !t._fw_grad(/*level=*/0).defined()) return true;
  PyErr_SetString(PyExc_NotImplementedError, "the sparse operations have no forward-mode derivative");
  return false;
}

GraphPtr graph_of(PyObject* c) {
  auto* p = static_cast<GraphPtr*>(PyCapsule_GetPointer(c, GRAPH));
  if (!p) throw python_error();
  return *p;
}

// (cell of A, the CSR object, values or None) -> graph
PyObject* py_graph(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  ISP_ARGS(3)
  auto* c = static_cast<CellPtr*>(PyCapsule_GetPointer(a[0], CELL));
  if (!c || (a[2] != Py_None && !is_tensor(a[2]))) return nullptr;
  auto g = std::make_shared<Graph>();
  g->A = *c;
  Py_INCREF(a[1]);
  g->csr = a[1];
  if (a[2] != Py_None) {
    g->values = THPVariable_Unpack(a[2]);
    g->version = g->values._version();
  }
  return wrap(std::move(g), GRAPH);
  END_HANDLE_TH_ERRORS
}

PyObject* py_graph_sync(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  ISP_ARGS(1)
  sync_values(*graph_of(a[0]));
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

// (graph, values or None, X) -> Y = A X
PyObject* py_ag_spmm(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  ISP_ARGS(3)
  GraphPtr g = graph_of(a[0]);
  if ((a[1] != Py_None && !is_tensor(a[1])) || !is_tensor(a[2])) return nullptr;
  const Tensor values = a[1] == Py_None ? Tensor() : THPVariable_Unpack(a[1]);
  const Tensor x = THPVariable_Unpack(a[2]);
  if (!no_tangent(values) || !no_tangent(x)) return nullptr;
  Tensor Y;
  {
    pybind11::gil_scoped_release release;
    Tensor xc;
    {
      at::NoGradGuard no_grad;
      xc = x.contiguous();
      const Dense X = dense(xc);
      if (X.rows != g->A->n_cols) assertion("X has A's columns as rows");
      Y = new_like(xc, g->A->n_rows, X.d);
      const Dense O = dense(Y);
      sync_values(*g);
      run(*g->A, [&](isp_csr_t* h, void* s) { return isp_spmm(h, X.p, X.ld, (int32_t)X.d, O.p, O.ld, s); });
    }
    if (torch::autograd::compute_requires_grad(values, x)) {
      auto node = std::shared_ptr<SpmmBackward>(new SpmmBackward(), torch::autograd::deleteNode);
      node->set_next_edges(torch::autograd::collect_next_edges(values, x));
      node->graph = g;
      node->need_dA = values.defined() && values.requires_grad();
      if (node->need_dA) node->X = torch::autograd::SavedVariable(xc, false);
      torch::autograd::set_history(Y, node);
    }
  }
  return THPVariable_Wrap(Y);
  END_HANDLE_TH_ERRORS
}

// (graph, X, reduce) -> Y of mean / min / max
PyObject* py_ag_reduce(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  ISP_ARGS(3)
  GraphPtr g = graph_of(a[0]);
  if (!is_tensor(a[1])) return nullptr;
  const Tensor x = THPVariable_Unpack(a[1]);
  if (!no_tangent(x)) return nullptr;
  const int reduce = (int)PyLong_AsLong(a[2]);
  if (PyErr_Occurred()) return nullptr;
  Tensor Y, arg;
  {
    pybind11::gil_scoped_release release;
    {
      at::NoGradGuard no_grad;
      const Tensor xc = x.contiguous();
      const Dense X = dense(xc);
      if (X.rows != g->A->n_cols) assertion("X has A's columns as rows");
      Y = new_like(xc, g->A->n_rows, X.d);
      if (reduce != ISP_REDUCE_MEAN) arg = at::empty({g->A->n_rows, X.d}, Y.options().dtype(at::kInt));
      const Dense O = dense(Y);
      sync_values(*g);
      run(*g->A, [&](isp_csr_t* h, void* s) {
        return isp_spmm_reduce(h, X.p, X.ld, (int32_t)X.d, reduce, O.p, O.ld, arg.defined() ? static_cast<int32_t*>(arg.data_ptr()) : nullptr, s);
      });
    }
    if (torch::autograd::compute_requires_grad(x)) {
      auto node = std::shared_ptr<ReduceBackward>(new ReduceBackward(), torch::autograd::deleteNode);
      node->set_next_edges(torch::autograd::collect_next_edges(x));
      node->graph = g;
      node->reduce = reduce;
      node->arg = arg;
      torch::autograd::set_history(Y, node);
    }
  }
  return THPVariable_Wrap(Y);
  END_HANDLE_TH_ERRORS
}

// (graph, X) -> Y of the sigmoid FusedMM
PyObject* py_ag_fused(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  ISP_ARGS(2)
  GraphPtr g = graph_of(a[0]);
  if (!is_tensor(a[1])) return nullptr;
  const Tensor x = THPVariable_Unpack(a[1]);
  if (!no_tangent(x)) return nullptr;
  Tensor Y;
  {
    pybind11::gil_scoped_release release;
    Tensor xc;
    {
      at::NoGradGuard no_grad;
      xc = x.contiguous();
      const Dense X = dense(xc);
      if (X.rows != g->A->n_rows) assertion("X has A's rows");
      Y = new_like(xc, X.rows, X.d);
      const Dense O = dense(Y);
      sync_values(*g);
      run(*g->A, [&](isp_csr_t* h, void* s) { return isp_fusedmm(h, X.p, X.ld, (int32_t)X.d, ISP_OP_SIGMOID, O.p, O.ld, s); });
    }
    if (torch::autograd::compute_requires_grad(x)) {
      auto node = std::shared_ptr<FusedBackward>(new FusedBackward(), torch::autograd::deleteNode);
      node->set_next_edges(torch::autograd::collect_next_edges(x));
      node->graph = g;
      node->X = torch::autograd::SavedVariable(xc, false);
      torch::autograd::set_history(Y, node);
    }
  }
  return THPVariable_Wrap(Y);
  END_HANDLE_TH_ERRORS
}

// (binding._check, binding.csr_transpose_cached)
PyObject* py_init(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  ISP_ARGS(2)
  Py_INCREF(a[0]);
  Py_INCREF(a[1]);
  g_check = a[0];
  g_transpose = a[1];
  Py_RETURN_NONE;
}

// No C++ exception leaves an entry point: asking some tensors (vmap's, sparse ones) for strides or storage throws.
template <PyObject* (*FN)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
  try {
    return FN(self, a, nargs);
  } catch (...) {
    torch::translate_exception_to_python(std::current_exception());
    return nullptr;
  }
}

#define ISP_DEF(name, fn) {name, (PyCFunction)(void (*)(void))(PyObject * (*)(PyObject*, PyObject* const*, Py_ssize_t)) guarded<fn>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ISP_DEF("init", py_init),
    ISP_DEF("cell", py_cell),
    ISP_DEF("cell_clear", py_cell_clear),
    ISP_DEF("cell_ran", py_cell_ran),
    ISP_DEF("cell_foreign", py_cell_foreign),
    ISP_DEF("cells_release", py_cells_release),
    ISP_DEF("spmm", py_spmm<isp_spmm>),
    ISP_DEF("spmm_static_scratch", py_spmm<isp_spmm_static_scratch>),
    ISP_DEF("sddmm", py_sddmm),
    ISP_DEF("fusedmm", py_fusedmm),
    ISP_DEF("fusedmm_backward", py_fusedmm_backward),
    ISP_DEF("spmm_reduce", py_spmm_reduce),
    ISP_DEF("spmm_reduce_backward", py_spmm_reduce_backward),
    ISP_DEF("graph", py_graph),
    ISP_DEF("graph_sync", py_graph_sync),
    ISP_DEF("ag_spmm", py_ag_spmm),
    ISP_DEF("ag_reduce", py_ag_reduce),
    ISP_DEF("ag_fused", py_ag_fused),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_isp_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__isp_torch() { return PyModule_Create(&module); }
