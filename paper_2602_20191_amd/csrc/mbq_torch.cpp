// The stage call of the Python binding in native code: allocates what the caller left to the binding, checks the tensors,
// hands their addresses to the C ABI.  The same work in Python (six allocations, nine argument arrays, two size queries, the
// stream's handle) took 22.6 us a call of one 2048 x 2048 linear, twice what its two launches take on the GPU.
// Nothing is kept from one call for the next.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

#include <string>

namespace {

constexpr int kMaxGroup = 16;  // more than the C ABI takes: it refuses those itself

// addresses of the library's calls and what the binding raises, handed over once by bind()
typedef int (*StageFn)(const void*, int64_t, int64_t, int, const void* const*, const void* const*, int, const void* const*,
                       const int64_t*, void* const*, void* const*, void* const*, void* const*, void*, size_t, void*, size_t, int,
                       void*);
typedef int (*StageCfgFn)(const void*, int64_t, int64_t, int, const void* const*, const void* const*, const void*,
                          const void* const*, const int64_t*, void* const*, void* const*, void* const*, void* const*, void*,
                          size_t, void*, size_t, int, void*);
struct Library {
  StageFn stage = nullptr;
  StageCfgFn stage_cfg = nullptr;
  size_t (*route_bytes)(int64_t, int64_t) = nullptr;
  size_t (*linear_bytes)(int64_t, int64_t, int64_t) = nullptr;
  const char* (*last_error)() = nullptr;
  PyObject *error = nullptr, *device = nullptr, *stream = nullptr;  // MbqError; current device, its stream's handle
};
Library lib;

struct PythonError {};  // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PythonError{};
}
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a tensor");
  return THPVariable_Unpack(o);
}
void* pointer(const at::Tensor& t) {
  if (!t.is_cuda() || !t.is_contiguous()) fail(lib.error, "tensors handed to libmbq must be contiguous device tensors");
  return t.data_ptr();
}

struct Owned {  // a reference of one's own
  PyObject* o;
  explicit Owned(PyObject* p) : o(p) {
    if (!p) throw PythonError{};
  }
  Owned(const Owned&) = delete;
  Owned& operator=(const Owned&) = delete;
  ~Owned() { Py_XDECREF(o); }
  PyObject* take() {
    PyObject* p = o;
    o = nullptr;
    return p;
  }
};
// the elements of any sequence (borrowed for as long as the object lives)
struct Items {
  Owned fast;
  explicit Items(PyObject* o) : fast(PySequence_Fast(o, "expected a sequence")) {}
  Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(fast.o); }
  PyObject* operator[](Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(fast.o, i); }
};
int64_t whole(PyObject* o) {
  Owned v(PyNumber_Long(o));
  const long long r = PyLong_AsLongLong(v.o);
  if (r == -1 && PyErr_Occurred()) throw PythonError{};
  return r;
}

// stage(X, Wr, br, blobs, Ns, routing, Y, ws_route, ws_linear, algo, cfg): routing, Y and the workspaces may be None; cfg: the
// address of an mbq_config, or 0 for the default slices
PyObject* stage_call(PyObject* const* args) {
  const at::Tensor& X = tensor(args[0]);
  const int64_t cfg = whole(args[10]);
  if (X.dim() != 2 || X.scalar_type() != at::kBFloat16) fail(PyExc_AssertionError, "X must be a bf16 matrix");
  const int64_t T = X.size(0), K = X.size(1);
  const Items Wr(args[1]), br(args[2]), blobs(args[3]), Ns(args[4]);
  const Py_ssize_t n = Ns.size();
  const auto fits = [&](const Items& items) { return cfg ? items.size() >= n : items.size() == n; };
  if (n < 1 || !fits(Wr) || !fits(br) || !fits(blobs))
    fail(PyExc_AssertionError, "Wr, br, blobs and Ns must have the same length of at least 1");
  if (n > kMaxGroup) fail(lib.error, "too many matrices for one call");
  const int P = (int)tensor(Wr[0]).size(0);
  const auto of = [&](at::ScalarType type) { return at::TensorOptions().dtype(type).device(X.device()); };

  const void *w[kMaxGroup], *b[kMaxGroup], *blob[kMaxGroup];
  void *prec[kMaxGroup], *perm[kMaxGroup], *offsets[kMaxGroup], *y[kMaxGroup];
  int64_t rows[kMaxGroup], most = 0;
  for (Py_ssize_t i = 0; i < n; ++i) {
    w[i] = pointer(tensor(Wr[i]));
    b[i] = pointer(tensor(br[i]));
    blob[i] = pointer(tensor(blobs[i]));
    rows[i] = whole(Ns[i]);
    if (rows[i] > most) most = rows[i];
  }
  // what the caller gave comes back as it is, also beyond the n that are used
  const auto given = [&](PyObject* o, const char* what) {
    Owned all(PySequence_List(o));
    if (PyList_GET_SIZE(all.o) < n) fail(PyExc_AssertionError, what);
    return all.take();
  };
  Owned routing(args[5] != Py_None ? given(args[5], "one routing per matrix") : PyList_New(n));
  if (args[5] != Py_None) {
    for (Py_ssize_t i = 0; i < PyList_GET_SIZE(routing.o); ++i) {
      Owned r(PySequence_Tuple(PyList_GET_ITEM(routing.o, i)));
      if (PyTuple_GET_SIZE(r.o) < 3) fail(PyExc_IndexError, "a routing has precisions, order and offsets");
      if (i < n) {
        prec[i] = pointer(tensor(PyTuple_GET_ITEM(r.o, 0)));
        perm[i] = pointer(tensor(PyTuple_GET_ITEM(r.o, 1)));
        offsets[i] = pointer(tensor(PyTuple_GET_ITEM(r.o, 2)));
      }
      PyList_SetItem(routing.o, i, r.take());
    }
  } else {
    for (Py_ssize_t i = 0; i < n; ++i) {
      Owned r(PyTuple_New(3));
      void** const to[3] = {&prec[i], &perm[i], &offsets[i]};
      // (the tokens of a configuration are still sorted into the default's four buckets)
      const int64_t size[3] = {T, T, cfg ? 5 : P + 1};
      for (int k = 0; k < 3; ++k) {
        at::Tensor t = at::empty({size[k]}, of(at::kInt));
        *to[k] = t.data_ptr();
        Owned o(THPVariable_Wrap(std::move(t)));
        PyTuple_SET_ITEM(r.o, k, o.take());
      }
      PyList_SET_ITEM(routing.o, i, r.take());
    }
  }
  Owned Y(args[6] != Py_None ? given(args[6], "one output per matrix") : PyList_New(n));
  for (Py_ssize_t i = 0; i < n; ++i) {
    if (args[6] != Py_None) {
      y[i] = pointer(tensor(PyList_GET_ITEM(Y.o, i)));
    } else {
      at::Tensor t = at::empty({T, rows[i]}, of(at::kFloat));
      y[i] = t.data_ptr();
      Owned o(THPVariable_Wrap(std::move(t)));
      PyList_SET_ITEM(Y.o, i, o.take());
    }
  }
  // workspaces: of the caller, or one allocation for what is missing (in use until the stream has passed the call, which is
  // as long as the allocator keeps it from others)
  void *ws_route = nullptr, *ws_linear = nullptr;
  size_t route_bytes = 0, linear_bytes = 0;
  at::Tensor own;
  if (args[7] != Py_None) {
    const at::Tensor& t = tensor(args[7]);
    ws_route = pointer(t);
    route_bytes = (size_t)t.numel();
  }
  if (args[8] != Py_None) {
    const at::Tensor& t = tensor(args[8]);
    ws_linear = pointer(t);
    linear_bytes = (size_t)t.numel();
  }
  if (!ws_route || !ws_linear) {
    size_t at_linear = 0;
    if (args[7] == Py_None) {
      route_bytes = lib.route_bytes(T, K);
      at_linear = (route_bytes + 255) / 256 * 256;
    }
    if (args[8] == Py_None) linear_bytes = lib.linear_bytes(T, most, K);
    own = at::empty({(int64_t)(at_linear + (args[8] == Py_None ? linear_bytes : 0))}, of(at::kByte));
    char* const base = static_cast<char*>(own.data_ptr());
    if (args[7] == Py_None) ws_route = base;
    if (args[8] == Py_None) ws_linear = base + at_linear;
  }
  Owned device(PyObject_CallNoArgs(lib.device));
  Owned handle(PyObject_CallFunctionObjArgs(lib.stream, device.o, nullptr));
  void* const stream = PyLong_AsVoidPtr(handle.o);
  if (!stream && PyErr_Occurred()) throw PythonError{};
  const int algo = (int)whole(args[9]);
  void* const x = pointer(X);
  int status;
  Py_BEGIN_ALLOW_THREADS;
  status = cfg ? lib.stage_cfg(x, T, K, (int)n, w, b, reinterpret_cast<const void*>((intptr_t)cfg), blob, rows, prec, perm, offsets,
                               y, ws_route, route_bytes, ws_linear, linear_bytes, algo, stream)
               : lib.stage(x, T, K, (int)n, w, b, P, blob, rows, prec, perm, offsets, y, ws_route, route_bytes, ws_linear,
                           linear_bytes, algo, stream);
  Py_END_ALLOW_THREADS;
  if (status != 0) {
    const std::string text = std::string(cfg ? "mbq_routed_linear_group_cfg" : "mbq_routed_linear_group") +
                             " failed with status " + std::to_string(status) + ": " + lib.last_error();
    fail(lib.error, text.c_str());
  }
  return PyTuple_Pack(2, routing.o, Y.o);
}

PyObject* stage(PyObject*, PyObject* const* args, Py_ssize_t count) {
  HANDLE_TH_ERRORS  // torch's errors as the Python exceptions that they are elsewhere (torch.OutOfMemoryError among them)
  try {
    if (!lib.stage) fail(PyExc_RuntimeError, "bind() comes first");
    if (count != 11) fail(PyExc_TypeError, "stage() takes 11 arguments");
    return stage_call(args);
  } catch (const PythonError&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// bind(stage, stage_cfg, route_bytes, linear_bytes, last_error, MbqError, current_device, raw_stream)
PyObject* bind(PyObject*, PyObject* args) {
  Py_ssize_t a[5];
  PyObject* o[3];
  if (!PyArg_ParseTuple(args, "nnnnnOOO", &a[0], &a[1], &a[2], &a[3], &a[4], &o[0], &o[1], &o[2])) return nullptr;
  lib.stage = reinterpret_cast<StageFn>(a[0]);
  lib.stage_cfg = reinterpret_cast<StageCfgFn>(a[1]);
  lib.route_bytes = reinterpret_cast<decltype(lib.route_bytes)>(a[2]);
  lib.linear_bytes = reinterpret_cast<decltype(lib.linear_bytes)>(a[3]);
  lib.last_error = reinterpret_cast<decltype(lib.last_error)>(a[4]);
  PyObject** const to[3] = {&lib.error, &lib.device, &lib.stream};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(o[i]);
    Py_XSETREF(*to[i], o[i]);
  }
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"stage", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(stage)), METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mbq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mbq_torch(void) { return PyModule_Create(&module); }
