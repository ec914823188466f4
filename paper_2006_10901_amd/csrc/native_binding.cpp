// The part of the Python binding that runs on every call: checks the tensors, takes their device
// pointers and the current stream, and calls the C entry point.  What it checks and what it raises
// is what the ctypes form of the binding did; only the cost differs.  On a 512 x 512 matrix, where
// a kernel takes 5 us, interpreted marshalling took 9 us a call and set the rate of a train of calls.
//
// bind(address, where, signature) returns a callable for one C entry point.  `signature` has one
// "kind:name" field per argument:  i = int,  f = float,  then tensors on the GPU by element type:
// I = int32, S = int16, F = float32, H = float16; a '?' before the kind (e.g. "?I:row_order") also
// takes None.  The last argument is always the stream: None (the current one), a
// torch.cuda.Stream or the handle as an int.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <string>
#include <vector>

namespace {

struct Argument { char kind; bool optional; std::string name; };

struct Entry {
  void* address;
  std::string where;
  std::vector<Argument> args;
  int form;                          // index into kForms
};

// The C entry points' parameter classes before the stream: i = int, f = float, p = pointer.
const char* const kForms[] = {"iiiipppppp", "iiiippppp", "iiiippppppip", "iippfp", "iippp"};
constexpr int kFormCount = sizeof(kForms) / sizeof(kForms[0]);

// Raised through a callback, so that the exception class lives in Python.
PyObject* g_raise_status = nullptr;

const char* dtype_name(char kind) {
  switch (kind) {
    case 'I': return "torch.int32";
    case 'S': return "torch.int16";
    case 'F': return "torch.float32";
    default: return "torch.float16";
  }
}

at::ScalarType dtype_of(char kind) {
  switch (kind) {
    case 'I': return at::kInt;
    case 'S': return at::kShort;
    case 'F': return at::kFloat;
    default: return at::kHalf;
  }
}

const char* scalar_type_name(at::ScalarType t) {
  switch (t) {
    case at::kByte: return "torch.uint8";
    case at::kChar: return "torch.int8";
    case at::kShort: return "torch.int16";
    case at::kInt: return "torch.int32";
    case at::kLong: return "torch.int64";
    case at::kHalf: return "torch.float16";
    case at::kFloat: return "torch.float32";
    case at::kDouble: return "torch.float64";
    case at::kBFloat16: return "torch.bfloat16";
    case at::kBool: return "torch.bool";
    default: return c10::toString(t);
  }
}

// int(x), reduced to 64 bits
bool as_int(PyObject* o, int64_t* out) {
  if (PyLong_CheckExact(o)) {
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
  }
  PyObject* v = PyNumber_Long(o);
  if (!v) return false;
  *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

bool as_pointer(PyObject* o, const Argument& a, void** out) {
  if (o == Py_None) {
    *out = nullptr;
    if (a.optional) return true;
    PyErr_Format(PyExc_ValueError, "%s is required", a.name.c_str());
    return false;
  }
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_ValueError, "%s must be a GPU tensor", a.name.c_str());
    return false;
  }
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda()) {
    PyErr_Format(PyExc_ValueError, "%s must be a GPU tensor", a.name.c_str());
    return false;
  }
  if (t.scalar_type() != dtype_of(a.kind)) {
    PyErr_Format(PyExc_ValueError, "%s must have dtype %s, got %s", a.name.c_str(), dtype_name(a.kind),
                 scalar_type_name(t.scalar_type()));
    return false;
  }
  if (!t.is_contiguous()) {
    PyErr_Format(PyExc_ValueError, "%s must be contiguous", a.name.c_str());
    return false;
  }
  *out = t.data_ptr();
  return true;
}

bool as_stream(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  int64_t v = 0;
  if (PyLong_Check(o)) {
    if (!as_int(o, &v)) return false;
  } else {
    PyObject* handle = PyObject_GetAttrString(o, "cuda_stream");
    if (!handle) {
      PyErr_Clear();
      if (!as_int(o, &v)) return false;
    } else {
      const bool ok = as_int(handle, &v);
      Py_DECREF(handle);
      if (!ok) return false;
    }
  }
  *out = reinterpret_cast<void*>((uintptr_t)v);
  return true;
}

constexpr int kMaxArgs = 12;         // the longest of kForms

PyObject* call_entry(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  const Entry& e = *static_cast<const Entry*>(PyCapsule_GetPointer(self, nullptr));
  const int count = (int)e.args.size();
  if (nargs != count + 1) {
    PyErr_Format(PyExc_TypeError, "%s takes %d arguments (%zd given)", e.where.c_str(), count + 1, nargs);
    return nullptr;
  }
  int i[kMaxArgs];
  void* p[kMaxArgs];
  float f = 0.f;
  int ni = 0, np = 0, status = 0;
  void* st = nullptr;
  try {
    for (int a = 0; a < count; ++a) {
      const Argument& arg = e.args[a];
      if (arg.kind == 'i') {
        int64_t v = 0;
        if (!as_int(args[a], &v)) return nullptr;
        i[ni++] = (int)v;
      } else if (arg.kind == 'f') {
        const double v = PyFloat_AsDouble(args[a]);
        if (v == -1.0 && PyErr_Occurred()) return nullptr;
        f = (float)v;
      } else if (!as_pointer(args[a], arg, &p[np++])) {
        return nullptr;
      }
    }
    if (!as_stream(args[count], &st)) return nullptr;
  } catch (const std::exception& ex) {
    PyErr_SetString(PyExc_RuntimeError, ex.what());
    return nullptr;
  }
  using P = void*;
  Py_BEGIN_ALLOW_THREADS
  switch (e.form) {
    case 0:
      status = reinterpret_cast<int (*)(int, int, int, int, P, P, P, P, P, P, P)>(e.address)(
          i[0], i[1], i[2], i[3], p[0], p[1], p[2], p[3], p[4], p[5], st);
      break;
    case 1:
      status = reinterpret_cast<int (*)(int, int, int, int, P, P, P, P, P, P)>(e.address)(
          i[0], i[1], i[2], i[3], p[0], p[1], p[2], p[3], p[4], st);
      break;
    case 2:
      status = reinterpret_cast<int (*)(int, int, int, int, P, P, P, P, P, P, int, P, P)>(e.address)(
          i[0], i[1], i[2], i[3], p[0], p[1], p[2], p[3], p[4], p[5], i[4], p[6], st);
      break;
    case 3:
      status = reinterpret_cast<int (*)(int, int, P, P, float, P, P)>(e.address)(i[0], i[1], p[0], p[1], f, p[2], st);
      break;
    default:
      status = reinterpret_cast<int (*)(int, int, P, P, P, P)>(e.address)(i[0], i[1], p[0], p[1], p[2], st);
  }
  Py_END_ALLOW_THREADS
  if (status != 0) {
    PyObject* r = PyObject_CallFunction(g_raise_status, "is", status, e.where.c_str());
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.where.c_str());
    return nullptr;
  }
  Py_RETURN_NONE;
}

PyMethodDef g_call_def = {"entry", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call_entry)), METH_FASTCALL,
                          nullptr};

PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long address = 0;
  const char *where = nullptr, *signature = nullptr;
  PyObject* raise_status = nullptr;
  if (!PyArg_ParseTuple(args, "KssO", &address, &where, &signature, &raise_status)) return nullptr;
  auto* e = new Entry;
  e->address = reinterpret_cast<void*>((uintptr_t)address);
  e->where = where;
  e->form = -1;
  std::string s(signature), form;
  for (size_t at = 0; at < s.size();) {
    size_t end = s.find(' ', at);
    if (end == std::string::npos) end = s.size();
    Argument a;
    a.optional = s[at] == '?';
    if (a.optional) ++at;
    a.kind = s[at];
    a.name = s.substr(at + 2, end - at - 2);
    form += a.kind == 'i' || a.kind == 'f' ? a.kind : 'p';
    e->args.push_back(a);
    at = end + 1;
  }
  for (int q = 0; q < kFormCount; ++q)
    if (form == kForms[q]) e->form = q;
  if (e->form < 0) {
    PyErr_Format(PyExc_ValueError, "%s: no call of the form %s", where, form.c_str());
    delete e;
    return nullptr;
  }
  Py_INCREF(raise_status);
  Py_XSETREF(g_raise_status, raise_status);
  PyObject* capsule = PyCapsule_New(e, nullptr, nullptr);
  if (!capsule) {
    delete e;
    return nullptr;
  }
  PyObject* fn = PyCFunction_New(&g_call_def, capsule);
  Py_DECREF(capsule);
  return fn;
}

PyMethodDef g_methods[] = {{"bind", bind, METH_VARARGS, "bind(address, where, signature, raise_status) -> callable"},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
