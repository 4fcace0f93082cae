// Host side of the Python binding: the tensor checks of a step and the pointer
// arrays it passes to libprm, natively.  In Python they cost about 0.4 us a
// tensor, four times the GPU time of an AdamW step over a few hundred small
// tensors (880 tensors: 350 us against 90).
//
// spec(dims, dtype, shapes): what a list of tensors has to be; dims a list of
// tuples (shapes true: whole shapes) or of ints (element counts), dtype 0 fp32,
// 1 bf16.
// pointers(spec, tensors, address): checks every entry, every time, and writes
// its data pointer to the array at `address`.  True if all of them are plain
// contiguous device tensors as specified; False for anything else (raw
// pointers, None, other types, tensors that are wrong or under a transform), and
// the caller's own checks then say what is wrong or take it.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <vector>

namespace {

struct Spec {
  bool shapes = false;
  at::ScalarType dtype = at::kFloat;
  std::vector<std::vector<int64_t>> dims;
};

constexpr const char* kName = "prm.spec";

void spec_free(PyObject* o) { delete static_cast<Spec*>(PyCapsule_GetPointer(o, kName)); }

PyObject* make_spec(PyObject*, PyObject* args) {
  PyObject* list;
  int dtype, shapes;
  if (!PyArg_ParseTuple(args, "O!ip", &PyList_Type, &list, &dtype, &shapes)) return nullptr;
  auto* s = new Spec();
  s->shapes = shapes;
  s->dtype = dtype == 1 ? at::kBFloat16 : at::kFloat;
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(list); ++i) {
    PyObject* e = PyList_GET_ITEM(list, i);
    std::vector<int64_t> d;
    if (shapes && PyTuple_Check(e)) {
      for (Py_ssize_t k = 0; k < PyTuple_GET_SIZE(e); ++k) d.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(e, k)));
    } else {
      d.push_back(PyLong_AsLongLong(e));
    }
    s->dims.push_back(std::move(d));
  }
  if (PyErr_Occurred()) {
    delete s;
    return nullptr;
  }
  return PyCapsule_New(s, kName, spec_free);
}

PyObject* g_parameter = nullptr;  // torch.nn.Parameter

// A tensor whose metadata and pointer are its own: no subclass (those answer for
// themselves in Python), a storage, no functional transform's wrapper.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o) && (PyObject*)Py_TYPE(o) != g_parameter) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.has_storage() || t.layout() != at::kStrided) return nullptr;
  if (t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                               c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                               c10::DispatchKey::ZeroTensor})))
    return nullptr;
  return &t;
}

PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) {
    PyErr_SetString(PyExc_TypeError, "pointers(spec, tensors, address)");
    return nullptr;
  }
  const auto* s = static_cast<const Spec*>(PyCapsule_GetPointer(args[0], kName));
  if (!s) return nullptr;
  PyObject* xs = args[1];
  auto* out = static_cast<void**>(PyLong_AsVoidPtr(args[2]));
  if (!out && PyErr_Occurred()) return nullptr;
  if (!PyList_CheckExact(xs) && !PyTuple_CheckExact(xs)) Py_RETURN_FALSE;
  if ((size_t)PySequence_Fast_GET_SIZE(xs) != s->dims.size()) Py_RETURN_FALSE;
  try {
    for (size_t i = 0; i < s->dims.size(); ++i) {
      const at::Tensor* t = plain(PySequence_Fast_GET_ITEM(xs, i));
      if (!t || !t->is_cuda() || t->scalar_type() != s->dtype || !t->is_contiguous()) Py_RETURN_FALSE;
      if (s->shapes ? t->sizes() != c10::IntArrayRef(s->dims[i]) : t->numel() != s->dims[i][0]) Py_RETURN_FALSE;
      out[i] = t->data_ptr();
    }
  } catch (...) {
    Py_RETURN_FALSE;  // the Python checks raise what there is to raise
  }
  Py_RETURN_TRUE;
}

PyMethodDef kMethods[] = {
    {"spec", make_spec, METH_VARARGS, "spec(dims, dtype, shapes): what a list of tensors has to be"},
    {"pointers", (PyCFunction)(void (*)(void))pointers, METH_FASTCALL, "pointers(spec, tensors, address) -> bool"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  PyObject* nn = PyImport_ImportModule("torch.nn");
  if (!nn) return nullptr;
  g_parameter = PyObject_GetAttrString(nn, "Parameter");
  Py_DECREF(nn);
  if (!g_parameter) return nullptr;
  return PyModule_Create(&kModule);
}
