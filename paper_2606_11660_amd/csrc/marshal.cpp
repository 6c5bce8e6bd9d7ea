// Module descriptors of a projection call, gathered from the Python objects.
//
// A call over a model's modules passes four tensors each: checking them and
// reading their pointers, shapes and strides attribute by attribute from Python
// took 250 us for 48 modules, several times what the kernels of a short batch
// take (here: 15 us).  modules() makes the binding's checks on exact torch
// tensors and returns None as soon as one does not hold or anything is of
// another kind (a subclass, a wrapper without storage, a CPU tensor): the
// binding's own Python checks then run, and raise or accept.
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <vector>

#include "attr.h"

namespace {

struct Names {
  PyObject *a, *g, *R, *S, *out_col, *v_out, *v_in;
} names;

// a new reference, or NULL
struct Ref {
  PyObject* p;
  explicit Ref(PyObject* o) : p(o) {}
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
  ~Ref() { Py_XDECREF(p); }
};

const at::Tensor* tensor_of(PyObject* o) {
  return o && THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr;
}

// rows, width and row stride of a tensor whose last dimension is contiguous
// and whose leading dimensions are packed
bool rows_of(const at::Tensor& t, int64_t& rows, int64_t& width, int64_t& ld) {
  const int64_t n = t.dim();
  if (n < 2 || t.stride(n - 1) != 1) return false;
  rows = 1;
  for (int64_t d = 0; d < n - 1; ++d) rows *= t.size(d);
  for (int64_t d = 0; d < n - 2; ++d)
    if (t.stride(d) != t.stride(d + 1) * t.size(d + 1)) return false;
  width = t.size(n - 1);
  ld = t.stride(n - 2);
  return true;
}

bool on(const at::Tensor& t, const at::Device& dev) { return t.is_cuda() && t.device() == dev; }

// None, or a contiguous vector of `type` on dev with at least n elements
bool vector_ok(PyObject* o, at::ScalarType type, int64_t n, const at::Device& dev) {
  if (o == Py_None) return true;
  const at::Tensor* t = tensor_of(o);
  return t && t->scalar_type() == type && t->is_contiguous() && t->numel() >= n && on(*t, dev);
}

bool matrix_ok(const at::Tensor* t, at::ScalarType type, int64_t r, int64_t c, const at::Device& dev) {
  return t && t->scalar_type() == type && t->dim() == 2 && t->size(0) == r && t->size(1) == c &&
         t->is_contiguous() && on(*t, dev);
}

// an optional fp32 factor of n elements; sets *p (NULL for None)
bool factor_ok(PyObject* o, int64_t n, const at::Device& dev, const float** p) {
  *p = nullptr;
  if (!o) return false;
  if (o == Py_None) return true;
  const at::Tensor* t = tensor_of(o);
  if (!t || t->scalar_type() != at::kFloat || !t->is_contiguous() || t->numel() != n || !on(*t, dev))
    return false;
  *p = static_cast<const float*>(t->mutable_data_ptr());
  return true;
}

bool gather(PyObject* mods, PyObject* module_type, int64_t k, int64_t n_ex, int64_t T, PyObject* row_offset,
            PyObject* length, PyObject* out_o, int64_t rows_needed, std::vector<attr_module>& cm, int& dtype) {
  if (!PyList_CheckExact(mods) && !PyTuple_CheckExact(mods)) return false;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(mods);
  const at::Tensor* out = tensor_of(out_o);
  if (n < 1 || !out || !out->is_cuda() || out->scalar_type() != at::kFloat || out->dim() != 2 ||
      out->stride(1) != 1 || out->size(0) < rows_needed || n_ex < 0 || T < 1)
    return false;
  const at::Device dev = out->device();
  if (!vector_ok(row_offset, at::kLong, n_ex, dev) || !vector_ok(length, at::kInt, n_ex, dev)) return false;
  at::ScalarType type = at::kFloat;
  cm.resize((size_t)n);
  for (Py_ssize_t j = 0; j < n; ++j) {
    PyObject* m = PySequence_Fast_GET_ITEM(mods, j);
    if ((PyObject*)Py_TYPE(m) != module_type) return false;
    const Ref a(PyObject_GetAttr(m, names.a)), g(PyObject_GetAttr(m, names.g)), R(PyObject_GetAttr(m, names.R)),
        S(PyObject_GetAttr(m, names.S)), col(PyObject_GetAttr(m, names.out_col)),
        vo(PyObject_GetAttr(m, names.v_out)), vi(PyObject_GetAttr(m, names.v_in));
    const at::Tensor *ta = tensor_of(a.p), *tg = tensor_of(g.p);
    if (!ta || !tg || !col.p || !PyLong_CheckExact(col.p)) return false;
    if (j == 0) {
      type = ta->scalar_type();
      if (type != at::kFloat && type != at::kBFloat16) return false;
    }
    attr_module& c = cm[(size_t)j];
    int64_t na, ng, d_in, d_out, lda, ldg;
    if (ta->scalar_type() != type || tg->scalar_type() != type || !on(*ta, dev) || !on(*tg, dev) ||
        !rows_of(*ta, na, d_in, lda) || !rows_of(*tg, ng, d_out, ldg))
      return false;
    if (row_offset == Py_None && (na < n_ex * T || ng < n_ex * T)) return false;
    const at::Tensor *tR = tensor_of(R.p), *tS = tensor_of(S.p);
    if (!matrix_ok(tR, type, d_out, k, dev) || !matrix_ok(tS, type, d_in, k, dev)) return false;
    if (!factor_ok(vo.p, d_out, dev, &c.v_out) || !factor_ok(vi.p, d_in, dev, &c.v_in)) return false;
    c.out_col = PyLong_AsLongLong(col.p);
    if (PyErr_Occurred() || c.out_col < 0 || c.out_col > out->size(1) - k * k) return false;
    c.a = ta->mutable_data_ptr();
    c.g = tg->mutable_data_ptr();
    c.R = tR->mutable_data_ptr();
    c.S = tS->mutable_data_ptr();
    c.lda = lda;
    c.ldg = ldg;
    c.d_in = d_in;
    c.d_out = d_out;
  }
  dtype = type == at::kFloat ? ATTR_F32 : ATTR_BF16;
  return true;
}

// modules(mods, Module, k, n_examples, T, row_offset, length, out, rows_needed)
// -> (dtype code, bytearray of attr_module) or None
PyObject* py_modules(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 9) {
    PyErr_SetString(PyExc_TypeError, "modules() takes 9 arguments");
    return nullptr;
  }
  int64_t v[4];
  const int at_arg[4] = {2, 3, 4, 8};
  bool ok = true;
  for (int i = 0; ok && i < 4; ++i) {
    ok = PyLong_CheckExact(args[at_arg[i]]);
    if (ok) v[i] = PyLong_AsLongLong(args[at_arg[i]]);
    // sizes whose products stay inside 64 bits
    ok = ok && !PyErr_Occurred() && v[i] >= 0 && v[i] <= ((int64_t)1 << 31);
  }
  std::vector<attr_module> cm;
  int dtype = 0;
  try {
    ok = ok && gather(args[0], args[1], v[0], v[1], v[2], args[5], args[6], args[7], v[3], cm, dtype);
  } catch (...) {  // a tensor without storage, for one
    ok = false;
  }
  if (!ok) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  PyObject* buf = PyByteArray_FromStringAndSize(reinterpret_cast<const char*>(cm.data()),
                                                (Py_ssize_t)(cm.size() * sizeof(attr_module)));
  return buf ? Py_BuildValue("iN", dtype, buf) : nullptr;
}

PyMethodDef methods[] = {{"modules", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_modules)),
                          METH_FASTCALL, "module descriptors of a projection call, or None"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  names.a = PyUnicode_InternFromString("a");
  names.g = PyUnicode_InternFromString("g");
  names.R = PyUnicode_InternFromString("R");
  names.S = PyUnicode_InternFromString("S");
  names.out_col = PyUnicode_InternFromString("out_col");
  names.v_out = PyUnicode_InternFromString("v_out");
  names.v_in = PyUnicode_InternFromString("v_in");
  if (!names.a || !names.g || !names.R || !names.S || !names.out_col || !names.v_out || !names.v_in) return nullptr;
  return PyModule_Create(&module_def);
}
