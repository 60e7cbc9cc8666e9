// Python boundary of the calls a training loop makes every iteration: torch tensors in, one C-ABI call out.
//
// What bounds a call on a small batch is the host: the step of a 32-sample batch takes 12 us of kernels and 7 us of
// launching, and took 12 us more when its dozen tensors were checked and turned into pointers in Python (two torch
// method calls and a ctypes object each, 2 us for the current stream alone; 19.3 us per step then, launch included).
// Here a tensor costs a few nanoseconds.  The checks and their messages are those of per.py; results of the C-ABI
// calls are returned as they are and turned into exceptions there.
//
// As under ctypes, the interpreter lock is released while the library runs.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdexcept>
#include <string>

#include "../../include/per.h"

namespace {

struct Raised {};   // a Python exception is set

[[noreturn]] void raise_value(const std::string& what) {
  PyErr_SetString(PyExc_ValueError, what.c_str());
  throw Raised{};
}

const at::Tensor* tensor(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor or None, got %.100s", Py_TYPE(o)->tp_name);
    throw Raised{};
  }
  return &THPVariable_Unpack(o);
}

[[noreturn]] void raise_dtype(const at::Tensor& t, at::ScalarType want) {
  PyObject* o = THPVariable_Wrap(t);
  PyObject* got = o ? PyObject_GetAttrString(o, "dtype") : nullptr;
  if (got) PyErr_Format(PyExc_ValueError, "expected dtype %s, got %S", want == at::kFloat ? "torch.float32" : "torch.int32", got);
  Py_XDECREF(got);
  Py_XDECREF(o);
  throw Raised{};
}

// Device address of a contiguous tensor of the given type (Undefined: any); null for None.
void* address(const at::Tensor* t, at::ScalarType want = at::ScalarType::Undefined) {
  if (!t) return nullptr;
  if (!t->is_cuda() || !t->is_contiguous()) raise_value("expected a contiguous device tensor");
  if (want != at::ScalarType::Undefined && t->scalar_type() != want)
    raise_dtype(*t, want);
  return t->data_ptr();
}
float* f32(const at::Tensor* t) { return static_cast<float*>(address(t, at::kFloat)); }
uint32_t* u32(const at::Tensor* t) { return static_cast<uint32_t*>(address(t, at::kInt)); }
float* f32(PyObject* o) { return f32(tensor(o)); }
uint32_t* u32(PyObject* o) { return u32(tensor(o)); }

// Number of elements; None is refused (where an argument may be left out, the caller asks for None first).
uint64_t count(PyObject* o) {
  const at::Tensor* t = tensor(o);
  if (!t) {
    PyErr_SetString(PyExc_TypeError, "expected a tensor, got None");
    throw Raised{};
  }
  return (uint64_t)t->numel();
}

// Counts may be any whole number (NumPy's are not Python ints).
uint32_t whole(PyObject* o) {
  PyObject* i = PyNumber_Index(o);
  if (!i) throw Raised{};
  const unsigned long v = PyLong_AsUnsignedLong(i);
  Py_DECREF(i);
  if (v == (unsigned long)-1 && PyErr_Occurred()) throw Raised{};
  if (v > 0xFFFFFFFFul) {
    PyErr_SetString(PyExc_OverflowError, "count does not fit 32 bits");
    throw Raised{};
  }
  return (uint32_t)v;
}
double real(PyObject* o) {   // as float(o)
  if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
  PyObject* f = PyNumber_Float(o);
  if (!f) throw Raised{};
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}

struct Calls {
  PyObject_HEAD
  per_t* h;
  uint64_t T;
  uint32_t n_fields;
  uint64_t width[PER_MAX_FIELDS];
  c10::DeviceIndex device;
};

void* stream_of(const Calls* c) { return c10::hip::getCurrentHIPStream(c->device).stream(); }

// Addresses of one tensor (or None) per payload field, `rows` rows per tree each.
struct Fields {
  void* at[PER_MAX_FIELDS] = {};
  void** table = nullptr;
  Fields(const Calls* c, PyObject* list, uint64_t rows) {
    if (list == Py_None) return;
    PyObject* seq = PySequence_Fast(list, "one tensor (or None) per payload field is required");
    if (!seq) throw Raised{};
    struct Drop { PyObject* o; ~Drop() { Py_DECREF(o); } } drop{seq};
    if (PySequence_Fast_GET_SIZE(seq) != (Py_ssize_t)c->n_fields) raise_value("one tensor (or None) per payload field is required");
    for (uint32_t f = 0; f < c->n_fields; ++f) {
      const at::Tensor* t = tensor(PySequence_Fast_GET_ITEM(seq, f));
      if (!t) continue;
      if ((uint64_t)t->nbytes() != c->T * rows * c->width[f])
        raise_value("field " + std::to_string(f) + ": expected " + std::to_string(c->T) + "x" + std::to_string(rows) + "x" +
                    std::to_string(c->width[f]) + " bytes");
      at[f] = address(t);
    }
    table = at;
  }
  const void* const* source() const { return const_cast<const void* const*>(table); }
};

template <typename F>
PyObject* unlocked(F call) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

void need(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  throw Raised{};
}

// Batch per tree: from the uniforms, or given where the call draws its own.
uint32_t batch(const Calls* c, PyObject* u, PyObject* B) {
  if (u == Py_None) {
    if (B == Py_None) raise_value("without uniforms the batch size B must be given");
    return whole(B);
  }
  return (uint32_t)(count(u) / c->T);
}

using Args = PyObject* const*;

// (n, rows, prio, out_idx, protect)
PyObject* do_insert(Calls* c, Args a, Py_ssize_t n_args) {
  need(n_args, 5);
  const uint32_t n = whole(a[0]);
  Fields rows(c, a[1], n);
  if (a[2] != Py_None && count(a[2]) != c->T * n) raise_value("prio must hold T*n values");
  if (a[3] != Py_None && count(a[3]) != c->T * n) raise_value("out_idx must hold T*n values");
  const float* prio = f32(a[2]);
  uint32_t* out = u32(a[3]);
  void* s = stream_of(c);
  if (a[4] == Py_None) return unlocked([&] { return per_insert(c->h, n, rows.source(), prio, out, s); });
  const uint32_t n_protect = (uint32_t)(count(a[4]) / c->T);
  const uint32_t* protect = u32(a[4]);
  return unlocked([&] { return per_insert_protected(c->h, n, rows.source(), prio, out, n_protect, protect, s); });
}

// (u, beta, out_idx, out_weight, out_prio, rows_out, B, upd_idx, upd_prio): upd_idx None: no update
PyObject* do_sample(Calls* c, Args a, Py_ssize_t n_args) {
  need(n_args, 9);
  const uint32_t B = batch(c, a[0], a[6]);
  if (a[0] != Py_None && count(a[0]) != c->T * B) raise_value("u must hold T*B values");
  const float beta = (float)real(a[1]);
  const float* u = f32(a[0]);
  uint32_t* idx = u32(a[2]);
  float *w = f32(a[3]), *v = f32(a[4]);
  Fields rows(c, a[5], B);
  const bool update = a[7] != Py_None || a[8] != Py_None;
  const uint64_t n = update ? count(a[7]) : 0;
  if (update && (a[8] == Py_None || count(a[8]) != n)) raise_value("update idx and prio must have the same number of elements");
  const uint32_t* ui = u32(a[7]);
  const float* up = f32(a[8]);
  void* s = stream_of(c);
  if (update) {
    return unlocked([&] { return per_sample_gather_update(c->h, B, beta, u, idx, w, v, rows.table, (uint32_t)(n / c->T), ui, up, s); });
  }
  if (!rows.table) return unlocked([&] { return per_sample(c->h, B, beta, u, idx, w, v, s); });
  return unlocked([&] { return per_sample_gather(c->h, B, beta, u, idx, w, v, rows.table, s); });
}

// (u, beta, upd_prio, upd_pos, out_idx, out_weight, out_prio, rows_out, B, insert): insert None or (n, rows, prio, out_idx)
PyObject* do_step(Calls* c, Args a, Py_ssize_t n_args) {
  need(n_args, 10);
  const uint32_t B = batch(c, a[0], a[8]);
  if (a[2] == Py_None || count(a[2]) != c->T * B || (a[3] != Py_None && count(a[3]) != c->T * B))
    raise_value("upd_prio and upd_pos must hold T*B values");
  const float beta = (float)real(a[1]);
  const float* u = f32(a[0]);
  const float* up = f32(a[2]);
  const uint32_t* pos = u32(a[3]);
  uint32_t* idx = u32(a[4]);
  float *w = f32(a[5]), *v = f32(a[6]);
  Fields rows(c, a[7], B);
  void* s = stream_of(c);
  if (a[9] == Py_None) return unlocked([&] { return per_step(c->h, B, beta, u, idx, w, v, rows.table, up, pos, s); });
  PyObject* ins = PySequence_Fast(a[9], "insert must be (n, rows, prio, out_idx)");
  if (!ins) throw Raised{};
  struct Drop { PyObject* o; ~Drop() { Py_DECREF(o); } } drop{ins};
  if (PySequence_Fast_GET_SIZE(ins) != 4) raise_value("insert must be (n, rows, prio, out_idx)");
  PyObject** it = PySequence_Fast_ITEMS(ins);
  const uint32_t n = whole(it[0]);
  Fields src(c, it[1], n);
  if (it[2] != Py_None && count(it[2]) != c->T * n) raise_value("the insertion's prio must hold T*n values");
  if (it[3] != Py_None && count(it[3]) != c->T * n) raise_value("the insertion's out_idx must hold T*n values");
  const float* ip = f32(it[2]);
  uint32_t* io = u32(it[3]);
  return unlocked([&] {
    return per_insert_step(c->h, n, src.source(), ip, io, B, beta, u, idx, w, v, rows.table, up, pos, s);
  });
}

// (idx, out): out holds one tensor or None per field
PyObject* do_gather(Calls* c, Args a, Py_ssize_t n_args) {
  need(n_args, 2);
  const uint32_t B = (uint32_t)(count(a[0]) / c->T);
  Fields rows(c, a[1], B);
  const uint32_t* idx = u32(a[0]);
  void* s = stream_of(c);
  return unlocked([&] { return per_gather(c->h, B, idx, rows.table, s); });
}

uint32_t pairs(const Calls* c, PyObject* idx, PyObject* val, const char* what) {
  const uint64_t n = count(idx);
  if (val == Py_None || count(val) != n) raise_value(std::string("idx and ") + what + " must have the same number of elements");
  return (uint32_t)(n / c->T);
}

PyObject* do_update(Calls* c, Args a, Py_ssize_t n_args) {   // (idx, prio)
  need(n_args, 2);
  const uint32_t B = pairs(c, a[0], a[1], "prio");
  const uint32_t* idx = u32(a[0]);
  const float* v = f32(a[1]);
  void* s = stream_of(c);
  return unlocked([&] { return per_update(c->h, B, idx, v, s); });
}
PyObject* do_update_td(Calls* c, Args a, Py_ssize_t n_args) {   // (idx, td, eps, alpha)
  need(n_args, 4);
  const uint32_t B = pairs(c, a[0], a[1], "td");
  const uint32_t* idx = u32(a[0]);
  const float* v = f32(a[1]);
  const double eps = real(a[2]), alpha = real(a[3]);
  void* s = stream_of(c);
  return unlocked([&] { return per_update_td(c->h, B, idx, v, eps, alpha, s); });
}
PyObject* do_update_delta(Calls* c, Args a, Py_ssize_t n_args) {   // (idx, delta)
  need(n_args, 2);
  const uint32_t B = pairs(c, a[0], a[1], "delta");
  const uint32_t* idx = u32(a[0]);
  const float* v = f32(a[1]);
  void* s = stream_of(c);
  return unlocked([&] { return per_update_delta(c->h, B, idx, v, s); });
}
PyObject* do_get_priority(Calls* c, Args a, Py_ssize_t n_args) {   // (idx, out)
  need(n_args, 2);
  const uint32_t n = (uint32_t)(count(a[0]) / c->T);
  const uint32_t* idx = u32(a[0]);
  float* out = f32(a[1]);
  void* s = stream_of(c);
  return unlocked([&] { return per_get_priority(c->h, n, idx, out, s); });
}

// (u, beta, out_idx, out_weight, out_prio, rows_out, upd_prio, upd_idx, n_insert, ins_rows, ins_prio)
PyObject* do_run_steps(Calls* c, Args a, Py_ssize_t n_args) {
  need(n_args, 11);
  const at::Tensor* u = tensor(a[0]);
  const at::Tensor* beta = tensor(a[1]);
  if (!u || !beta || u->dim() < 1) raise_value("u must be [steps, T, B] and beta [steps]");
  const uint64_t steps = (uint64_t)u->size(0), B = (uint64_t)u->size(-1), n = (uint64_t)u->numel();
  if (n != steps * c->T * B || (uint64_t)beta->numel() != steps) raise_value("u must be [steps, T, B] and beta [steps]");
  const char* const names[5] = {"out_idx", "out_weight", "out_prio", "upd_prio", "upd_idx"};
  const int at[5] = {2, 3, 4, 6, 7};
  for (int i = 0; i < 5; ++i)
    if (a[at[i]] != Py_None && count(a[at[i]]) != n) raise_value(std::string(names[i]) + " must hold steps*T*B values");
  const uint32_t n_insert = whole(a[8]);
  if (a[10] != Py_None && count(a[10]) != steps * c->T * n_insert) raise_value("ins_prio must hold steps*T*n_insert values");
  per_stream_io io{};
  io.struct_size = sizeof(io);
  auto table = [&](PyObject* list, uint64_t rows, void** where) -> void** {   // (as Fields, the list of steps in front)
    if (list == Py_None) return nullptr;
    PyObject* seq = PySequence_Fast(list, "one tensor (or None) per payload field is required");
    if (!seq) throw Raised{};
    struct Drop { PyObject* o; ~Drop() { Py_DECREF(o); } } drop{seq};
    if (PySequence_Fast_GET_SIZE(seq) != (Py_ssize_t)c->n_fields) raise_value("one tensor (or None) per payload field is required");
    for (uint32_t f = 0; f < c->n_fields; ++f) {
      const at::Tensor* t = tensor(PySequence_Fast_GET_ITEM(seq, f));
      if (!t) continue;
      if ((uint64_t)t->nbytes() != steps * c->T * rows * c->width[f])
        raise_value("field " + std::to_string(f) + ": expected steps*T*rows*" + std::to_string(c->width[f]) + " bytes");
      where[f] = address(t);
    }
    return where;
  };
  void *ins[PER_MAX_FIELDS] = {}, *rows[PER_MAX_FIELDS] = {};
  io.d_ins_rows = const_cast<const void* const*>(table(a[9], n_insert, ins));
  io.d_ins_prio = f32(a[10]);
  io.d_u = f32(u);
  io.d_beta = f32(beta);
  io.d_out_idx = u32(a[2]);
  io.d_out_weight = f32(a[3]);
  io.d_out_prio = f32(a[4]);
  io.d_rows_out = table(a[5], B, rows);
  io.d_upd_idx = u32(a[7]);
  io.d_upd_prio = f32(a[6]);
  void* s = stream_of(c);
  return unlocked([&] { return per_run_steps(c->h, (uint32_t)steps, n_insert, (uint32_t)B, &io, s); });
}

// Every method: C++ and library errors become Python exceptions, nothing is thrown past the interpreter.
template <PyObject* (*F)(Calls*, Args, Py_ssize_t)>
PyObject* method(PyObject* self, Args a, Py_ssize_t n) {
  try {
    Calls* c = reinterpret_cast<Calls*>(self);
    if (!c->h) raise_value("no buffer");   // (an object that __init__ has not been through)
    return F(c, a, n);
  } catch (const Raised&) {
  } catch (const std::exception& e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}
template <PyObject* (*F)(Calls*, Args, Py_ssize_t)>
constexpr PyMethodDef entry(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<F>)), METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {
    entry<do_insert>("insert"), entry<do_sample>("sample"), entry<do_step>("step"), entry<do_gather>("gather"),
    entry<do_update>("update"), entry<do_update_td>("update_td"), entry<do_update_delta>("update_delta"),
    entry<do_get_priority>("get_priority"), entry<do_run_steps>("run_steps"), {nullptr, nullptr, 0, nullptr}};

int init(PyObject* self, PyObject* args, PyObject*) {   // (handle, n_trees, field widths, device index)
  Calls* c = reinterpret_cast<Calls*>(self);
  unsigned long long h, T;
  PyObject* widths;
  int device;
  if (!PyArg_ParseTuple(args, "KKO!i", &h, &T, &PyTuple_Type, &widths, &device)) return -1;
  if (!h || !T || PyTuple_GET_SIZE(widths) > PER_MAX_FIELDS) {
    PyErr_SetString(PyExc_ValueError, "bad handle or field table");
    return -1;
  }
  c->h = reinterpret_cast<per_t*>(h);
  c->T = T;
  c->n_fields = (uint32_t)PyTuple_GET_SIZE(widths);
  for (uint32_t f = 0; f < c->n_fields; ++f) {
    c->width[f] = PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(widths, f));
    if (PyErr_Occurred()) return -1;
  }
  c->device = (c10::DeviceIndex)device;
  return 0;
}

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_per_binding", "Calls of one replay buffer, tensors in, C-ABI calls out.", -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__per_binding() {
  calls_type.tp_name = "_per_binding.Calls";
  calls_type.tp_basicsize = sizeof(Calls);
  calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
  calls_type.tp_doc = "The per-iteration calls of one buffer (the buffer owns the handle).";
  calls_type.tp_methods = methods;
  calls_type.tp_init = init;
  calls_type.tp_new = PyType_GenericNew;
  if (PyType_Ready(&calls_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (!m) return nullptr;
  Py_INCREF(&calls_type);
  if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject*>(&calls_type)) < 0) return nullptr;
  return m;
}
