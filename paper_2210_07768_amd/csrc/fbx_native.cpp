// The part of the Python binding that runs once per call: handing the arguments to fbx_extract and the
// slot table of its result to Python.  A batch of a few records takes the GPU some tens of microseconds;
// marshalling through ctypes and one torch slice per array took longer than that (24 slots: 49 us a call,
// 164 slots: 120 us; here 5 and 15), which is why this is native.  Views share the caller's storage and
// are made when first asked for, without the dispatcher (a slice costs 1.7 us, a view made here 0.3).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "fbx.h"

namespace {

decltype(&fbx_extract) g_extract = nullptr;
decltype(&fbx_extract_static) g_extract_static = nullptr;
decltype(&fbx_last_error) g_last_error = nullptr;

// One emitted slot of a result: plain numbers, and where its arrays lie in the caller's buffer (in
// 64-bit words from the start of its storage; -1: there is no such array).
struct Slot {
  PyObject_HEAD
  PyObject* home;  // the buffer, a torch tensor
  unsigned int slot_id, fixed_arity;
  unsigned long long n_values;
  long long values_at, offsets_at, tile_ends_at, n_offsets, n_tiles;
  PyObject *values, *offsets, *tile_ends;  // views, once made
};

PyObject* view(PyObject* home, long long at, long long n) {
  const at::Tensor& t = THPVariable_Unpack(home);
  at::Tensor v = at::detail::make_tensor<at::TensorImpl>(c10::TensorImpl::VIEW, c10::Storage(t.storage()), t.key_set(),
                                                         caffe2::TypeMeta::Make<int64_t>());
  c10::TensorImpl* impl = v.unsafeGetTensorImpl();
  impl->set_storage_offset(at);
  impl->set_sizes_contiguous({n});
  impl->set_version_counter(t.unsafeGetTensorImpl()->version_counter());
  return THPVariable_Wrap(std::move(v));
}

PyObject* cached(PyObject*& slot, PyObject* home, long long at, long long n) {
  if (at < 0) Py_RETURN_NONE;
  if (!slot) {
    try {
      slot = view(home, at, n);
    } catch (const std::exception& e) {
      PyErr_SetString(PyExc_RuntimeError, e.what());
      return nullptr;
    }
    if (!slot) return nullptr;
  }
  Py_INCREF(slot);
  return slot;
}

PyObject* slot_values(PyObject* o, void*) {
  Slot* s = reinterpret_cast<Slot*>(o);
  return cached(s->values, s->home, s->values_at, static_cast<long long>(s->n_values));
}
PyObject* slot_offsets(PyObject* o, void*) {
  Slot* s = reinterpret_cast<Slot*>(o);
  return cached(s->offsets, s->home, s->offsets_at, s->n_offsets);
}
PyObject* slot_tile_ends(PyObject* o, void*) {
  Slot* s = reinterpret_cast<Slot*>(o);
  return cached(s->tile_ends, s->home, s->tile_ends_at, s->n_tiles);
}
PyObject* slot_id(PyObject* o, void*) { return PyLong_FromUnsignedLong(reinterpret_cast<Slot*>(o)->slot_id); }
PyObject* slot_arity(PyObject* o, void*) { return PyLong_FromUnsignedLong(reinterpret_cast<Slot*>(o)->fixed_arity); }
PyObject* slot_n(PyObject* o, void*) { return PyLong_FromUnsignedLongLong(reinterpret_cast<Slot*>(o)->n_values); }

void slot_dealloc(PyObject* o) {
  Slot* s = reinterpret_cast<Slot*>(o);
  Py_XDECREF(s->home);
  Py_XDECREF(s->values);
  Py_XDECREF(s->offsets);
  Py_XDECREF(s->tile_ends);
  Py_TYPE(o)->tp_free(o);
}

PyGetSetDef slot_getset[] = {
    {"slot_id", slot_id, nullptr, "slot number given in the spec", nullptr},
    {"fixed_arity", slot_arity, nullptr, "signs per record, 0 for a ragged slot", nullptr},
    {"n_values", slot_n, nullptr, "signs in this slot", nullptr},
    {"values", slot_values, nullptr, "the signs, an int64 view of the caller's buffer", nullptr},
    {"offsets", slot_offsets, nullptr, "None for a slot of fixed arity (offsets are implicit)", nullptr},
    {"tile_ends", slot_tile_ends, nullptr,
     "Arrival order only (ExtractResult.arrival_tile_records != 0, ragged slot): where each tile's share ends.", nullptr},
    {nullptr, nullptr, nullptr, nullptr, nullptr}};

PyTypeObject SlotType = {PyVarObject_HEAD_INIT(nullptr, 0)};

const char kStrided[] = "the buffer must be contiguous";

// slots(table, home, base, n_offsets, n_tiles) -> (dict of slot id -> Slot, list of slot ids).  table: the library's
// slot table as bytes; home: the tensor whose first byte lies at address base.
PyObject* slots(PyObject*, PyObject* args) {
  const char* table;
  Py_ssize_t bytes;
  PyObject* home;
  unsigned long long base;
  long long n_offsets, n_tiles;
  if (!PyArg_ParseTuple(args, "y#OKLL", &table, &bytes, &home, &base, &n_offsets, &n_tiles)) return nullptr;
  if (!THPVariable_Check(home)) {
    PyErr_SetString(PyExc_TypeError, "the buffer must be a torch tensor");
    return nullptr;
  }
  const at::Tensor& t = THPVariable_Unpack(home);
  if (!t.is_contiguous()) {  // (a view made from places in the storage would show what lies between its elements)
    PyErr_SetString(PyExc_RuntimeError, kStrided);
    return nullptr;
  }
  const unsigned long long size = t.numel() * t.element_size() / 8 * 8;
  const long long first_byte = t.storage_offset() * static_cast<long long>(t.element_size());
  if (first_byte % 8 != 0) {
    PyErr_SetString(PyExc_RuntimeError, "the buffer must start at a multiple of 8 bytes of its storage");
    return nullptr;
  }
  // where an array of the table lies, in words of the storage; -1 when it is not there or lies outside the buffer
  // (the table of tile ends of the entry point that allocates nothing lies in the library's own memory)
  auto word = [&](const void* p) -> long long {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    if (!p || a < base || a >= base + size) return -1;
    return (first_byte + static_cast<long long>(a - base)) / 8;
  };
  PyObject *dict = PyDict_New(), *list = PyList_New(bytes / static_cast<Py_ssize_t>(sizeof(fbx_slot_view)));
  if (!dict || !list) {
    Py_XDECREF(dict);
    Py_XDECREF(list);
    return nullptr;
  }
  const Py_ssize_t n = PyList_GET_SIZE(list);
  for (Py_ssize_t i = 0; i < n; ++i) {
    fbx_slot_view v;
    memcpy(&v, table + i * sizeof v, sizeof v);
    Slot* s = reinterpret_cast<Slot*>(SlotType.tp_alloc(&SlotType, 0));
    PyObject* key = PyLong_FromUnsignedLong(v.slot_id);
    if (!s || !key) {
      Py_XDECREF(reinterpret_cast<PyObject*>(s));
      Py_XDECREF(key);
      Py_DECREF(dict);
      Py_DECREF(list);
      return nullptr;
    }
    Py_INCREF(home);
    s->home = home;
    s->slot_id = v.slot_id;
    s->fixed_arity = v.fixed_arity;
    s->n_values = v.n_values;
    s->values_at = word(v.values);
    if (s->values_at < 0) s->values_at = first_byte / 8;  // (an array of nothing)
    s->offsets_at = word(v.offsets);
    s->tile_ends_at = word(v.tile_ends);
    s->n_offsets = n_offsets;
    s->n_tiles = n_tiles;
    const int bad = PyDict_SetItem(dict, key, reinterpret_cast<PyObject*>(s));
    Py_DECREF(reinterpret_cast<PyObject*>(s));
    PyList_SET_ITEM(list, i, key);
    if (bad) {
      Py_DECREF(dict);
      Py_DECREF(list);
      return nullptr;
    }
  }
  return Py_BuildValue("(NN)", dict, list);
}

// Elements and address (0 for none of them) of a tensor, or of anything else that has numel() and data_ptr().
bool array(PyObject* o, uint64_t& n, uint64_t& address) {
  if (THPVariable_Check(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    n = t.numel();
    address = n ? reinterpret_cast<uint64_t>(t.data_ptr()) : 0;
    return true;
  }
  auto ask = [&](const char* method, uint64_t& v) -> bool {
    PyObject* r = PyObject_CallMethod(o, method, nullptr);
    if (!r) return false;
    v = PyLong_AsUnsignedLongLong(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
  };
  address = 0;
  return ask("numel", n) && (!n || ask("data_ptr", address));
}

// extract(plan, raw, rec_off, stream, out_buffer or None) -> (status, records, signs, malformed numerics, high water,
// layers, tile launches, records of a tile in arrival order, note, slot table as bytes)
PyObject* extract(PyObject*, PyObject* args) {
  unsigned long long plan, stream;
  PyObject *raw, *off, *buffer;
  if (!PyArg_ParseTuple(args, "KOOKO", &plan, &raw, &off, &stream, &buffer)) return nullptr;
  if (buffer != Py_None && !THPVariable_Check(buffer)) {
    PyErr_SetString(PyExc_TypeError, "the output buffer must be a torch tensor");
    return nullptr;
  }
  fbx_plan* p = reinterpret_cast<fbx_plan*>(plan);
  fbx_result r{};
  fbx_status st;
  const char* error = nullptr;
  try {
    if (buffer != Py_None && !THPVariable_Unpack(buffer).is_contiguous()) {
      PyErr_SetString(PyExc_RuntimeError, kStrided);
      return nullptr;
    }
    uint64_t raw_len, n_offsets, raw_at, off_at;
    if (!array(raw, raw_len, raw_at) || !array(off, n_offsets, off_at)) return nullptr;
    const uint64_t n_records = n_offsets - 1;
    const uint8_t* text = reinterpret_cast<const uint8_t*>(raw_at);
    const uint64_t* offsets = reinterpret_cast<const uint64_t*>(off_at);
    void* out = buffer == Py_None ? nullptr : THPVariable_Unpack(buffer).data_ptr();
    const uint64_t out_bytes = buffer == Py_None ? 0 : THPVariable_Unpack(buffer).numel();
    Py_BEGIN_ALLOW_THREADS
    st = buffer == Py_None ? g_extract(p, text, raw_len, offsets, n_records, reinterpret_cast<void*>(stream), &r)
                           : g_extract_static(p, text, raw_len, offsets, n_records, out, out_bytes, reinterpret_cast<void*>(stream), &r);
    error = g_last_error(p);
    Py_END_ALLOW_THREADS
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
  return Py_BuildValue("(iKKKKIIIsy#)", static_cast<int>(st), r.n_records, r.n_values_total, r.n_malformed_numeric, r.arena_high_water,
                       r.n_layers, r.tile_launches, r.arrival_tile_records, error ? error : "",
                       st == FBX_OK && r.n_slots ? reinterpret_cast<const char*>(r.slots) : "",
                       st == FBX_OK ? static_cast<Py_ssize_t>(r.n_slots * sizeof(fbx_slot_view)) : static_cast<Py_ssize_t>(0));
}

// bind(address of fbx_extract, of fbx_extract_static, of fbx_last_error): the library itself is loaded by the binding
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long a, b, c;
  if (!PyArg_ParseTuple(args, "KKK", &a, &b, &c)) return nullptr;
  g_extract = reinterpret_cast<decltype(g_extract)>(a);
  g_extract_static = reinterpret_cast<decltype(g_extract_static)>(b);
  g_last_error = reinterpret_cast<decltype(g_last_error)>(c);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"extract", extract, METH_VARARGS, nullptr},
                         {"slots", slots, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  SlotType.tp_name = "paper_2210_07768_amd._native.Slot";
  SlotType.tp_basicsize = sizeof(Slot);
  SlotType.tp_dealloc = slot_dealloc;
  SlotType.tp_flags = Py_TPFLAGS_DEFAULT;
  SlotType.tp_getset = slot_getset;
  SlotType.tp_doc = "One emitted slot of a result; values and offsets are views of the caller's buffer, made when first asked for.";
  if (PyType_Ready(&SlotType) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (!m) return nullptr;
  Py_INCREF(&SlotType);
  PyModule_AddObject(m, "Slot", reinterpret_cast<PyObject*>(&SlotType));
  return m;
}
