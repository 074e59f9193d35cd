// CPython module _launcher: the host path of a step.
//
// A step is a handful of C-ABI calls with ~20 arguments each.  Marshalling them through ctypes and
// re-checking the tensors of every call costs 5 us per launch for prepared calls and 10-25 us
// otherwise, against 3.6 us with the launch itself from here: a step of three launches was bound by the host
// (42 us for 19 us of kernels at 2 x 196 tokens).  Here the arguments of a call are kept as raw
// 8-byte values (Call), and a whole step as a list of them (Program) in which the caller's tensors, the
// pass's own buffers and the current stream are open places that every run fills in: per run, one check of
// dtype, shape, contiguity and device per tensor, one comparison per other attribute of the pass, then the
// launches, with the interpreter lock released.  Tensors are read through torch's C++ interface (a few ns
// each; five attribute reads through Python objects were 0.3 us).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <utility>
#include <vector>

#include "spa.h"

namespace {

// ---- the C entry points by name: argument kinds and a trampoline from raw values ------------
union Value {
  void* p;
  int i;
  int64_t l;
  size_t z;
  float f;
  uint64_t raw;
};

template <class A> struct Kind { static constexpr char c = 'p'; static A get(const Value& v) { return (A)v.p; } };
template <> struct Kind<int> { static constexpr char c = 'i'; static int get(const Value& v) { return v.i; } };
template <> struct Kind<int64_t> { static constexpr char c = 'l'; static int64_t get(const Value& v) { return v.l; } };
template <> struct Kind<size_t> { static constexpr char c = 'z'; static size_t get(const Value& v) { return v.z; } };
template <> struct Kind<float> { static constexpr char c = 'f'; static float get(const Value& v) { return v.f; } };

constexpr int kMaxArgs = 32;

template <class F> struct Signature;
template <class... A> struct Signature<int (*)(A...)> {
  static_assert(sizeof...(A) <= kMaxArgs, "raise kMaxArgs");
  static constexpr char kinds[] = {Kind<A>::c..., 0};
  template <size_t... I> static int apply(int (*fn)(A...), const Value* v, std::index_sequence<I...>) {
    return fn(Kind<A>::get(v[I])...);
  }
  static int call(void* fn, const Value* v) {
    return apply(reinterpret_cast<int (*)(A...)>(fn), v, std::index_sequence_for<A...>{});
  }
};

struct Entry {
  const char* name;
  const char* kinds;
  int (*call)(void*, const Value*);
};
#define ENTRY(fn) {#fn, Signature<decltype(&fn)>::kinds, &Signature<decltype(&fn)>::call}
const Entry kEntries[] = {
    ENTRY(spa_group_begin), ENTRY(spa_group_end),
    ENTRY(spa_gate_select), ENTRY(spa_gate_select_index), ENTRY(spa_gate_select_pooled), ENTRY(spa_gate_select_gumbel),
    ENTRY(spa_gate_bwd_straight_through), ENTRY(spa_maxpool2x2), ENTRY(spa_pack), ENTRY(spa_pack_pair),
    ENTRY(spa_pack_shifted), ENTRY(spa_container_segments), ENTRY(spa_packed_attention), ENTRY(spa_packed_attention_running_max),
    ENTRY(spa_packed_attention_unpack), ENTRY(spa_gathered_attention_unpack), ENTRY(spa_selected_attention_unpack),
    ENTRY(spa_gated_attention_unpack), ENTRY(spa_gated_attention_bwd_tokens),
    ENTRY(spa_gated_attention_unpack_dvec), ENTRY(spa_gated_attention_bwd_tokens_dvec), ENTRY(spa_segment_attention_unpack),
    ENTRY(spa_pack_containers), ENTRY(spa_packed_attention_bwd_spread), ENTRY(spa_gated_attention_bwd_tokens_spread),
    ENTRY(spa_gathered_segment_attention_unpack), ENTRY(spa_ceiling_copy), ENTRY(spa_linear_packed),
    ENTRY(spa_linear_packed_scatter), ENTRY(spa_linear_packed_unpack), ENTRY(spa_linear_packed_bwd_input), ENTRY(spa_linear_packed_bwd_weight),
    ENTRY(spa_unpack), ENTRY(spa_unpack_bwd), ENTRY(spa_pack_bwd), ENTRY(spa_packed_attention_bwd),
    ENTRY(spa_packed_attention_bwd_tokens), ENTRY(spa_gate_bwd), ENTRY(spa_gate_bwd_static), ENTRY(spa_padded_attention),
};

PyObject* g_on_error = nullptr;      // called with the return code of a failing C call; raises
PyObject* g_device = nullptr;        // () -> current device index
PyObject* g_raw_stream = nullptr;    // (device index) -> current stream of the device

constexpr int kNoSlot = -2, kStreamSlot = -1;

// One step of a program.
struct Op {
  enum What : uint8_t { kCall, kRecord, kWait } what = kCall;
  const Entry* entry = nullptr;
  void* fn = nullptr;
  hipEvent_t event = nullptr;
  int nargs = 0;
  bool open = false;                  // some argument is filled in per run
  Value args[kMaxArgs];
  int16_t slot[kMaxArgs];             // kNoSlot | kStreamSlot | index of an open place (args[] then holds the byte offset)
};

// base[i]: address (or value) of open place i; stream: what kStreamSlot stands for
int issue(const Op& op, const Value* base, void* stream) {
  Value local[kMaxArgs];
  const Value* v = op.args;
  if (op.open) {
    for (int i = 0; i < op.nargs; ++i) {
      local[i] = op.args[i];
      if (op.slot[i] == kStreamSlot) local[i].p = stream;
      else if (op.slot[i] >= 0) local[i].l = base[op.slot[i]].l + op.args[i].l;
    }
    v = local;
  }
  if (op.what == Op::kCall) return op.entry->call(op.fn, v);
  const hipStream_t s = (hipStream_t)v[0].p;
  const hipError_t e = op.what == Op::kRecord ? hipEventRecord(op.event, s) : hipStreamWaitEvent(s, op.event, 0);
  return e == hipSuccess ? SPA_OK : SPA_ERR_HIP;
}

PyObject* raise_code(int rc) {
  if (g_on_error != nullptr) {
    PyObject* r = PyObject_CallFunction(g_on_error, "i", rc);
    Py_XDECREF(r);
  }
  if (!PyErr_Occurred()) PyErr_Format(PyExc_RuntimeError, "libspa error %d", rc);
  return nullptr;
}

// An argument as the binding hands it over: None, a number, or (index, byte offset) for a place
// that is filled in per run ((-1, 0) = the current stream; a number of the pass: (index, 0))
bool parse_arg(PyObject* o, char kind, Op& op, int i) {
  op.args[i].raw = 0;
  op.slot[i] = kNoSlot;
  if (o == Py_None) return true;
  if (PyTuple_Check(o)) {
    const long idx = PyLong_AsLong(PyTuple_GET_ITEM(o, 0));
    op.args[i].l = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 1));
    op.slot[i] = (int16_t)idx;
    op.open = true;
  } else if (kind == 'f') {
    op.args[i].f = (float)PyFloat_AsDouble(o);
  } else if (kind == 'i') {
    const long n = PyLong_AsLong(o);
    if (n > 2147483647L || n < -2147483648L) PyErr_SetString(PyExc_OverflowError, "argument does not fit an int");
    op.args[i].i = (int)n;
  } else if (kind == 'l') {
    op.args[i].l = PyLong_AsLongLong(o);
  } else {
    op.args[i].z = PyLong_AsSize_t(o);
  }
  return !PyErr_Occurred();
}

// ---- Event ---------------------------------------------------------------------------------
struct EventObject {
  PyObject_HEAD
  hipEvent_t event;
};

PyObject* event_new(PyTypeObject* type, PyObject*, PyObject*) {
  hipEvent_t ev;
  if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
    PyErr_SetString(PyExc_RuntimeError, "hipEventCreate failed");
    return nullptr;
  }
  EventObject* self = (EventObject*)type->tp_alloc(type, 0);
  if (self != nullptr) self->event = ev;
  return (PyObject*)self;
}

void event_dealloc(PyObject* o) {
  (void)hipEventDestroy(((EventObject*)o)->event);
  Py_TYPE(o)->tp_free(o);
}

PyTypeObject EventType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---- Call: one C-ABI call (or event operation) with its arguments ---------------------------
struct CallObject {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  Op* op;
  PyObject* keep;      // the tensors (streams, events) the arguments point into
};

extern PyTypeObject CallType;

PyObject* call_vectorcall(PyObject* o, PyObject* const*, size_t nargsf, PyObject* kwnames) {
  CallObject* self = (CallObject*)o;
  if (PyVectorcall_NARGS(nargsf) != 0 || (kwnames != nullptr && PyTuple_GET_SIZE(kwnames) != 0)) {
    PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
    return nullptr;
  }
  if (self->op->open) {
    PyErr_SetString(PyExc_RuntimeError, "a recorded call runs inside its program only");
    return nullptr;
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = issue(*self->op, nullptr, nullptr);
  Py_END_ALLOW_THREADS
  if (rc != SPA_OK) return raise_code(rc);
  Py_RETURN_NONE;
}

// Call(name, address, args, keep)
PyObject* call_new(PyTypeObject* type, PyObject* a, PyObject*) {
  const char* name;
  unsigned long long addr;
  PyObject *args, *keep;
  if (!PyArg_ParseTuple(a, "sKO!O", &name, &addr, &PyTuple_Type, &args, &keep)) return nullptr;
  const Entry* entry = nullptr;
  for (const Entry& e : kEntries)
    if (!std::strcmp(e.name, name)) entry = &e;
  if (entry == nullptr || (Py_ssize_t)std::strlen(entry->kinds) != PyTuple_GET_SIZE(args)) {
    PyErr_Format(PyExc_TypeError, "%s: unknown entry point or wrong number of arguments", name);
    return nullptr;
  }
  CallObject* self = (CallObject*)type->tp_alloc(type, 0);
  if (self == nullptr) return nullptr;
  self->vectorcall = call_vectorcall;
  self->op = new Op;
  self->op->entry = entry;
  self->op->fn = (void*)(uintptr_t)addr;
  self->op->nargs = (int)PyTuple_GET_SIZE(args);
  Py_INCREF(keep);
  self->keep = keep;
  for (int i = 0; i < self->op->nargs; ++i)
    if (!parse_arg(PyTuple_GET_ITEM(args, i), entry->kinds[i], *self->op, i)) {
      Py_DECREF(self);
      return nullptr;
    }
  return (PyObject*)self;
}

void call_dealloc(PyObject* o) {
  CallObject* self = (CallObject*)o;
  delete self->op;
  Py_XDECREF(self->keep);
  Py_TYPE(o)->tp_free(o);
}

PyTypeObject CallType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// event_op(event, stream, is_wait, keep) -> Call: record the event on the stream / let the stream wait for it
PyObject* event_op(PyObject*, PyObject* a) {
  PyObject *ev, *stream, *keep;
  int wait;
  if (!PyArg_ParseTuple(a, "O!OpO", &EventType, &ev, &stream, &wait, &keep)) return nullptr;
  CallObject* self = (CallObject*)CallType.tp_alloc(&CallType, 0);
  if (self == nullptr) return nullptr;
  self->vectorcall = call_vectorcall;
  self->op = new Op;
  self->op->what = wait ? Op::kWait : Op::kRecord;
  self->op->event = ((EventObject*)ev)->event;
  self->op->nargs = 1;
  self->keep = PyTuple_Pack(2, ev, keep);
  if (self->keep == nullptr || !parse_arg(stream, 'p', *self->op, 0)) {
    Py_DECREF(self);
    return nullptr;
  }
  return (PyObject*)self;
}

// ---- Program: a step --------------------------------------------------------------------------
// What a tensor has to be for the recorded launches to hold for it.
struct TensorSpec {
  bool absent = false;          // None
  at::ScalarType dtype = at::kFloat;
  std::vector<int64_t> shape;
};

// What a step depends on beside its inputs: the attributes of its owner (object 0) and of the passes inside it
// (object k, found from object `of`, which comes before it).  `index` >= 0: element of the list `name` holds.
struct Place {
  enum What : uint8_t {
    kObject,      // the next object: of exactly the type `value`
    kTensor,      // an open place: the next slot
    kNumber,      // likewise, a float argument of the calls
    kConstant,    // equal to `value`
    kLength       // a list or tuple of `index` elements
  } what = kConstant;
  int of = 0;
  PyObject* name = nullptr;
  Py_ssize_t index = -1;
  PyObject* value = nullptr;
  TensorSpec tensor;
};

struct ProgramObject {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  std::vector<const Op*>* ops;
  std::vector<TensorSpec>* inputs;
  std::vector<Place>* places;
  PyObject* keep;               // the Call objects
  long runs;                    // steps issued
  size_t slots, objects;
  bool owned;                   // called with the owner of the places in front of the inputs
  bool open;                    // some op names the current stream or a tensor
  bool part;                    // of a step being recorded: its calls name tensors of the program it goes into
};
constexpr size_t kMaxSlots = 512, kMaxObjects = 16;

PyTypeObject ProgramType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// true: as recorded, address in *out.  Exactly torch's own tensor types: what a subclass makes of its
// attributes is not read here (such a step goes call by call).
bool match(const TensorSpec& spec, PyObject* o, Value* out) {
  out->raw = 0;
  if (spec.absent) return o == Py_None;
  if (!THPVariable_CheckExact(o)) return false;
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != spec.dtype || t.sizes() != at::IntArrayRef(spec.shape) || !t.is_contiguous()) return false;
    out->p = t.data_ptr();
    return true;
  } catch (...) {               // a tensor without memory of its own: the call-by-call path says so
    return false;
  }
}

// The attribute (or list element) a place names, borrowed; nullptr when it is not there.
PyObject* look_up(const Place& p, PyObject* const* dicts) {
  PyObject* v = PyDict_GetItemWithError(dicts[p.of], p.name);
  if (v == nullptr || p.index < 0 || p.what == Place::kLength) return v;
  if (PyList_CheckExact(v)) return p.index < PyList_GET_SIZE(v) ? PyList_GET_ITEM(v, p.index) : nullptr;
  if (PyTuple_CheckExact(v)) return p.index < PyTuple_GET_SIZE(v) ? PyTuple_GET_ITEM(v, p.index) : nullptr;
  return nullptr;
}

// Tensors of the owner's state, held while the launches go out: a program's other threads may replace them.
struct Held {
  PyObject* t[kMaxSlots];
  size_t n = 0;
  void add(PyObject* o) {
    Py_INCREF(o);
    t[n++] = o;
  }
  ~Held() {
    while (n > 0) Py_DECREF(t[--n]);
  }
};

// The owner's state against the recording; fills the slots from `slot` on, whose tensors `held` then holds.
bool match_places(const ProgramObject* self, PyObject* owner, Value* base, size_t slot, Held& held) {
  PyObject* dicts[kMaxObjects];
  size_t n = 0;
  auto enter = [&](PyObject* o) {                    // (the object keeps its dict alive, its holder the object)
    PyObject* d = PyObject_GenericGetDict(o, nullptr);
    if (d == nullptr) return false;
    dicts[n++] = d;
    Py_DECREF(d);
    return true;
  };
  if (!enter(owner)) return false;
  for (const Place& p : *self->places) {
    PyObject* v = look_up(p, dicts);
    if (v == nullptr) return false;
    switch (p.what) {
      case Place::kObject:
        if ((PyObject*)Py_TYPE(v) != p.value || !enter(v)) return false;
        break;
      case Place::kTensor:
        if (!match(p.tensor, v, &base[slot++])) return false;
        held.add(v);
        break;
      case Place::kNumber: {
        if (!PyFloat_CheckExact(v) && !PyLong_CheckExact(v)) return false;
        const double d = PyFloat_AsDouble(v);
        if (d == -1.0 && PyErr_Occurred()) return false;
        base[slot].raw = 0;
        base[slot++].f = (float)d;
        break;
      }
      case Place::kConstant:
        if (v != p.value) {
          Py_INCREF(v);
          const int eq = PyObject_RichCompareBool(v, p.value, Py_EQ);
          Py_DECREF(v);
          if (eq != 1) return false;
        }
        break;
      case Place::kLength:
        if (!(PyList_CheckExact(v) && PyList_GET_SIZE(v) == p.index) && !(PyTuple_CheckExact(v) && PyTuple_GET_SIZE(v) == p.index))
          return false;
        break;
    }
  }
  return true;
}

void* current_stream() {
  PyObject* dev = PyObject_CallNoArgs(g_device);
  if (dev == nullptr) return nullptr;
  PyObject* s = PyObject_CallOneArg(g_raw_stream, dev);
  Py_DECREF(dev);
  if (s == nullptr) return nullptr;
  void* p = (void*)(uintptr_t)PyLong_AsUnsignedLongLong(s);
  Py_DECREF(s);
  return p;
}

// program([owner,] *inputs) -> True when the step was issued, False when the inputs or the owner's attributes are
// not those it was recorded for
PyObject* program_vectorcall(PyObject* o, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  ProgramObject* self = (ProgramObject*)o;
  const size_t n = (size_t)PyVectorcall_NARGS(nargsf), first = self->owned ? 1 : 0;
  if (kwnames != nullptr && PyTuple_GET_SIZE(kwnames) != 0) {
    PyErr_SetString(PyExc_TypeError, "a program takes positional inputs");
    return nullptr;
  }
  if (self->part) {
    PyErr_SetString(PyExc_RuntimeError, "a part of a recorded step runs inside its program only");
    return nullptr;
  }
  if (n != self->inputs->size() + first) Py_RETURN_FALSE;
  Value base[kMaxSlots];
  for (size_t i = first; i < n; ++i)
    if (!match((*self->inputs)[i - first], args[i], &base[i - first])) Py_RETURN_FALSE;
  Held held;
  if (self->owned && !match_places(self, args[0], base, n - first, held)) {
    PyErr_Clear();              // an attribute that cannot be compared is one that is not as recorded
    Py_RETURN_FALSE;
  }
  void* stream = nullptr;
  if (self->open) {
    stream = current_stream();
    if (PyErr_Occurred()) return nullptr;
  }
  int rc = SPA_OK;
  Py_BEGIN_ALLOW_THREADS
  for (const Op* op : *self->ops) {
    rc = issue(*op, base, stream);
    if (rc != SPA_OK) break;
  }
  Py_END_ALLOW_THREADS
  ++self->runs;
  if (rc != SPA_OK) return raise_code(rc);
  Py_RETURN_TRUE;
}

// None | an example of the tensor (dtype and shape are taken from it)
bool parse_tensor(PyObject* o, TensorSpec* out) {
  if (o == Py_None) {
    out->absent = true;
    return true;
  }
  if (!THPVariable_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "an input is described by None or a tensor");
    return false;
  }
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    out->dtype = t.scalar_type();
    out->shape = t.sizes().vec();
    return true;
  } catch (...) {
    PyErr_SetString(PyExc_TypeError, "an input needs a dtype and a shape");
    return false;
  }
}

// (what, object, name, index, value)
bool parse_place(PyObject* o, Place* out, size_t objects) {
  const char* what;
  if (!PyTuple_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "a place is a tuple");
    return false;
  }
  if (!PyArg_ParseTuple(o, "siUnO", &what, &out->of, &out->name, &out->index, &out->value)) {
    out->name = out->value = nullptr;
    return false;
  }
  Py_INCREF(out->name);
  Py_INCREF(out->value);
  out->what = what[0] == 'o' ? Place::kObject : what[0] == 't' ? Place::kTensor : what[0] == 'n' ? Place::kNumber : what[0] == 'l' ? Place::kLength : Place::kConstant;
  if (out->of < 0 || (size_t)out->of >= objects) {
    PyErr_SetString(PyExc_ValueError, "a place names an object that comes after it");
    return false;
  }
  return out->what != Place::kTensor || parse_tensor(out->value, &out->tensor);
}

// Program(calls, inputs, places = None): calls = Calls and input-less Programs; inputs = None or an example tensor per
// input; places = what the step reads of its owner (None: it has none)
PyObject* program_new(PyTypeObject* type, PyObject* a, PyObject*) {
  PyObject *calls, *inputs, *places = Py_None;
  if (!PyArg_ParseTuple(a, "O!O!|O", &PyTuple_Type, &calls, &PyTuple_Type, &inputs, &places)) return nullptr;
  if (places != Py_None && !PyTuple_CheckExact(places)) {
    PyErr_SetString(PyExc_TypeError, "places are a tuple");
    return nullptr;
  }
  ProgramObject* self = (ProgramObject*)type->tp_alloc(type, 0);
  if (self == nullptr) return nullptr;
  self->vectorcall = program_vectorcall;
  self->ops = new std::vector<const Op*>;
  self->inputs = new std::vector<TensorSpec>;
  self->places = new std::vector<Place>;
  Py_INCREF(calls);
  self->keep = calls;
  auto fail = [&]() -> PyObject* {
    Py_DECREF(self);
    return nullptr;
  };
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(calls); ++i) {
    PyObject* c = PyTuple_GET_ITEM(calls, i);
    if (Py_TYPE(c) == &CallType) {
      self->ops->push_back(((CallObject*)c)->op);
    } else if (Py_TYPE(c) == &ProgramType && ((ProgramObject*)c)->inputs->empty() && !((ProgramObject*)c)->owned) {
      for (const Op* op : *((ProgramObject*)c)->ops) self->ops->push_back(op);
    } else {
      PyErr_SetString(PyExc_TypeError, "a program is made of calls");
      return fail();
    }
  }
  for (const Op* op : *self->ops) self->open = self->open || op->open;
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(inputs); ++i) {
    self->inputs->emplace_back();
    if (!parse_tensor(PyTuple_GET_ITEM(inputs, i), &self->inputs->back())) return fail();
  }
  self->slots = self->inputs->size();
  self->objects = 1;
  if (places != Py_None) {
    self->owned = true;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(places); ++i) {
      self->places->emplace_back();
      if (!parse_place(PyTuple_GET_ITEM(places, i), &self->places->back(), self->objects)) return fail();
      self->slots += self->places->back().what == Place::kTensor || self->places->back().what == Place::kNumber;
      self->objects += self->places->back().what == Place::kObject;
    }
  }
  if (self->slots > kMaxSlots || self->objects > kMaxObjects) {
    PyErr_SetString(PyExc_ValueError, "too many tensors or passes in a program");
    return fail();
  }
  for (const Op* op : *self->ops)
    for (int i = 0; i < op->nargs; ++i) self->part = self->part || op->slot[i] >= (int)self->slots;
  if (self->part && self->slots > 0) {
    PyErr_SetString(PyExc_ValueError, "a call names a tensor the program does not have");
    return fail();
  }
  return (PyObject*)self;
}

void program_dealloc(PyObject* o) {
  ProgramObject* self = (ProgramObject*)o;
  for (Place& p : *self->places) {
    Py_XDECREF(p.name);
    Py_XDECREF(p.value);
  }
  delete self->places;
  delete self->inputs;
  delete self->ops;
  Py_XDECREF(self->keep);
  Py_TYPE(o)->tp_free(o);
}

PyMemberDef kProgramMembers[] = {{"runs", T_LONG, offsetof(ProgramObject, runs), READONLY, "steps issued"}, {nullptr, 0, 0, 0, nullptr}};

// setup(on_error, current_device, raw_stream)
PyObject* setup(PyObject*, PyObject* a) {
  PyObject *e, *d, *s;
  if (!PyArg_ParseTuple(a, "OOO", &e, &d, &s)) return nullptr;
  Py_INCREF(e);
  Py_INCREF(d);
  Py_INCREF(s);
  g_on_error = e;
  g_device = d;
  g_raw_stream = s;
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {{"event_op", event_op, METH_VARARGS, nullptr}, {"setup", setup, METH_VARARGS, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_launcher", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

bool ready(PyTypeObject& t, const char* name, size_t size, newfunc make, destructor del, Py_ssize_t vectorcall_offset) {
  t.tp_name = name;
  t.tp_basicsize = (Py_ssize_t)size;
  t.tp_flags = Py_TPFLAGS_DEFAULT;
  t.tp_new = make;
  t.tp_dealloc = del;
  if (vectorcall_offset != 0) {
    t.tp_flags |= Py_TPFLAGS_HAVE_VECTORCALL;
    t.tp_vectorcall_offset = vectorcall_offset;
    t.tp_call = PyVectorcall_Call;
  }
  return PyType_Ready(&t) == 0;
}

}  // namespace

PyMODINIT_FUNC PyInit__launcher(void) {
  ProgramType.tp_members = kProgramMembers;
  if (!ready(EventType, "_launcher.Event", sizeof(EventObject), event_new, event_dealloc, 0) ||
      !ready(CallType, "_launcher.Call", sizeof(CallObject), call_new, call_dealloc, offsetof(CallObject, vectorcall)) ||
      !ready(ProgramType, "_launcher.Program", sizeof(ProgramObject), program_new, program_dealloc,
             offsetof(ProgramObject, vectorcall)))
    return nullptr;
  PyObject* m = PyModule_Create(&kModule);
  if (m == nullptr) return nullptr;
  for (PyTypeObject* t : {&EventType, &CallType, &ProgramType}) Py_INCREF(t);
  PyModule_AddObject(m, "Event", (PyObject*)&EventType);
  PyModule_AddObject(m, "Call", (PyObject*)&CallType);
  PyModule_AddObject(m, "Program", (PyObject*)&ProgramType);
  return m;
}
