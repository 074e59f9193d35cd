// CPython module _launcher: the host path of a step.
//
// A step is a handful of C-ABI calls with ~20 arguments each.  Marshalling them through ctypes and
// re-checking the tensors of every call costs 5 us per launch for prepared calls and 10-25 us
// otherwise, against 2.9 us for the launch itself: a step of three launches was bound by the host
// (42 us for 19 us of kernels at 2 x 196 tokens).  Here the arguments of a call are kept as raw
// 8-byte values (Call), and a whole step as a list of them (Program) in which the caller's tensors
// and the current stream are open places that every run fills in: per run, one check of dtype,
// shape, contiguity and device per input, then the launches, with the interpreter lock released.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <hip/hip_runtime_api.h>

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
    ENTRY(spa_gated_attention_unpack), ENTRY(spa_gated_attention_bwd_tokens), ENTRY(spa_segment_attention_unpack),
    ENTRY(spa_pack_containers), ENTRY(spa_packed_attention_bwd_spread), ENTRY(spa_gated_attention_bwd_tokens_spread),
    ENTRY(spa_gathered_segment_attention_unpack), ENTRY(spa_ceiling_copy), ENTRY(spa_linear_packed),
    ENTRY(spa_linear_packed_scatter), ENTRY(spa_linear_packed_unpack), ENTRY(spa_linear_packed_bwd_input), ENTRY(spa_linear_packed_bwd_weight),
    ENTRY(spa_unpack), ENTRY(spa_unpack_bwd), ENTRY(spa_pack_bwd), ENTRY(spa_packed_attention_bwd),
    ENTRY(spa_packed_attention_bwd_tokens), ENTRY(spa_gate_bwd), ENTRY(spa_gate_bwd_static), ENTRY(spa_padded_attention),
};

PyObject* g_on_error = nullptr;      // called with the return code of a failing C call; raises
PyObject* g_device = nullptr;        // () -> current device index
PyObject* g_raw_stream = nullptr;    // (device index) -> current stream of the device
PyObject *s_dtype, *s_shape, *s_is_contiguous, *s_is_cuda, *s_data_ptr;

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
  int8_t slot[kMaxArgs];              // kNoSlot | kStreamSlot | index of an input (args[] then holds the byte offset)
};

// base[i]: address of input i; stream: what kStreamSlot stands for
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

// An argument as the binding hands it over: None, a number, or (input index, byte offset) for a place
// that is filled in per run ((-1, 0) = the current stream).
bool parse_arg(PyObject* o, char kind, Op& op, int i) {
  op.args[i].raw = 0;
  op.slot[i] = kNoSlot;
  if (o == Py_None) return true;
  if (PyTuple_Check(o)) {
    const long idx = PyLong_AsLong(PyTuple_GET_ITEM(o, 0));
    op.args[i].l = PyLong_AsLongLong(PyTuple_GET_ITEM(o, 1));
    op.slot[i] = (int8_t)idx;
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
struct Input {
  PyObject* dtype = nullptr;    // nullptr: the input is absent (None)
  PyObject* shape = nullptr;
};

struct ProgramObject {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  std::vector<const Op*>* ops;
  std::vector<Input>* inputs;
  PyObject* keep;               // the Call objects
  bool open;                    // some op names the current stream or an input
};

PyTypeObject ProgramType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// 1: as recorded, address in *out; 0: something else; -1: error
int match(const Input& in, PyObject* t, Value* out) {
  out->raw = 0;
  if (in.dtype == nullptr) return t == Py_None;
  if (t == Py_None) return 0;
  PyObject* o = PyObject_GetAttr(t, s_dtype);
  if (o == nullptr) return -1;
  bool ok = o == in.dtype;
  Py_DECREF(o);
  if (!ok) return 0;
  if ((o = PyObject_GetAttr(t, s_shape)) == nullptr) return -1;
  const int eq = PyObject_RichCompareBool(o, in.shape, Py_EQ);
  Py_DECREF(o);
  if (eq <= 0) return eq;
  if ((o = PyObject_GetAttr(t, s_is_cuda)) == nullptr) return -1;
  ok = o == Py_True;
  Py_DECREF(o);
  if (!ok) return 0;
  if ((o = PyObject_CallMethodNoArgs(t, s_is_contiguous)) == nullptr) return -1;
  ok = o == Py_True;
  Py_DECREF(o);
  if (!ok) return 0;
  if ((o = PyObject_CallMethodNoArgs(t, s_data_ptr)) == nullptr) return -1;
  out->z = PyLong_AsSize_t(o);
  Py_DECREF(o);
  return PyErr_Occurred() ? -1 : 1;
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

// program(*inputs) -> True when the step was issued, False when the inputs are not those it was recorded for
PyObject* program_vectorcall(PyObject* o, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  ProgramObject* self = (ProgramObject*)o;
  const size_t n = (size_t)PyVectorcall_NARGS(nargsf);
  constexpr size_t kMaxInputs = 64;
  if (kwnames != nullptr && PyTuple_GET_SIZE(kwnames) != 0) {
    PyErr_SetString(PyExc_TypeError, "a program takes positional inputs");
    return nullptr;
  }
  if (n != self->inputs->size() || n > kMaxInputs) Py_RETURN_FALSE;
  Value base[kMaxInputs];
  for (size_t i = 0; i < n; ++i) {
    const int m = match((*self->inputs)[i], args[i], &base[i]);
    if (m < 0) return nullptr;
    if (m == 0) Py_RETURN_FALSE;
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
  if (rc != SPA_OK) return raise_code(rc);
  Py_RETURN_TRUE;
}

// Program(calls, inputs): calls = Calls and input-less Programs; inputs = (dtype, shape) or None per input
PyObject* program_new(PyTypeObject* type, PyObject* a, PyObject*) {
  PyObject *calls, *inputs;
  if (!PyArg_ParseTuple(a, "O!O!", &PyTuple_Type, &calls, &PyTuple_Type, &inputs)) return nullptr;
  ProgramObject* self = (ProgramObject*)type->tp_alloc(type, 0);
  if (self == nullptr) return nullptr;
  self->vectorcall = program_vectorcall;
  self->ops = new std::vector<const Op*>;
  self->inputs = new std::vector<Input>;
  Py_INCREF(calls);
  self->keep = calls;
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(calls); ++i) {
    PyObject* c = PyTuple_GET_ITEM(calls, i);
    if (Py_TYPE(c) == &CallType) {
      self->ops->push_back(((CallObject*)c)->op);
    } else if (Py_TYPE(c) == &ProgramType && ((ProgramObject*)c)->inputs->empty()) {
      for (const Op* op : *((ProgramObject*)c)->ops) self->ops->push_back(op);
    } else {
      PyErr_SetString(PyExc_TypeError, "a program is made of calls");
      Py_DECREF(self);
      return nullptr;
    }
  }
  for (const Op* op : *self->ops) self->open = self->open || op->open;
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(inputs); ++i) {
    PyObject* s = PyTuple_GET_ITEM(inputs, i);
    Input in;
    if (s != Py_None) {
      in.dtype = PyTuple_GetItem(s, 0);
      in.shape = in.dtype != nullptr ? PyTuple_GetItem(s, 1) : nullptr;
      if (in.shape == nullptr) {
        Py_DECREF(self);
        return nullptr;
      }
      Py_INCREF(in.dtype);
      Py_INCREF(in.shape);
    }
    self->inputs->push_back(in);
  }
  return (PyObject*)self;
}

void program_dealloc(PyObject* o) {
  ProgramObject* self = (ProgramObject*)o;
  for (Input& in : *self->inputs) {
    Py_XDECREF(in.dtype);
    Py_XDECREF(in.shape);
  }
  delete self->inputs;
  delete self->ops;
  Py_XDECREF(self->keep);
  Py_TYPE(o)->tp_free(o);
}

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
  s_dtype = PyUnicode_InternFromString("dtype");
  s_shape = PyUnicode_InternFromString("shape");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
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
