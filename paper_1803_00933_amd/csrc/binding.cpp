// The calls of the replay path for Python, argument marshalling only: numbers, tensors (device pointers) and streams in, the
// status code and what the call reports out.  Loaded by apex.py, which documents the calls; the library itself is opened
// there too, and its entry points are looked up here by name.
//
// What a call costs the host beside its launches, and why this is not done with ctypes: a call with eight tensors took 4 us
// for their checks and addresses and for ctypes' conversion of the arguments, which is more than its launch (2.4 us).
#include <Python.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <tuple>
#include <utility>

#include "apex_replay.h"

namespace {

PyObject *g_address = nullptr;                                  // apex._ptr: address of what is no torch.Tensor
PyObject *g_plain = nullptr;                                    // apex._plain: what an argument that is no number stands for
PyObject *g_current_device = nullptr, *g_current_stream = nullptr;  // torch's raw handle of the current stream

struct Failed {};  // a Python error is set

// A reference that is given back when it goes out of scope.
struct Ref {
  PyObject *o;
  explicit Ref(PyObject *owned) : o(owned)
  {
    if (!o) throw Failed{};
  }
  Ref(const Ref &) = delete;
  ~Ref() { Py_DECREF(o); }
};

// An integer, whatever has an index (numpy's integers), or what g_plain makes one of; the value modulo 2^64.
unsigned long long integer(PyObject *o, bool plain = false)
{
  if (!PyLong_Check(o)) {
    if (PyIndex_Check(o)) return integer(Ref(PyNumber_Index(o)).o);
    if (!plain) return integer(Ref(PyObject_CallOneArg(g_plain, o)).o, true);
    PyErr_Format(PyExc_TypeError, "an integer is required, not %.80s", Py_TYPE(o)->tp_name);
    throw Failed{};
  }
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
  if (PyErr_Occurred()) throw Failed{};
  return v;
}

// The same for addresses and handles, with None for a null pointer.
void *pointer(PyObject *o)
{
  if (o == Py_None) return nullptr;
  if (PyLong_Check(o) || PyIndex_Check(o)) return reinterpret_cast<void *>(integer(o));
  const Ref p(PyObject_CallOneArg(g_plain, o));
  return p.o == Py_None ? nullptr : reinterpret_cast<void *>(integer(p.o, true));
}

// Device addresses: a contiguous tensor on the GPU, or None.
void *address(PyObject *o)
{
  if (o == Py_None) return nullptr;
  if (THPVariable_Check(o)) {
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
      PyErr_SetString(PyExc_AssertionError, "device, contiguous tensors only");
      throw Failed{};
    }
    return t.data_ptr();
  }
  return pointer(Ref(PyObject_CallOneArg(g_address, o)).o);
}

// A stream object's handle; None: the current device's current stream.
void *stream_handle(PyObject *o)
{
  if (o != Py_None) return pointer(Ref(PyObject_GetAttrString(o, "cuda_stream")).o);
  const Ref device(PyObject_CallNoArgs(g_current_device));
  return pointer(Ref(PyObject_CallOneArg(g_current_stream, device.o)).o);
}

template <typename T>
struct From {  // pointers to device memory
  static_assert(std::is_pointer<T>::value, "");
  static T get(PyObject *o) { return static_cast<T>(address(o)); }
};
template <>
struct From<apex_replay_t *> {
  static apex_replay_t *get(PyObject *o) { return static_cast<apex_replay_t *>(pointer(o)); }
};
template <>
struct From<apex_pipeline_t *> {
  static apex_pipeline_t *get(PyObject *o) { return static_cast<apex_pipeline_t *>(pointer(o)); }
};
template <>
struct From<apex_pe_replay_t *> {
  static apex_pe_replay_t *get(PyObject *o) { return static_cast<apex_pe_replay_t *>(pointer(o)); }
};
template <>
struct From<uint32_t> {
  static uint32_t get(PyObject *o) { return static_cast<uint32_t>(integer(o)); }
};
template <>
struct From<uint64_t> {
  static uint64_t get(PyObject *o) { return static_cast<uint64_t>(integer(o)); }
};
template <>
struct From<int> {
  static int get(PyObject *o) { return static_cast<int>(integer(o)); }
};
template <>
struct From<float> {
  static float get(PyObject *o)
  {
    double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred() && PyErr_ExceptionMatches(PyExc_TypeError)) {
      PyErr_Clear();
      v = PyFloat_AsDouble(Ref(PyObject_CallOneArg(g_plain, o)).o);
    }
    if (v == -1.0 && PyErr_Occurred()) throw Failed{};
    return static_cast<float>(v);
  }
};

// The last argument of the verbs that take a stream.
struct Stream {
  void *h;
  operator void *() const { return h; }
};
template <>
struct From<Stream> {
  static Stream get(PyObject *o) { return Stream{stream_handle(o)}; }
};

// What the calls give back: the status, or the status and what the call reports.
template <int N>
struct Reported {
  int rc;
  uint64_t v[N];
};
PyObject *to_python(int rc) { return PyLong_FromLong(rc); }
PyObject *to_python(const Reported<1> &r) { return Py_BuildValue("iK", r.rc, (unsigned long long)r.v[0]); }
PyObject *to_python(const Reported<2> &r)
{
  return Py_BuildValue("iKK", r.rc, (unsigned long long)r.v[0], (unsigned long long)r.v[1]);
}

// Gives the interpreter's lock up, until the end of the scope: also where an exception leaves it.
struct Unlocked {
  PyThreadState *const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

template <typename R, typename... A, size_t... I>
PyObject *invoke(R (*f)(A...), PyObject *const *args, std::index_sequence<I...>)
{
  const std::tuple<A...> a{From<A>::get(args[I])...};
  const R r = [&] {
    const Unlocked unlocked;
    return f(std::get<I>(a)...);
  }();
  return to_python(r);
}

template <typename R, typename... A>
PyObject *call(R (*f)(A...), PyObject *const *args, Py_ssize_t n)
{
  if (n != (Py_ssize_t)sizeof...(A)) {
    PyErr_Format(PyExc_TypeError, "%zd arguments are expected, not %zd", (Py_ssize_t)sizeof...(A), n);
    return nullptr;
  }
  try {
    return invoke(f, args, std::index_sequence_for<A...>{});
  } catch (const Failed &) {
  } catch (const std::exception &e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

// Entry points of the library, filled in by load().
#define APEX_ENTRIES(X)                                                                                             \
  X(apex_nstep_priorities) X(apex_replay_add) X(apex_replay_add_payload) X(apex_replay_add_publish)                 \
  X(apex_replay_add_payload_encoded) X(apex_replay_sample) X(apex_replay_sample_noalloc)                            \
  X(apex_replay_update_priorities) X(apex_replay_update_from_q) X(apex_replay_evict) X(apex_pipeline_fork)          \
  X(apex_pipeline_join) X(apex_pipeline_steps) X(apex_pipeline_add_begin) X(apex_pipeline_add_end) X(apex_pe_add)   \
  X(apex_pe_sample) X(apex_pe_update_priorities) X(apex_pe_evict_enqueue) X(apex_pe_add_round) X(apex_pe_sample_update)
#define X(name) decltype(&::name) p_##name = nullptr;
APEX_ENTRIES(X)
#undef X

#define VERB(name, ...)                                                       \
  PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n)             \
  {                                                                           \
    return call(+__VA_ARGS__, args, n);                                       \
  }

typedef apex_replay_t *Rep;
typedef apex_pipeline_t *Pipe;
typedef apex_pe_replay_t *Pe;
typedef const float *F;
typedef const uint64_t *U64;
typedef const void *V;

VERB(nstep_priorities, [](uint32_t S, uint32_t T, uint32_t n_, uint32_t A, F qo, F qt, const int32_t *ac, F rw, F dc, float alpha,
                          float eps, uint32_t frac_bits, uint64_t slots, float *prio, float *ret, float *gacc, uint64_t *fx, Stream s) {
  return p_apex_nstep_priorities(S, T, n_, A, qo, qt, ac, rw, dc, alpha, eps, frac_bits, slots, prio, ret, gacc, fx, s);
})
VERB(add, [](Rep r, uint64_t count, V obs, V act, F ret, F gacc, F prio, Stream s) {
  Reported<1> o{0, {0}};
  o.rc = p_apex_replay_add(r, count, obs, act, ret, gacc, prio, &o.v[0], s);
  return o;
})
VERB(add_payload, [](Rep r, uint64_t count, V obs, V act, F ret, F gacc, Stream s) {
  return p_apex_replay_add_payload(r, count, obs, act, ret, gacc, s);
})
VERB(add_publish, [](Rep r, uint64_t count, F prio, Stream s) {
  Reported<1> o{0, {0}};
  o.rc = p_apex_replay_add_publish(r, count, prio, &o.v[0], s);
  return o;
})
VERB(add_payload_encoded, [](Rep r, uint64_t count, V raw, uint32_t raw_bytes, V act, F ret, F gacc, Stream s) {
  return p_apex_replay_add_payload_encoded(r, count, raw, raw_bytes, act, ret, gacc, s);
})
VERB(sample, [](Rep r, uint32_t nb, uint32_t k, float beta, U64 rnd, uint64_t *key, uint32_t *slot, float *weight, void *obs,
                void *act, float *ret, float *gacc, Stream s) {
  return p_apex_replay_sample(r, nb, k, beta, rnd, key, slot, weight, obs, act, ret, gacc, s);
})
VERB(sample_noalloc, [](Rep r, uint32_t nb, uint32_t k, float beta, U64 rnd, uint64_t *key, uint32_t *slot, float *weight,
                        void *obs, void *act, float *ret, float *gacc, Stream s) {
  return p_apex_replay_sample_noalloc(r, nb, k, beta, rnd, key, slot, weight, obs, act, ret, gacc, s);
})
VERB(update_priorities, [](Rep r, uint64_t m, U64 key, F prio, Stream s) {
  return p_apex_replay_update_priorities(r, m, key, prio, s);
})
VERB(update_from_q, [](Rep r, uint64_t m, U64 key, uint32_t A, F taken, F online, F target, float *prio_out, Stream s) {
  return p_apex_replay_update_from_q(r, m, key, A, taken, online, target, prio_out, s);
})
VERB(evict, [](Rep r, Stream s) {
  Reported<1> o{0, {0}};
  o.rc = p_apex_replay_evict(r, &o.v[0], s);
  return o;
})
VERB(pipeline_fork, [](Pipe p, Stream s) { return p_apex_pipeline_fork(p, s); })
VERB(pipeline_join, [](Pipe p, Stream s) { return p_apex_pipeline_join(p, s); })
VERB(pipeline_steps, [](Pipe p, uint32_t n_, float beta, U64 rnd, F new_prio) {
  uint32_t first = 0;
  Reported<1> o{0, {0}};
  o.rc = p_apex_pipeline_steps(p, n_, beta, rnd, new_prio, &first);
  o.v[0] = first;
  return o;
})
VERB(pipeline_add_begin, [](Pipe p, uint32_t S, uint32_t T, uint32_t n_, uint32_t A, F qo, F qt, const int32_t *ac, F rw, F dc,
                            V obs, V act, float *prio, float *ret, float *gacc) {
  return p_apex_pipeline_add_begin(p, S, T, n_, A, qo, qt, ac, rw, dc, obs, act, prio, ret, gacc);
})
VERB(pipeline_add_end, [](Pipe p, int evict_) {
  Reported<2> o{0, {0, 0}};
  o.rc = p_apex_pipeline_add_end(p, evict_, &o.v[0], &o.v[1]);
  return o;
})
VERB(pe_add, [](Pe r, uint64_t count, V obs, V act, F ret, F gacc, F prio, Stream s) {
  return p_apex_pe_add(r, count, obs, act, ret, gacc, prio, s);
})
VERB(pe_sample, [](Pe r, uint32_t nb, uint32_t k, float beta, U64 rnd, uint64_t *key, uint32_t *slot, float *weight, void *obs,
                   void *act, float *ret, float *gacc, Stream s) {
  return p_apex_pe_sample(r, nb, k, beta, rnd, key, slot, weight, obs, act, ret, gacc, s);
})
VERB(pe_update_priorities, [](Pe r, uint64_t m, U64 key, F prio, Stream s) {
  return p_apex_pe_update_priorities(r, m, key, prio, s);
})
VERB(pe_evict_enqueue, [](Pe r, uint32_t rounds, U64 rnd, Stream s) {
  Reported<1> o{0, {0}};
  o.rc = p_apex_pe_evict_enqueue(r, rounds, rnd, &o.v[0], s);
  return o;
})
VERB(pe_add_round, [](Pe r, uint32_t S, uint32_t T, uint32_t n_, uint32_t A, F qo, F qt, const int32_t *ac, F rw, F dc, V obs,
                      V act, Stream s) { return p_apex_pe_add_round(r, S, T, n_, A, qo, qt, ac, rw, dc, obs, act, s); })
VERB(pe_sample_update, [](Pe r, uint32_t k, float beta, U64 rnd, F new_prio, uint64_t *key, uint32_t *slot, float *weight,
                          void *obs, void *act, float *ret, float *gacc, Stream s) {
  return p_apex_pe_sample_update(r, k, beta, rnd, new_prio, key, slot, weight, obs, act, ret, gacc, s);
})

// load(path of the library, _ptr, _plain, current device, current raw stream)
PyObject *load(PyObject *, PyObject *args)
{
  const char *path;
  PyObject *address_of, *plain, *device, *stream;
  if (!PyArg_ParseTuple(args, "sOOOO", &path, &address_of, &plain, &device, &stream)) return nullptr;
  void *const lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
  if (!lib) return PyErr_Format(PyExc_ImportError, "%s", dlerror());
#define X(name)                                                            \
  p_##name = reinterpret_cast<decltype(&::name)>(dlsym(lib, #name));       \
  if (!p_##name) return PyErr_Format(PyExc_ImportError, "%s lacks %s", path, #name);
  APEX_ENTRIES(X)
#undef X
  Py_INCREF(address_of), Py_INCREF(plain), Py_INCREF(device), Py_INCREF(stream);
  Py_XSETREF(g_address, address_of);
  Py_XSETREF(g_plain, plain);
  Py_XSETREF(g_current_device, device);
  Py_XSETREF(g_current_stream, stream);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"load", load, METH_VARARGS, nullptr},
    FAST(nstep_priorities), FAST(add), FAST(add_payload), FAST(add_publish), FAST(add_payload_encoded), FAST(sample),
    FAST(sample_noalloc), FAST(update_priorities), FAST(update_from_q), FAST(evict), FAST(pipeline_fork), FAST(pipeline_join),
    FAST(pipeline_steps), FAST(pipeline_add_begin), FAST(pipeline_add_end), FAST(pe_add), FAST(pe_sample),
    FAST(pe_update_priorities), FAST(pe_evict_enqueue), FAST(pe_add_round), FAST(pe_sample_update),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "apex_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_apex_binding(void) { return PyModule_Create(&module); }
