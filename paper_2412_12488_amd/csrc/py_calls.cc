// CPython side of the binding: the calls an engine makes per layer or per request, from Python
// objects to the C ABI in native code.  binding.py keeps the public functions (names, arguments,
// defaults, errors) and hands their arguments here positionally; every function returns the
// mc_status, or a tuple that starts with it.
//
// Why not ctypes for these: a launch takes about 2 us, and marshalling its 10 to 16 arguments
// through ctypes took another 5 to 7 (one decode row through eight layers, 17 calls: 157 -> 149 us);
// a request's token list went through three Python-level loops (eight requests: 3.5 -> 0.55 ms).
//
// Accepted: tensors (anything with data_ptr()), integer addresses or None for buffers; c_void_p,
// integers or None for handles of host objects; the library's own mc_pool_desc; for counts what
// ctypes takes as c_int32 (integers wrap to 32 bits as C's do); sequences of numbers for token and
// page lists.  Anything else is an ArgumentError before the library is called.
//
// The interpreter lock is released around the calls that launch.  The host calls keep it: they take
// microseconds, and their objects (allocator, prefix index) are not made for several threads at once.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include <exception>
#include <memory>
#include <new>
#include <stdexcept>
#include <vector>

#include "mc_kv.h"

namespace {

PyObject* s_data_ptr;      // interned attribute names
PyObject* s_cuda_stream;
PyObject* s_value;
PyObject* s_as_parameter;
// from binding.py (setup): the types whose content is taken over, and the error for other objects
PyObject *t_pool, *t_pointer, *t_i32, *t_size, *t_error;
PyObject* g_get_device;    // torch's current-device and current-stream look-ups
PyObject* g_get_stream;

// A reference, a buffer and the released interpreter lock: given back on every way out, a C++
// exception's included.
struct Ref {
  PyObject* p;
  explicit Ref(PyObject* p_) : p(p_) {}
  ~Ref() { Py_XDECREF(p); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

struct Buffer {
  Py_buffer b;
  bool held;
  Buffer(PyObject* o, int flags) : held(PyObject_GetBuffer(o, &b, flags) == 0) {}
  ~Buffer() {
    if (held) PyBuffer_Release(&b);
  }
  Buffer(const Buffer&) = delete;
  Buffer& operator=(const Buffer&) = delete;
};

struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// Room for n >= 0 results, not cleared: the library writes what is read of it.
std::unique_ptr<int32_t[]> room(int64_t n) {
  return std::unique_ptr<int32_t[]>(new int32_t[(size_t)n + 1]);
}

// ---- one argument each; false with a Python error set ----
bool is_a(PyObject* o, PyObject* type) {
  return type && PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type));
}

bool wrong_type(PyObject* o, const char* wanted) {
  PyErr_Format(t_error ? t_error : PyExc_TypeError, "%s is expected, not %.200s", wanted,
               Py_TYPE(o)->tp_name);
  return false;
}

// What stands for o in a C call: the value of a ctypes number, or its _as_parameter_.  Null (and
// no error) if nothing does.
PyObject* stand_in(PyObject* o, PyObject* type) {
  if (is_a(o, type)) return PyObject_GetAttr(o, s_value);
  PyObject* v = PyObject_GetAttr(o, s_as_parameter);
  if (!v && PyErr_ExceptionMatches(PyExc_AttributeError)) PyErr_Clear();
  return v;
}

// An integer of any size, wrapped; type is the ctypes number that stands for it too.
bool to_u64(PyObject* o, PyObject* type, unsigned long long* out) {
  if (PyIndex_Check(o)) {
    *out = PyLong_AsUnsignedLongLongMask(o);
    return *out != (unsigned long long)-1 || !PyErr_Occurred();
  }
  const Ref v(stand_in(o, type));
  if (!v.p) return !PyErr_Occurred() && wrong_type(o, "an integer");
  if (Py_EnterRecursiveCall(" in an integer argument")) return false;
  const bool ok = to_u64(v.p, type, out);
  Py_LeaveRecursiveCall();
  return ok;
}

bool to_i32(PyObject* o, int32_t* out) {
  unsigned long long v = 0;
  if (!to_u64(o, t_i32, &v)) return false;
  *out = (int32_t)(uint32_t)v;
  return true;
}

bool to_size(PyObject* o, size_t* out) {
  unsigned long long v = 0;
  if (!to_u64(o, t_size, &v)) return false;
  *out = (size_t)v;
  return true;
}

// address or host handle: None, an integer, or a c_void_p
bool to_handle(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  if (PyLong_Check(o)) {
    *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
  }
  const Ref v(stand_in(o, t_pointer));
  if (!v.p) return !PyErr_Occurred() && wrong_type(o, "an address or a handle of this library");
  if (Py_EnterRecursiveCall(" in a pointer argument")) return false;
  const bool ok = to_handle(v.p, out);
  Py_LeaveRecursiveCall();
  return ok;
}

// device buffer: None, an integer address, or an object with data_ptr()
bool to_ptr(PyObject* o, void** out) {
  if (o == Py_None || PyLong_Check(o)) return to_handle(o, out);
  const Ref v(PyObject_CallMethodNoArgs(o, s_data_ptr));
  return v.p && to_handle(v.p, out);
}

// pool descriptor: the ctypes structure's own bytes
bool to_pool(PyObject* o, mc_pool_desc* out) {
  if (!is_a(o, t_pool)) return wrong_type(o, "an mc_pool_desc");
  const Buffer v(o, PyBUF_SIMPLE);
  if (!v.held || v.b.len < (Py_ssize_t)sizeof(mc_pool_desc)) return false;
  memcpy(out, v.b.buf, sizeof(mc_pool_desc));
  return true;
}

// stream: None = torch's current stream, an integer handle, or an object with cuda_stream
bool to_stream(PyObject* o, void** out) {
  if (o == Py_None) {
    if (!g_get_stream) {
      const Ref c(PyImport_ImportModule("torch._C"));
      if (!c.p) return false;
      if (!g_get_device) g_get_device = PyObject_GetAttrString(c.p, "_cuda_getDevice");
      if (!g_get_device) return false;
      g_get_stream = PyObject_GetAttrString(c.p, "_cuda_getCurrentRawStream");
      if (!g_get_stream) return false;
    }
    const Ref dev(PyObject_CallNoArgs(g_get_device));
    if (!dev.p) return false;
    const Ref v(PyObject_CallOneArg(g_get_stream, dev.p));
    return v.p && to_handle(v.p, out);
  }
  if (PyLong_Check(o)) return to_handle(o, out);
  const Ref v(PyObject_GetAttr(o, s_cuda_stream));
  return v.p && to_handle(v.p, out);
}

// an exact int's low 32 bits: nothing of it can fail
int32_t wrapped(PyObject* o) { return (int32_t)(uint32_t)PyLong_AsUnsignedLongLongMask(o); }

// the numbers of any iterable; int32 buffers (numpy) in one copy
bool to_numbers(PyObject* o, std::vector<int32_t>* out) {
  if (!PyList_Check(o) && !PyTuple_Check(o) && PyObject_CheckBuffer(o)) {
    const Buffer v(o, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS);
    if (!v.held) {
      PyErr_Clear();
    } else if (v.b.ndim == 1 && v.b.itemsize == 4 && v.b.format && !strcmp(v.b.format, "i")) {
      out->resize((size_t)v.b.shape[0]);
      if (v.b.len) memcpy(out->data(), v.b.buf, (size_t)v.b.len);
      return true;
    }
  }
  // Exact ints are read in place: no Python code runs between two of them.  Any other number goes
  // through its __int__, which may change the caller's own list or let another thread do so: the
  // items are then read from a copy that holds them.
  if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) {
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    PyObject** items = PySequence_Fast_ITEMS(o);
    Py_ssize_t i = 0;
    out->resize((size_t)n);
    int32_t* to = out->data();
    for (; i < n && PyLong_CheckExact(items[i]); ++i) to[i] = wrapped(items[i]);
    if (i == n) return true;
  }
  const Ref t(PySequence_Tuple(o));
  if (!t.p) return false;
  const Py_ssize_t n = PyTuple_GET_SIZE(t.p);
  out->resize((size_t)n);
  for (Py_ssize_t i = 0; i < n; ++i) {         // numpy scalars, floats: as int(x)
    const Ref v(PyNumber_Long(PyTuple_GET_ITEM(t.p, i)));
    if (!v.p || !to_i32(v.p, &(*out)[(size_t)i])) return false;
  }
  return true;
}

// page or token list: anything with a length (an iterator may be empty by the second look at it)
bool to_list(PyObject* o, std::vector<int32_t>* out) {
  return PyObject_Size(o) >= 0 && to_numbers(o, out);
}

PyObject* from_list(const int32_t* v, int64_t n) {
  PyObject* l = PyList_New((Py_ssize_t)n);
  if (!l) return nullptr;
  for (int64_t i = 0; i < n; ++i) {
    PyObject* x = PyLong_FromLong(v[i]);
    if (!x) { Py_DECREF(l); return nullptr; }
    PyList_SET_ITEM(l, (Py_ssize_t)i, x);
  }
  return l;
}

PyObject* status(mc_status st) { return PyLong_FromLong((long)st); }

// (status, value): takes the reference
PyObject* with_status(mc_status st, PyObject* value) {
  return value ? Py_BuildValue("(iN)", (int)st, value) : nullptr;
}

// Positional arguments, read in order.
struct Args {
  PyObject* const* a;
  Py_ssize_t n, at = 0;
  bool ok = true;
  Args(PyObject* const* a_, Py_ssize_t n_, Py_ssize_t want) : a(a_), n(n_) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "%zd arguments given, %zd expected", n, want);
      ok = false;
    }
  }
  template <typename T, typename F>
  T get(F f) {
    T v{};
    if (ok) ok = f(a[at++], &v);
    return v;
  }
  int32_t i32() { return get<int32_t>(to_i32); }
  // a count that sizes a result: Python integers only
  int32_t count() {
    if (ok && !PyIndex_Check(a[at])) ok = wrong_type(a[at], "an integer");
    return i32();
  }
  size_t size() { return get<size_t>(to_size); }
  void* ptr() { return get<void*>(to_ptr); }
  void* handle() { return get<void*>(to_handle); }
  void* stream() { return get<void*>(to_stream); }
  mc_pool_desc pool() { return get<mc_pool_desc>(to_pool); }
  std::vector<int32_t> list() { return get<std::vector<int32_t>>(to_list); }
  const int32_t* pi32() { return static_cast<const int32_t*>(ptr()); }
  float f32() {
    if (!ok) return 0.f;
    const Ref v(PyNumber_Float(a[at++]));      // as float(x), text included
    if (!v.p) ok = false;
    return v.p ? (float)PyFloat_AS_DOUBLE(v.p) : 0.f;
  }
};

#define CALL(expr)        \
  mc_status st;           \
  {                       \
    const Unlocked u;     \
    st = (expr);          \
  }                       \
  return status(st)

// ---- device calls ----
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 11);
  const mc_pool_desc pool = g.pool();
  const int32_t layer = g.i32();
  const void *k = g.ptr(), *v = g.ptr();
  const int32_t batch = g.i32(), tq = g.i32();
  const int32_t *cu_q = g.pi32(), *begin = g.pi32(), *table = g.pi32(), *cu_pages = g.pi32();
  void* stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_kv_append(&pool, layer, k, v, batch, tq, cu_q, begin, table, cu_pages, stream));
}

PyObject* append_send(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 16);
  const mc_pool_desc pool = g.pool();
  const int32_t layer = g.i32();
  const void *k = g.ptr(), *v = g.ptr();
  const int32_t batch = g.i32(), tq = g.i32();
  const int32_t *cu_q = g.pi32(), *begin = g.pi32(), *table = g.pi32(), *cu_pages = g.pi32();
  const int32_t first = g.i32();
  const int32_t *s0 = g.pi32(), *s1 = g.pi32();
  const int64_t* off = static_cast<const int64_t*>(g.ptr());
  void *buf = g.ptr(), *stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_kv_append_send(&pool, layer, k, v, batch, tq, cu_q, begin, table, cu_pages, first, s0,
                         s1, off, buf, stream));
}

// plan(pool, hq, batch, total_q, cu_q, begin, table, cu_pages, ahead, ws, ws_bytes, stream)
PyObject* plan(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 12);
  const mc_pool_desc pool = g.pool();
  const int32_t hq = g.i32(), batch = g.i32(), tq = g.i32();
  const int32_t *cu_q = g.pi32(), *begin = g.pi32(), *table = g.pi32(), *cu_pages = g.pi32();
  const int32_t ahead = g.i32();
  void* ws = g.ptr();
  const size_t bytes = g.size();
  void* stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_attn_plan_ahead(&pool, hq, batch, tq, cu_q, begin, table, cu_pages, ahead, ws, bytes,
                          stream));
}

PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 16);
  const mc_pool_desc pool = g.pool();
  const int32_t layer = g.i32();
  const void* q = g.ptr();
  const int32_t hq = g.i32(), batch = g.i32(), tq = g.i32();
  const int32_t *cu_q = g.pi32(), *begin = g.pi32(), *table = g.pi32(), *cu_pages = g.pi32();
  const float scale = g.f32();
  void* out = g.ptr();
  float* lse = static_cast<float*>(g.ptr());
  void* ws = g.ptr();
  const size_t bytes = g.size();
  void* stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_prefix_prefill_attn(&pool, layer, q, hq, batch, tq, cu_q, begin, table, cu_pages, scale,
                              out, lse, ws, bytes, stream));
}

PyObject* attn_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 14);
  const mc_pool_desc pool = g.pool();
  const int32_t layer = g.i32();
  const void* q = g.ptr();
  const int32_t hq = g.i32(), batch = g.i32(), tq = g.i32();
  const int32_t *cu_q = g.pi32(), *begin = g.pi32(), *table = g.pi32(), *cu_pages = g.pi32();
  const float scale = g.f32();
  void* out = g.ptr();
  float* lse = static_cast<float*>(g.ptr());
  void* stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_prefix_prefill_attn_noalloc(&pool, layer, q, hq, batch, tq, cu_q, begin, table, cu_pages,
                                      scale, out, lse, stream));
}

template <bool kPack>
PyObject* copy_range(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 9);
  const mc_pool_desc pool = g.pool();
  const int32_t l0 = g.i32(), l1 = g.i32();
  const int32_t* pages = g.pi32();
  const int32_t n_pages = g.i32(), s0 = g.i32(), s1 = g.i32();
  void *buf = g.ptr(), *stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(kPack ? mc_kv_pack_range(&pool, l0, l1, pages, n_pages, s0, s1, buf, stream)
             : mc_kv_unpack_range(&pool, l0, l1, pages, n_pages, s0, s1, buf, stream));
}

template <bool kPack>
PyObject* copy_batch(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 12);
  const mc_pool_desc pool = g.pool();
  const int32_t l0 = g.i32(), l1 = g.i32(), batch = g.i32();
  const int32_t *table = g.pi32(), *cu_pages = g.pi32(), *s0 = g.pi32(), *s1 = g.pi32();
  const int64_t* off = static_cast<const int64_t*>(g.ptr());
  const int32_t most = g.i32();
  void *buf = g.ptr(), *stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(kPack ? mc_kv_pack_batch(&pool, l0, l1, batch, table, cu_pages, s0, s1, off, most, buf, stream)
             : mc_kv_unpack_batch(&pool, l0, l1, batch, table, cu_pages, s0, s1, off, most, buf,
                                  stream));
}

PyObject* copy_page(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 7);
  const mc_pool_desc pool = g.pool();
  const int32_t l0 = g.i32(), l1 = g.i32(), src = g.i32(), dst = g.i32(), slots = g.i32();
  void* stream = g.stream();
  if (!g.ok) return nullptr;
  CALL(mc_kv_copy_page(&pool, l0, l1, src, dst, slots, stream));
}

// ---- host calls ----
PyObject* alloc_pages(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 2);
  void* alloc = g.handle();
  const int32_t want = g.count();
  if (!g.ok) return nullptr;
  // room for what the pool can give: the library refuses more before it writes any
  int32_t free_now = 0;
  mc_kv_allocator_num_free(alloc, &free_now);
  const auto out = room(want > free_now ? free_now : want > 0 ? want : 0);
  const mc_status st = mc_kv_alloc_pages(alloc, want, out.get());
  return with_status(st, from_list(out.get(), st == MC_OK ? want : 0));
}

PyObject* free_pages(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 2);
  void* alloc = g.handle();
  const std::vector<int32_t> pages = g.list();
  if (!g.ok) return nullptr;
  return status(mc_kv_free_pages(alloc, (int32_t)pages.size(), pages.data()));
}

PyObject* check_page_table(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 2);
  const std::vector<int32_t> pages = g.list();
  const int32_t num_pages = g.i32();
  if (!g.ok) return nullptr;
  return status(mc_kv_check_page_table(pages.data(), (int64_t)pages.size(), num_pages));
}

PyObject* plan_remote_send(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 4);
  const int32_t sm = g.i32(), rm = g.i32(), begin = g.i32(), end = g.i32();
  if (!g.ok) return nullptr;
  mc_send_plan p = {};
  const mc_status st = mc_plan_remote_send(sm, rm, begin, end, &p);
  return Py_BuildValue("(i(ii)(ii)(ii))", (int)st, p.copy_begin, p.copy_end, p.prefill_begin,
                       p.prefill_end, p.send_begin, p.send_end);
}

PyObject* addr_compress(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 1);
  const std::vector<int32_t> pages = g.list();
  if (!g.ok) return nullptr;
  const auto runs = room(2 * (int64_t)pages.size());
  int32_t nr = 0;
  const mc_status st = mc_addr_compress(pages.data(), (int32_t)pages.size(), runs.get(), &nr);
  if (st != MC_OK) nr = 0;
  PyObject* l = PyList_New(nr);
  for (int32_t i = 0; l && i < nr; ++i) {
    PyObject* t = PyTuple_New(2);
    PyObject *first = PyLong_FromLong(runs[2 * i]), *count = PyLong_FromLong(runs[2 * i + 1]);
    if (!t || !first || !count) {
      Py_XDECREF(t); Py_XDECREF(first); Py_XDECREF(count);
      Py_CLEAR(l);
      break;
    }
    PyTuple_SET_ITEM(t, 0, first);
    PyTuple_SET_ITEM(t, 1, count);
    PyList_SET_ITEM(l, i, t);
  }
  return with_status(st, l);
}

// addr_expand(runs, capacity or None)
PyObject* addr_expand(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 2);
  if (!g.ok) return nullptr;
  if (PyObject_Size(a[0]) < 0) return nullptr;
  const Ref f(PySequence_Tuple(a[0]));   // a run's own numbers may run Python code: see to_numbers
  if (!f.p) return nullptr;
  const Py_ssize_t n_runs = PyTuple_GET_SIZE(f.p);
  std::vector<int32_t> flat;
  flat.reserve(2 * (size_t)n_runs);
  std::vector<int32_t> pair;
  int64_t sum = 0;
  for (Py_ssize_t i = 0; i < n_runs; ++i) {
    PyObject* r = PyTuple_GET_ITEM(f.p, i);
    if (PyTuple_CheckExact(r) && PyTuple_GET_SIZE(r) == 2 && PyLong_CheckExact(PyTuple_GET_ITEM(r, 0)) &&
        PyLong_CheckExact(PyTuple_GET_ITEM(r, 1))) {
      pair.assign({wrapped(PyTuple_GET_ITEM(r, 0)), wrapped(PyTuple_GET_ITEM(r, 1))});
    } else if (!to_numbers(r, &pair)) {
      return nullptr;
    }
    // joined without this check, numbers of a malformed run would be read as the next run's
    if (pair.size() != 2)
      return PyErr_Format(PyExc_ValueError, "run %zd holds %zu numbers, not (first page, count)", i,
                          pair.size());
    if (pair[1] > 0) sum += pair[1];
    flat.insert(flat.end(), pair.begin(), pair.end());
  }
  int32_t capacity = 0;
  if (a[1] != Py_None) {
    if (!PyIndex_Check(a[1])) { wrong_type(a[1], "an integer"); return nullptr; }
    if (!to_i32(a[1], &capacity)) return nullptr;
  } else {
    capacity = (int32_t)(sum < 0x7fffffff ? sum : 0x7fffffff);
  }
  // The runs come from another engine: no room is taken for counts that the capacity refuses.
  if (capacity > 0 && sum > capacity) capacity = 0;
  const auto out = room(sum <= capacity ? sum : 0);
  int32_t got = 0;
  const mc_status st = mc_addr_expand(flat.data(), (int32_t)n_runs, out.get(), capacity, &got);
  return with_status(st, from_list(out.get(), st == MC_OK ? got : 0));
}

PyObject* index_insert(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 3);
  void* index = g.handle();
  const std::vector<int32_t> tokens = g.list(), pages = g.list();
  if (!g.ok) return nullptr;
  if (pages.size() < tokens.size() / 16) {
    PyErr_SetString(PyExc_IndexError, "fewer pages than whole blocks of tokens");
    return nullptr;
  }
  return status(mc_prefix_index_insert(index, tokens.data(), (int32_t)tokens.size(), pages.data()));
}

PyObject* index_match(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 2);
  void* index = g.handle();
  const std::vector<int32_t> tokens = g.list();
  if (!g.ok) return nullptr;
  const auto out = room((int64_t)tokens.size() / 16);
  int32_t m = 0;
  const mc_status st =
      mc_prefix_index_match(index, tokens.data(), (int32_t)tokens.size(), out.get(), &m);
  PyObject* l = from_list(out.get(), st == MC_OK ? m / 16 : 0);
  return l ? Py_BuildValue("(iiN)", (int)st, (int)m, l) : nullptr;
}

// prep_recv(index, alloc, prompt, end) -> (status, match_len, pages)
PyObject* prep_recv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  Args g(a, n, 4);
  void *index = g.handle(), *alloc = g.handle();
  const std::vector<int32_t> prompt = g.list();
  const int32_t end = g.count();
  if (!g.ok) return nullptr;
  if (end > 0 && (size_t)end > prompt.size()) {
    PyErr_SetString(PyExc_IndexError, "end lies beyond the prompt");
    return nullptr;
  }
  const int64_t pages = end > 0 ? ((int64_t)end + 15) / 16 : 0;
  const auto out = room(pages);
  int32_t m = 0;
  const mc_status st = mc_prep_recv(index, alloc, prompt.data(), end, out.get(), &m);
  PyObject* l = from_list(out.get(), st == MC_OK ? pages : 0);
  return l ? Py_BuildValue("(iiN)", (int)st, (int)m, l) : nullptr;
}

// C++ exceptions end here: one that reached the interpreter would end the process.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (const std::bad_alloc&) {
    return PyErr_NoMemory();
  } catch (const std::length_error&) {
    return PyErr_NoMemory();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// setup(mc_pool_desc, c_void_p, c_int32, c_size_t, error): once, by binding.py
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5) return PyErr_Format(PyExc_TypeError, "%zd arguments given, 5 expected", n);
  PyObject** to[5] = {&t_pool, &t_pointer, &t_i32, &t_size, &t_error};
  for (int i = 0; i < 5; ++i)
    if (!PyType_Check(a[i])) return PyErr_Format(PyExc_TypeError, "types are expected");
  for (int i = 0; i < 5; ++i) {
    Py_INCREF(a[i]);
    Py_XSETREF(*to[i], a[i]);
  }
  Py_RETURN_NONE;
}

#define ENTRY(name, fn) {name, (PyCFunction)(void (*)(void))guarded<fn>, METH_FASTCALL, nullptr}
#define FN(fn) ENTRY(#fn, fn)
PyMethodDef kMethods[] = {
    FN(setup), FN(append), FN(append_send), FN(plan), FN(attn), FN(attn_noalloc), FN(copy_page),
    ENTRY("pack_range", copy_range<true>), ENTRY("unpack_range", copy_range<false>),
    ENTRY("pack_batch", copy_batch<true>), ENTRY("unpack_batch", copy_batch<false>),
    FN(alloc_pages), FN(free_pages), FN(check_page_table), FN(plan_remote_send),
    FN(addr_compress), FN(addr_expand), FN(index_insert), FN(index_match), FN(prep_recv),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_calls",
                       "Native argument marshalling for the calls of libmc_kv.so.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_value = PyUnicode_InternFromString("value");
  s_as_parameter = PyUnicode_InternFromString("_as_parameter_");
  if (!s_data_ptr || !s_cuda_stream || !s_value || !s_as_parameter) return nullptr;
  return PyModule_Create(&kModule);
}
