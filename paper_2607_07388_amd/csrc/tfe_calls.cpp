// The per-step calls of the Python binding (lookups, prefetches, head top-K)
// as functions of a CPython module: a decode step's launch is a few
// microseconds, of which marshalling its arguments through ctypes took about
// half.  Each function takes the plain case -- positional arguments, exact
// ints, floats and None, objects with data_ptr() -- and hands everything else
// to the ctypes function of the same name, whose conversions and errors
// apply.  The library's functions are bound by address, so this module links
// with nothing.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

namespace {

PyObject* g_check;         // raises for a negative status
PyObject* g_data_ptr;      // "data_ptr"
PyObject* g_cuda_stream;   // "cuda_stream"

struct Call {
  PyObject* slow;  // the ctypes function
  void* fn;
};
Call g_lookup, g_multi, g_prefetch, g_scored, g_topk;

// Each conversion returns false, with no exception set, for what the plain
// case does not cover.
bool from_int(PyObject* o, void** out) {
  if (!PyLong_CheckExact(o)) return false;
  *out = PyLong_AsVoidPtr(o);
  if (*out == nullptr && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}
bool handle(PyObject* o, void** out) {
  *out = nullptr;
  return o == Py_None || from_int(o, out);
}
bool pointer(PyObject* o, void** out) {
  if (handle(o, out)) return true;
  if (PyLong_Check(o)) return false;
  PyObject* r = PyObject_CallMethodNoArgs(o, g_data_ptr);
  if (!r) {
    PyErr_Clear();
    return false;
  }
  const bool ok = from_int(r, out);
  Py_DECREF(r);
  return ok;
}
bool stream(PyObject* o, void** out) {
  if (handle(o, out)) return true;
  if (PyLong_Check(o)) return false;
  PyObject* r = PyObject_GetAttr(o, g_cuda_stream);
  if (!r) {
    PyErr_Clear();
    return false;
  }
  const bool ok = from_int(r, out);
  Py_DECREF(r);
  return ok;
}
bool int32(PyObject* o, int32_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  const long v = PyLong_AsLongAndOverflow(o, &over);
  if (over || v < INT32_MIN || v > INT32_MAX) return false;
  *out = (int32_t)v;
  return true;
}
bool number(PyObject* o, float* out) {
  if (!PyFloat_CheckExact(o)) return false;
  *out = (float)PyFloat_AS_DOUBLE(o);
  return true;
}

PyObject* slow(const Call& c, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  return PyObject_Vectorcall(c.slow, a, (size_t)n, kw);
}
PyObject* status(int st) {
  if (st < 0) return PyObject_CallFunction(g_check, "i", st);
  return PyLong_FromLong(st);
}

#define SLOW_UNLESS(c, cond) \
  if (!(cond)) return slow(c, a, n, kw)
// Arguments [0, need) and an optional stream behind them.
#define PLAIN(c, need) \
  void* s = nullptr;   \
  SLOW_UNLESS(c, !kw && (n == (need) || (n == (need) + 1 && stream(a[need], &s))))

PyObject* lookup_inject(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  PLAIN(g_lookup, 12);
  void *t, *tok, *hin, *hout, *hit, *slot, *len;
  int32_t B, ctx, S, gate;
  float scale;
  SLOW_UNLESS(g_lookup, handle(a[0], &t) && pointer(a[1], &tok) && int32(a[2], &B) &&
                            int32(a[3], &ctx) && int32(a[4], &S) && pointer(a[5], &hin) &&
                            pointer(a[6], &hout) && pointer(a[7], &hit) && pointer(a[8], &slot) &&
                            pointer(a[9], &len) && int32(a[10], &gate) && number(a[11], &scale));
  using Fn = int (*)(void*, void*, int32_t, int32_t, int32_t, void*, void*, void*, void*, void*,
                     int32_t, float, void*);
  int st;
  Py_BEGIN_ALLOW_THREADS;
  st = ((Fn)g_lookup.fn)(t, tok, B, ctx, S, hin, hout, hit, slot, len, gate, scale, s);
  Py_END_ALLOW_THREADS;
  return status(st);
}

PyObject* lookup_inject_multi(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  PLAIN(g_multi, 12);
  void *t, *tok, *hin, *hout, *mask, *slot;
  int32_t B, ctx, S, weighting, gate;
  float scale;
  SLOW_UNLESS(g_multi, handle(a[0], &t) && pointer(a[1], &tok) && int32(a[2], &B) &&
                           int32(a[3], &ctx) && int32(a[4], &S) && pointer(a[5], &hin) &&
                           pointer(a[6], &hout) && pointer(a[7], &mask) && pointer(a[8], &slot) &&
                           int32(a[9], &weighting) && int32(a[10], &gate) && number(a[11], &scale));
  using Fn = int (*)(void*, void*, int32_t, int32_t, int32_t, void*, void*, void*, void*, int32_t,
                     int32_t, float, void*);
  int st;
  Py_BEGIN_ALLOW_THREADS;
  st = ((Fn)g_multi.fn)(t, tok, B, ctx, S, hin, hout, mask, slot, weighting, gate, scale, s);
  Py_END_ALLOW_THREADS;
  return status(st);
}

PyObject* prefetch(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  PLAIN(g_prefetch, 6);
  void *t, *tail, *cand;
  int32_t tl, B, K;
  SLOW_UNLESS(g_prefetch, handle(a[0], &t) && pointer(a[1], &tail) && int32(a[2], &tl) &&
                              pointer(a[3], &cand) && int32(a[4], &B) && int32(a[5], &K));
  using Fn = int (*)(void*, void*, int32_t, void*, int32_t, int32_t, void*);
  int st;
  Py_BEGIN_ALLOW_THREADS;
  st = ((Fn)g_prefetch.fn)(t, tail, tl, cand, B, K, s);
  Py_END_ALLOW_THREADS;
  return status(st);
}

PyObject* prefetch_scored(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  PLAIN(g_scored, 8);
  void *t, *tail, *cand, *prob;
  int32_t tl, B, K, budget;
  SLOW_UNLESS(g_scored, handle(a[0], &t) && pointer(a[1], &tail) && int32(a[2], &tl) &&
                            pointer(a[3], &cand) && pointer(a[4], &prob) && int32(a[5], &B) &&
                            int32(a[6], &K) && int32(a[7], &budget));
  using Fn = int (*)(void*, void*, int32_t, void*, void*, int32_t, int32_t, int32_t, void*);
  int st;
  Py_BEGIN_ALLOW_THREADS;
  st = ((Fn)g_scored.fn)(t, tail, tl, cand, prob, B, K, budget, s);
  Py_END_ALLOW_THREADS;
  return status(st);
}

PyObject* head_topk(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* kw) {
  PLAIN(g_topk, 6);
  void *h, *hid, *ids, *prob;
  int32_t B, K;
  SLOW_UNLESS(g_topk, handle(a[0], &h) && pointer(a[1], &hid) && int32(a[2], &B) &&
                          int32(a[3], &K) && pointer(a[4], &ids) && pointer(a[5], &prob));
  using Fn = int (*)(void*, void*, int32_t, int32_t, void*, void*, void*);
  int st;
  Py_BEGIN_ALLOW_THREADS;
  st = ((Fn)g_topk.fn)(h, hid, B, K, ids, prob, s);
  Py_END_ALLOW_THREADS;
  return status(st);
}

// bind(check, {name: (ctypes function wrapper, address)})
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *check, *calls;
  if (!PyArg_ParseTuple(args, "OO!", &check, &PyDict_Type, &calls)) return nullptr;
  const struct {
    const char* name;
    Call* c;
  } all[] = {{"tfe_lookup_inject", &g_lookup},
             {"tfe_lookup_inject_multi", &g_multi},
             {"tfe_prefetch", &g_prefetch},
             {"tfe_prefetch_scored", &g_scored},
             {"tfe_head_topk", &g_topk}};
  for (const auto& e : all) {
    PyObject* v = PyDict_GetItemString(calls, e.name);
    PyObject *f, *p;
    if (!v || !PyArg_ParseTuple(v, "OO", &f, &p)) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, e.name);
      return nullptr;
    }
    void* fn = PyLong_AsVoidPtr(p);
    if (!fn) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, e.name);
      return nullptr;
    }
    Py_INCREF(f);
    Py_XDECREF(e.c->slow);
    e.c->slow = f;
    e.c->fn = fn;
  }
  Py_INCREF(check);
  Py_XDECREF(g_check);
  g_check = check;
  Py_RETURN_NONE;
}

#define FAST METH_FASTCALL | METH_KEYWORDS
PyMethodDef g_methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"tfe_lookup_inject", (PyCFunction)(void (*)(void))lookup_inject, FAST,
     "tfe_lookup_inject($module, table, tokens, B, ctx, S, hidden_in, hidden_out, hit_mask, "
     "slot_ids, match_len, gate, scale, stream=None)\n--\n\n"},
    {"tfe_lookup_inject_multi", (PyCFunction)(void (*)(void))lookup_inject_multi, FAST,
     "tfe_lookup_inject_multi($module, table, tokens, B, ctx, S, hidden_in, hidden_out, "
     "match_mask, slot_ids, weighting, gate, scale, stream=None)\n--\n\n"},
    {"tfe_prefetch", (PyCFunction)(void (*)(void))prefetch, FAST,
     "tfe_prefetch($module, table, tail, tail_len, candidates, B, K, side_stream=None)\n--\n\n"},
    {"tfe_prefetch_scored", (PyCFunction)(void (*)(void))prefetch_scored, FAST,
     "tfe_prefetch_scored($module, table, tail, tail_len, candidates, cand_prob, B, K, budget, "
     "side_stream=None)\n--\n\n"},
    {"tfe_head_topk", (PyCFunction)(void (*)(void))head_topk, FAST,
     "tfe_head_topk($module, head, hidden, B, K, top_ids, top_prob, stream=None)\n--\n\n"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_data_ptr || !g_cuda_stream) return nullptr;
  return PyModule_Create(&g_module);
}
