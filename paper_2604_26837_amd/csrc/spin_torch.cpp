// Python calls of the stage entry points with torch tensors as arguments, without ctypes.
//
// A decode step of a short context is a few launches of a few microseconds each, and marshalling a call's dozen
// tensors in Python (attribute look-ups, contiguity and type checks, ctypes conversions) took about 9 us per call,
// more than the kernel it launched.  Here a call's arguments are checked and converted in one C++ function: about 3 us
// with the launch, so that a step of one request of 4096 tokens is bound by its kernels (27.5 -> 14.0 us).
//
// Every function takes the C entry point's arguments in order, with these differences: tensors for pointers (None for
// NULL), no size after a pool or a leaf table (it is the tensor's own), no stream (the current one).  The checks are
// those of binding._ptr: on the GPU, contiguous, of the documented type.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <string>
#include <utility>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "spin.h"

namespace {

// the `index`-th of the comma-separated names (of the tensor arguments)
std::string nth_name(const char *names, int index) {
  const char *p = names;
  for (; index > 0 && p; --index) {
    p = strchr(p, ',');
    if (p) ++p;
  }
  if (!p) return "tensor";
  const char *e = strchr(p, ',');
  return e ? std::string(p, e) : std::string(p);
}

struct tensor_info {
  int64_t ptr, numel, itemsize, rows;
};

bool refuse(const std::string &text) {
  PyErr_SetString(PyExc_ValueError, text.c_str());
  return false;
}

bool wrong_type(PyObject *o, const std::string &name, const char *want) {
  PyObject *dtype = PyObject_GetAttrString(o, "dtype");
  if (!dtype) return false;
  PyErr_Format(PyExc_ValueError, "%s must be torch.%s, got %S", name.c_str(), want, dtype);
  Py_DECREF(dtype);
  return false;
}

const char *type_name(char kind) {
  switch (kind) {
    case 'b': return "bfloat16";
    case 'f': return "float32";
    case 'i': case 'L': return "int32";
    case 's': return "int16";
    case 'l': return "int64";
    default: return nullptr;   // any type
  }
}

bool is_type(const at::Tensor &t, char kind) {
  switch (kind) {
    case 'b': return t.scalar_type() == at::kBFloat16;
    case 'f': return t.scalar_type() == at::kFloat;
    case 'i': case 'L': return t.scalar_type() == at::kInt;
    case 's': return t.scalar_type() == at::kShort;
    case 'l': return t.scalar_type() == at::kLong;
    default: return true;
  }
}

// an integer attribute, or the integer a method without arguments returns
bool int_of(PyObject *o, const char *name, bool method, int64_t &out) {
  PyObject *v = method ? PyObject_CallMethod(o, name, nullptr) : PyObject_GetAttrString(o, name);
  if (!v) return false;
  out = PyLong_AsLongLong(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}
// 1, 0, or -1 with an exception set
int truth_of(PyObject *o, const char *name, bool method) {
  PyObject *v = method ? PyObject_CallMethod(o, name, nullptr) : PyObject_GetAttrString(o, name);
  if (!v) return -1;
  const int t = PyObject_IsTrue(v);
  Py_DECREF(v);
  return t;
}

// Objects that are no plain tensors (subclasses, or anything with a tensor's methods) are asked through Python.
bool foreign_tensor(PyObject *o, char kind, const std::string &name, tensor_info &t) {
  int yes = truth_of(o, "is_cuda", false);
  if (yes < 0) return false;
  if (!yes) return refuse(name + " must live on the GPU");
  yes = truth_of(o, "is_contiguous", true);
  if (yes < 0) return false;
  if (!yes) return refuse(name + " must be contiguous");
  if (const char *want = type_name(kind)) {
    PyObject *dtype = PyObject_GetAttrString(o, "dtype");
    PyObject *text = dtype ? PyObject_Str(dtype) : nullptr;
    Py_XDECREF(dtype);
    if (!text) return false;
    const char *s = PyUnicode_AsUTF8(text);
    const bool same = s && std::string(s) == std::string("torch.") + want;
    Py_DECREF(text);
    if (!s) return false;
    if (!same) return wrong_type(o, name, want);
  }
  if (!int_of(o, "data_ptr", true, t.ptr)) return false;
  if (kind == 'P') return int_of(o, "numel", true, t.numel) && int_of(o, "element_size", true, t.itemsize);
  if (kind == 'L') {
    PyObject *shape = PyObject_GetAttrString(o, "shape");
    PyObject *first = shape ? PySequence_GetItem(shape, 0) : nullptr;
    Py_XDECREF(shape);
    if (!first) return false;
    t.rows = PyLong_AsLongLong(first);
    Py_DECREF(first);
    return !PyErr_Occurred();
  }
  return true;
}

bool tensor_of(PyObject *o, char kind, const char *names, int index, tensor_info &t) {
  if (!THPVariable_CheckExact(o)) return foreign_tensor(o, kind, nth_name(names, index), t);
  const at::Tensor &x = THPVariable_Unpack(o);
  if (!x.is_cuda()) return refuse(nth_name(names, index) + " must live on the GPU");
  if (!x.is_contiguous()) return refuse(nth_name(names, index) + " must be contiguous");
  if (!is_type(x, kind)) return wrong_type(o, nth_name(names, index), type_name(kind));
  t.ptr = (int64_t)(uintptr_t)x.data_ptr();
  if (kind == 'P') {
    t.numel = x.numel();
    t.itemsize = (int64_t)x.element_size();
  } else if (kind == 'L') {
    t.rows = x.size(0);
  }
  return true;
}

// Kinds of the C arguments, one character each: n an integer (the context and addresses of host memory among them);
// tensors: a any type, b bfloat16, f float32, i int32, s int16, l int64, P the slot pool and L the leaf table, each
// followed by # for its size (slots of 8192 bytes, leaves); S the current stream.
template <size_t N>
bool gather_arguments(const char *kinds, const char *names, PyObject *const *args, Py_ssize_t nargs,
                      int64_t (&value)[N]) {
  Py_ssize_t at = 0;
  int tensors = 0;
  for (size_t i = 0; i < N; ++i) {
    const char kind = kinds[i];
    if (kind == 'S') {
      value[i] = (int64_t)(uintptr_t)c10::hip::getCurrentHIPStream().stream();
      continue;
    }
    if (at >= nargs) {
      PyErr_SetString(PyExc_TypeError, "too few arguments");
      return false;
    }
    PyObject *o = args[at++];
    if (kind == 'n') {
      if (!PyIndex_Check(o)) {            // (numpy's integers and tensors of one integer are none of Python's)
        PyErr_Format(PyExc_TypeError, "an integer is wanted, got %R", o);
        return false;
      }
      value[i] = (int64_t)PyLong_AsUnsignedLongLongMask(o);
      if (value[i] == -1 && PyErr_Occurred()) return false;
      continue;
    }
    tensor_info t = {0, 0, 0, 0};
    const bool sized = i + 1 < N && kinds[i + 1] == '#';
    if (o == Py_None && !sized) {
      value[i] = 0;
    } else {
      if (!tensor_of(o, kind, names, tensors, t)) return false;
      value[i] = t.ptr;
    }
    ++tensors;
    if (sized) value[++i] = kind == 'P' ? t.numel * t.itemsize / SPIN_SLOT_BYTES : t.rows;
  }
  if (at != nargs) {
    PyErr_SetString(PyExc_TypeError, "too many arguments");
    return false;
  }
  return true;
}

template <typename T>
T argument(int64_t v) {
  if constexpr (std::is_pointer_v<T>) return reinterpret_cast<T>((uintptr_t)v);
  else return static_cast<T>(v);
}

template <typename F>
struct entry;
template <typename... A>
struct entry<int(A...)> {
  static constexpr size_t count = sizeof...(A);
  template <size_t... I>
  static int invoke(void *address, const int64_t (&v)[sizeof...(A)], std::index_sequence<I...>) {
    return reinterpret_cast<int (*)(A...)>(address)(argument<A>(v[I])...);
  }
  static PyObject *call(void *address, const char *kinds, const char *names, PyObject *const *args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (!address) {
      PyErr_SetString(PyExc_RuntimeError, "the library's entry points are not bound yet");
      return nullptr;
    }
    int64_t v[sizeof...(A)];
    if (!gather_arguments(kinds, names, args, nargs, v)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = invoke(address, v, std::make_index_sequence<sizeof...(A)>());
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
    END_HANDLE_TH_ERRORS
  }
};

#define STEP_LISTS "slots,page_ids,valid_mask,npages"
// entry point, kinds of its arguments, names of its tensor arguments
#define SPIN_ENTRIES(E)                                                                                                \
  E(spin_pack_kv_pages, "nnbbiP#S", "src_k,src_v,slots,kv_pool")                                                       \
  E(spin_build_summaries, "nnP#iL#iiiaaS", "kv_pool,dir,leaf_pool,part_offsets,seq_lens,chan_idx,summaries,workspace") \
  E(spin_append_kv, "nnbbiP#iL#iiaaS",                                                                                 \
    "k_new,v_new,seq_lens,kv_pool,dir,leaf_pool,part_offsets,chan_idx,summaries,workspace")                            \
  E(spin_score_partitions, "nnbaiiifaS", "q,summaries,chan_idx,part_offsets,seq_lens,scores,workspace")                \
  E(spin_select_topk, "nnfiiiiaS", "scores,part_offsets,seq_lens,sel,nsel,workspace")                                  \
  E(spin_score_select_topk, "nnbaiiifiiaS", "q,summaries,chan_idx,part_offsets,seq_lens,scores,sel,nsel,workspace")    \
  E(spin_resolve_slots, "nnniiiiL#iiiisiiiiaS",                                                                        \
    "sel,nsel,seq_lens,dir,leaf_pool,rev_table,slot_base," STEP_LISTS ",miss_pages,miss_slots,nmiss,workspace")        \
  E(spin_select_resolve, "nnfiiiiiL#iisiaS",                                                                           \
    "scores,part_offsets,seq_lens,sel,nsel,dir,leaf_pool," STEP_LISTS ",workspace")                                    \
  E(spin_score_select_resolve, "nnbaiiifiiiL#iisiaS",                                                                  \
    "q,summaries,chan_idx,part_offsets,seq_lens,scores,sel,nsel,dir,leaf_pool," STEP_LISTS ",workspace")               \
  E(spin_select_resolve_forced, "nnfiiiiiL#iisibP#aS",                                                                 \
    "scores,part_offsets,seq_lens,sel,nsel,dir,leaf_pool," STEP_LISTS ",q,kv_pool,workspace")                          \
  E(spin_select_resolve_decode, "nnfiiiiiL#iisibP#bfaS",                                                               \
    "scores,part_offsets,seq_lens,sel,nsel,dir,leaf_pool," STEP_LISTS ",q,kv_pool,out,lse,workspace")                  \
  E(spin_decode_step, "nnbaiiifiiiL#iisiP#bfaS",                                                                       \
    "q,summaries,chan_idx,part_offsets,seq_lens,scores,sel,nsel,dir,leaf_pool," STEP_LISTS ",kv_pool,out,lse,workspace") \
  E(spin_gather_decode, "nnbnliiiP#iisisbfaS",                                                                         \
    "q,row_base,nmiss,miss_pages,miss_slots,kv_pool,slots,page_ids,valid_mask,npages,miss_mask,out,lse,workspace")     \
  E(spin_gather_misses, "nnnliiiP#aS", "row_base,nmiss,miss_pages,miss_slots,kv_pool,workspace")                       \
  E(spin_offload_pages, "nnP#nliiiaS", "kv_pool,row_base,count,pages,slots,workspace")                                 \
  E(spin_split_hits_misses, "nnisiiissS", "page_ids,valid_mask,npages,miss_pages,nmiss,mask_hits,mask_misses")         \
  E(spin_sparse_decode, "nnbP#isibfaS", "q,kv_pool,slots,valid_mask,npages,out,lse,workspace")                         \
  E(spin_sparse_decode_rest, "nnbP#isibfaS", "q,kv_pool,slots,valid_mask,npages,out,lse,workspace")                    \
  E(spin_sparse_decode_begin, "nnbP#isiaS", "q,kv_pool,slots,valid_mask,npages,workspace")                             \
  E(spin_sparse_decode_finish, "nnbP#isibfaS", "q,kv_pool,slots,valid_mask,npages,out,lse,workspace")                  \
  E(spin_sparse_decode_static, "nnbP#isibfiS", "q,kv_pool,slots,valid_mask,npages,out,lse,status")

#define SPIN_DEFINE(NAME, KINDS, NAMES)                                                                       \
  static_assert(sizeof(KINDS) - 1 == entry<decltype(NAME)>::count, "one kind per argument of " #NAME);       \
  void *address_of_##NAME = nullptr;                                                                          \
  PyObject *py_##NAME(PyObject *, PyObject *const *args, Py_ssize_t nargs) {                                  \
    return entry<decltype(NAME)>::call(address_of_##NAME, KINDS, NAMES, args, nargs);                         \
  }
SPIN_ENTRIES(SPIN_DEFINE)

// bind(name, address): where the loaded library has the entry point
PyObject *py_bind(PyObject *, PyObject *args) {
  const char *name;
  unsigned long long address;
  if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
#define SPIN_BIND(NAME, KINDS, NAMES) \
  if (!strcmp(name, #NAME)) { address_of_##NAME = reinterpret_cast<void *>((uintptr_t)address); Py_RETURN_NONE; }
  SPIN_ENTRIES(SPIN_BIND)
  PyErr_Format(PyExc_KeyError, "%s", name);
  return nullptr;
}

#define SPIN_METHOD(NAME, KINDS, NAMES) \
  {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    SPIN_ENTRIES(SPIN_METHOD)
    {"bind", py_bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

#define SPIN_NAME(NAME, KINDS, NAMES) #NAME ","
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_spin_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__spin_torch() {
  PyObject *m = PyModule_Create(&module);
  // "a,b,c,": the entry points there are
  if (m && PyModule_AddStringConstant(m, "ENTRIES", SPIN_ENTRIES(SPIN_NAME)) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
