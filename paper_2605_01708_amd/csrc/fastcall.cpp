// The short way from Python into libsplitzip.so for the calls that a serving loop repeats: what the ctypes binding does
// with a call's arguments, done here in one step (argument marshalling only; the library does everything else).
//
// A small call is bound by the host: one launch costs it 2.3 us, and marshalling a compress call in Python and ctypes
// cost 2.3 us on top of its two launches (numel, element_size, is_contiguous, data_ptr of four tensors: 1.3; ctypes:
// 1.0), a decompress call 2.0 on top of one; this way it is 0.7 a call.  compress + decompress of a 4 MiB tensor, enqueued one
// after the other: 11.9 us, now 8.5.
//
// Only the plain form of every argument is taken -- tensors that are torch.Tensor itself, on the GPU, Python integers,
// the binding's own ctypes structures, no torch function mode watching -- and only if the checks of the Python side hold.
// Anything else is left to the general way in binding.py, which also raises the errors: a function here answers the
// library's code (0 or negative), or 1 if it has done nothing.
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <type_traits>
#include <utility>

#include "splitzip.h"

namespace {

constexpr int kNotTaken = 1;
constexpr int kMost = 12;   // arguments of an entry point, at most

// the library's function called with its own types, from as many 64-bit words
template <typename A>
A arg(uint64_t w) {
  if constexpr (std::is_pointer_v<A>) return reinterpret_cast<A>(static_cast<uintptr_t>(w));
  else return static_cast<A>(w);
}
template <typename F>
struct Caller;
template <typename... A>
struct Caller<int(A...)> {
  static constexpr int kArgs = sizeof...(A);
  static_assert(kArgs <= kMost, "room for the words");
  template <size_t... I>
  static int with(void* fn, const uint64_t* w, std::index_sequence<I...>) { return reinterpret_cast<int (*)(A...)>(fn)(arg<A>(w[I])...); }
  static int call(void* fn, const uint64_t* w) { return with(fn, w, std::index_sequence_for<A...>()); }
};

// What a call's Python arguments are, a letter each (two letters where it says "and"), and the words they become:
//   W  words, a contiguous tensor: address and number of elements; the size of one is compared with the dtype that a
//      C, V or D names
//   P  a tensor: its address
//   Z  a sizes record, a tensor in the GPU's memory or (pinned) in the host's: its address      z  the same, or None: null
//   R  room, a tensor, and its capacity in bytes or None (all of it): address, bytes
//   Y  room for decoded words, a contiguous tensor of at least the elements that the N before it says: its address
//   I  an integer                       N  the same: the elements of a stream
//   D  an integer: the dtype
//   A  a ctypes array of items: its address                G  a page geometry: its address
//   C  a codebook: its dtype and its address               K  a codebook: its address alone
//   V  a format of the variants: its address
//   S  a stream's handle, or None: the current one
constexpr bool in(const char* set, char c) { return *set && (*set == c || in(set + 1, c)); }
constexpr int count(const char* spec, const char* twice) { return *spec ? (in(twice, *spec) ? 2 : 1) + count(spec + 1, twice) : 0; }
constexpr bool known(const char* spec) { return !*spec || (in("WPZzRYINDAGCKVS", *spec) && known(spec + 1)); }
struct Entry {
  const char* name;
  const char* spec;
  int n_words, n_args;   // of the library's function, of Python's
  int (*call)(void*, const uint64_t*);
};
#define ENTRY(NAME, SPEC) {#NAME, SPEC, Caller<decltype(NAME)>::kArgs, count(SPEC, "R"), &Caller<decltype(NAME)>::call}
constexpr Entry kEntries[] = {
    ENTRY(splitzip_compress, "WCRPIZS"),
    ENTRY(splitzip_decompress, "PINCYzS"),
    ENTRY(splitzip_compress_noalloc, "WCRZS"),
    ENTRY(splitzip_compress_dcb, "WDPRPIZS"),
    ENTRY(splitzip_decompress_dcb, "PINDPYzS"),
    ENTRY(splitzip_decompress_own, "PINDYzS"),
    ENTRY(splitzip_compress_paged, "GICRPIZS"),
    ENTRY(splitzip_decompress_paged, "PIICGzS"),
    ENTRY(splitzip_compress_batch, "AIIPIZS"),
    ENTRY(splitzip_decompress_batch, "AIIzS"),
    ENTRY(splitzip_compress_batch_dcb, "AIIPPIZS"),
    ENTRY(splitzip_decompress_batch_dcb, "AIIPzS"),
    ENTRY(splitzip_decompress_batch_own, "AIIzS"),
    ENTRY(splitzip_compress_batch_paged, "AIIGPIZS"),
    ENTRY(splitzip_decompress_batch_paged, "AIIGzS"),
    ENTRY(splitzip_calibrate_batch_device, "AIIPPS"),
    ENTRY(splitzip_variant_compress, "WVKRRZS"),
    ENTRY(splitzip_variant_decompress, "PINVKYzS"),
};
#undef ENTRY
constexpr bool fit(size_t k) {
  return k == 0 || (known(kEntries[k - 1].spec) && count(kEntries[k - 1].spec, "WRC") == kEntries[k - 1].n_words && fit(k - 1));
}
static_assert(fit(sizeof kEntries / sizeof kEntries[0]), "a letter for every argument of the library's functions");

// the binding's ctypes structures, as bind was given them
struct Types {
  PyObject *codebook, *variant, *paged;
};
struct Bound {
  void* fn;
  const Entry* entry;
  Types types;   // references held
};

// Nothing here is refused by a C++ exception: one takes 2.5 to 4 us, more than a launch, and a program that always passes
// another form (its default device set, parameters) would pay that with every call.
const at::Tensor* tensor(PyObject* o, bool host_too = false) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return (t.is_cuda() || (host_too && t.is_cpu())) && t.layout() == at::kStrided ? &t : nullptr;
}
bool integer(PyObject* o, uint64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsUnsignedLongLong(o);
  if (*v != ~0ull || !PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}
// the memory of a ctypes object, held until the call has returned
struct Views {
  Py_buffer held[4];
  int n = 0;
  void* of(PyObject* o, const PyObject* type, Py_ssize_t least) {
    if (type && reinterpret_cast<const PyObject*>(Py_TYPE(o)) != type) return nullptr;
    if (n == 4 || !PyObject_CheckBuffer(o)) return nullptr;
    if (PyObject_GetBuffer(o, &held[n], PyBUF_SIMPLE | PyBUF_WRITABLE) != 0) {
      PyErr_Clear();
      return nullptr;
    }
    ++n;
    return held[n - 1].len < least ? nullptr : held[n - 1].buf;
  }
  ~Views() {
    for (int i = 0; i < n; ++i) PyBuffer_Release(&held[i]);
  }
};
int64_t bytes_per_word(uint64_t dtype) { return dtype == SPLITZIP_BF16 ? 2 : 1; }

// false if an argument is not of the plain form: nothing has been done then
bool run(const Bound& b, PyObject* const* a, Py_ssize_t n_args, int* rc) {
  if (n_args != b.entry->n_args || at::impl::torch_function_mode_enabled()) return false;
  Views views;
  uint64_t w[kMost];
  int n = 0;
  int64_t word_size = 0, expected = 0;   // bytes of a word, of the tensor and by the dtype
  uint64_t elems = 0, v = 0;
  const auto word = [&](uint64_t x) { w[n++] = x; };
  const auto address = [](const void* p) { return static_cast<uint64_t>(reinterpret_cast<uintptr_t>(p)); };
  for (const char* s = b.entry->spec; *s; ++s) {
    PyObject* o = *a++;
    switch (*s) {
      case 'W': {
        const at::Tensor* t = tensor(o);
        if (!t || !t->is_contiguous()) return false;
        word_size = t->element_size();
        word(address(t->data_ptr()));
        word(static_cast<uint64_t>(t->numel()));
        break;
      }
      case 'Y': {
        const at::Tensor* t = tensor(o);
        if (!t || !t->is_contiguous() || static_cast<uint64_t>(t->numel()) < elems) return false;
        word_size = t->element_size();
        word(address(t->data_ptr()));
        break;
      }
      case 'z':
        if (o == Py_None) {
          word(0);
          break;
        }
        [[fallthrough]];
      case 'Z':
      case 'P': {
        const at::Tensor* t = tensor(o, *s != 'P');
        if (!t) return false;
        word(address(t->data_ptr()));
        break;
      }
      case 'R': {
        const at::Tensor* t = tensor(o);
        PyObject* cap = *a++;
        if (!t) return false;
        if (cap == Py_None) v = static_cast<uint64_t>(t->numel() * t->element_size());
        else if (!integer(cap, &v)) return false;
        word(address(t->data_ptr()));
        word(v);
        break;
      }
      case 'N':
        if (!integer(o, &elems) || elems >> 63) return false;
        word(elems);
        break;
      case 'I':
        if (!integer(o, &v)) return false;
        word(v);
        break;
      case 'D':
        if (!integer(o, &v)) return false;
        expected = bytes_per_word(v);
        word(v);
        break;
      case 'A':
      case 'G':
      case 'K': {
        const void* p = *s == 'A' ? views.of(o, nullptr, 1)
                        : *s == 'G' ? views.of(o, b.types.paged, sizeof(splitzip_paged)) : views.of(o, b.types.codebook, sizeof(splitzip_codebook));
        if (!p) return false;
        word(address(p));
        break;
      }
      case 'C': {
        const void* cb = views.of(o, b.types.codebook, sizeof(splitzip_codebook));
        if (!cb) return false;
        const uint32_t dtype = static_cast<const splitzip_codebook*>(cb)->dtype;
        expected = bytes_per_word(dtype);
        word(dtype);
        word(address(cb));
        break;
      }
      case 'V': {
        const void* f = views.of(o, b.types.variant, sizeof(splitzip_variant));
        if (!f) return false;
        expected = bytes_per_word(static_cast<const splitzip_variant*>(f)->dtype);
        word(address(f));
        break;
      }
      case 'S':
        if (o == Py_None) v = address(c10::hip::getCurrentHIPStream().stream());
        else if (!integer(o, &v)) return false;
        word(v);
        break;
    }
  }
  if (word_size && word_size != expected) return false;
  Py_BEGIN_ALLOW_THREADS
  *rc = b.entry->call(b.fn, w);
  Py_END_ALLOW_THREADS
  return true;
}

PyObject* fastcall(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  const Bound* b = static_cast<const Bound*>(PyCapsule_GetPointer(self, nullptr));
  if (!b) return nullptr;
  int rc = kNotTaken;
  try {
    if (!run(*b, a, n, &rc)) rc = kNotTaken;
  } catch (...) {   // what torch throws for a tensor without memory of its own, or without a GPU: the general way says what is wrong
    rc = kNotTaken;
    PyErr_Clear();
  }
  return PyLong_FromLong(rc);
}
PyMethodDef kFastcall = {"fastcall", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fastcall)), METH_FASTCALL, nullptr};

void forget(PyObject* capsule) {
  Bound* b = static_cast<Bound*>(PyCapsule_GetPointer(capsule, nullptr));
  Py_DECREF(b->types.codebook);
  Py_DECREF(b->types.variant);
  Py_DECREF(b->types.paged);
  delete b;
}

// bind(handle, codebook, variant, paged, torch): the entry points of the library that ctypes holds by this handle, name ->
// function, for the binding's structures of these types; an ImportError if the torch of this version is not the one that
// this was built for (torch's headers read the fields of its tensors)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject* handle = nullptr;
  Types types;
  const char* torch_version = nullptr;
  if (!PyArg_ParseTuple(args, "OOOOs", &handle, &types.codebook, &types.variant, &types.paged, &torch_version)) return nullptr;
  if (strcmp(torch_version, BUILT_FOR_TORCH) != 0) {
    PyErr_Format(PyExc_ImportError, "_fastcall was built for torch %s, this is %s", BUILT_FOR_TORCH, torch_version);
    return nullptr;
  }
  void* lib = PyLong_AsVoidPtr(handle);
  if (!lib && PyErr_Occurred()) return nullptr;
  PyObject* out = PyDict_New();
  if (!out) return nullptr;
  for (const Entry& e : kEntries) {
    void* fn = dlsym(lib, e.name);
    if (!fn) {
      PyErr_Format(PyExc_ImportError, "libsplitzip.so has no %s", e.name);
      Py_DECREF(out);
      return nullptr;
    }
    Bound* b = new Bound{fn, &e, types};
    PyObject* capsule = PyCapsule_New(b, nullptr, nullptr);
    if (capsule) {
      Py_INCREF(types.codebook);
      Py_INCREF(types.variant);
      Py_INCREF(types.paged);
      PyCapsule_SetDestructor(capsule, forget);
    } else {
      delete b;
    }
    PyObject* f = capsule ? PyCFunction_NewEx(&kFastcall, capsule, nullptr) : nullptr;
    Py_XDECREF(capsule);
    const int failed = f ? PyDict_SetItemString(out, e.name, f) : -1;
    Py_XDECREF(f);
    if (failed) {
      Py_DECREF(out);
      return nullptr;
    }
  }
  return out;
}

PyMethodDef kMethods[] = {{"bind", bind, METH_VARARGS, "bind(handle, codebook, variant, paged, torch): {name: function} for a libsplitzip.so that is loaded"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&kModule); }
