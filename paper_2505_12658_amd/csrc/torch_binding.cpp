// Python binding of include/hydra_attn.h for torch tensors: checks, data pointers, strides and the
// current stream, then one call through the C ABI.  Every step of the computation runs in the HIP kernels.
//
// The marshalling is native because a decode step or a single image is over in tens of microseconds: written
// in Python with ctypes, the same work took 8 (cache copies) to 12 us (attention) of host time per call, more
// than the kernels it launched, so small batches ran at the host's pace.
//
// The module is told where the library is (load) instead of linking to it, so that a missing library is an
// ImportError of the caller's and the library stays a plain C library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/hydra_attn.h"

namespace {

struct Library {
  decltype(&hydra_attn_workspace_bytes) attn_workspace_bytes = nullptr;
  decltype(&hydra_attn_varlen_fwd) attn_varlen_fwd = nullptr;
  decltype(&hydra_attn_varlen_fwd_static) attn_varlen_fwd_static = nullptr;
  decltype(&hydra_attn_build_worklist) attn_build_worklist = nullptr;
  decltype(&hydra_attn_varlen_fwd_prebuilt) attn_varlen_fwd_prebuilt = nullptr;
  decltype(&hydra_attn_varlen_fwd_shared) attn_varlen_fwd_shared = nullptr;
  decltype(&hydra_kv_cache_write) kv_cache_write = nullptr;
  decltype(&hydra_attn_paged_fwd) attn_paged_fwd = nullptr;
  decltype(&hydra_attn_paged_workspace_bytes) attn_paged_workspace_bytes = nullptr;
  decltype(&hydra_page_cache_write) page_cache_write = nullptr;
  decltype(&hydra_page_cache_gather) page_cache_gather = nullptr;
};
Library lib;
PyObject* hydra_error = nullptr;  // the HydraError class: HydraError(status, where)

struct Raised {};  // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised{};
}
[[noreturn]] void raise(PyObject* type, const char* name, const char* text) {
  PyErr_Format(type, "%s%s", name, text);
  throw Raised{};
}

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, name, " must be a torch tensor");
  return THPVariable_Unpack(o);
}
// The C ABI's int32 of a Python number: modulo 2^32, so that an absurd bound is what the library refuses (or not).
// `convert`: how anything but an int becomes one.
template <PyObject* (*convert)(PyObject*)>
int32_t to_int32(PyObject* o) {
  if (PyLong_Check(o)) return (int32_t)PyLong_AsUnsignedLongMask(o);
  PyObject* n = convert(o);
  if (!n) throw Raised{};
  const int32_t v = (int32_t)PyLong_AsUnsignedLongMask(n);
  Py_DECREF(n);
  return v;
}
int32_t whole(PyObject* o) { return to_int32<PyNumber_Index>(o); }  // a whole number; no float, no text
int32_t as_int(PyObject* o) { return to_int32<PyNumber_Long>(o); }  // whatever int() takes
int32_t size32(int64_t v) {
  if (v != (int32_t)v) raise(PyExc_OverflowError, "size does not fit 32 bits");
  return (int32_t)v;
}
double real(PyObject* o) {  // whatever float() takes
  if (PyFloat_Check(o)) return PyFloat_AS_DOUBLE(o);
  PyObject* f = PyNumber_Float(o);
  if (!f) throw Raised{};
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}
int truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised{};
  return v;
}
// a torch stream object, or None for the current stream of the current device
void* stream_handle(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
  if (!h) throw Raised{};
  void* p = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (!p && PyErr_Occurred()) throw Raised{};
  return p;
}

bool is_bf16(const at::Tensor& t) { return t.scalar_type() == at::kBFloat16; }

const at::Tensor& token_major(PyObject* o, const char* name) {
  const at::Tensor& t = tensor(o, name);
  if (!is_bf16(t) || t.dim() != 3 || !t.is_cuda()) raise(PyExc_TypeError, name, " must be a CUDA bf16 tensor [tokens, heads, head_dim]");
  if (t.stride(2) != 1 || t.stride(1) != t.size(2)) raise(PyExc_ValueError, name, ": head_dim must be contiguous and the head stride must equal head_dim");
  return t;
}
const at::Tensor& index_array(PyObject* o, at::ScalarType type, const char* name) {
  const at::Tensor& t = tensor(o, name);
  if (t.scalar_type() != type || !t.is_cuda() || !t.is_contiguous())
    raise(PyExc_TypeError, name, type == at::kInt ? " must be a contiguous CUDA int32 tensor" : " must be a contiguous CUDA int64 tensor");
  return t;
}
void check_out(const at::Tensor& out, const at::Tensor& q) {
  if (!is_bf16(out) || !out.is_contiguous() || out.sizes() != q.sizes()) raise(PyExc_ValueError, "out must be a contiguous bf16 tensor shaped like q");
}
at::Tensor out_like(PyObject* o, const at::Tensor& q) {
  if (o == Py_None) return at::empty(q.sizes(), q.options().memory_format(c10::nullopt));
  const at::Tensor& out = tensor(o, "out");
  check_out(out, q);
  return out;
}
at::Tensor bytes_on(const at::Tensor& like, size_t bytes) { return at::empty({(int64_t)bytes}, like.options().dtype(at::kByte)); }

// Runs f (one call of the C ABI) without the interpreter lock and turns its status into an exception.
template <typename F>
void call(const char* where, F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = f();
  Py_END_ALLOW_THREADS;
  if (rc == HYDRA_OK) return;
  PyObject* e = PyObject_CallFunction(hydra_error, "is", rc, where);
  if (e) {
    PyErr_SetObject(hydra_error, e);
    Py_DECREF(e);
  }
  throw Raised{};
}

// Runs one entry point; C++ and Python errors become the interpreter's.
template <typename F>
PyObject* guarded(const char* name, Py_ssize_t given, Py_ssize_t wanted, F&& f) {
  if (given != wanted) {
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments (%zd given)", name, wanted, given);
    return nullptr;
  }
  if (!lib.attn_varlen_fwd) {
    PyErr_SetString(PyExc_ImportError, "the library is not loaded");
    return nullptr;
  }
  try {
    return f();
  } catch (const Raised&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// The tensors and sizes that the packed attention calls have in common.
struct Packed {
  const at::Tensor &q, &k, &v, &cu;
  int32_t batch, tokens, longest, n_q, n_kv, d;
  int causal;
  float scale;
  // to_int: the conversion of max_seqlen
  Packed(PyObject* const* a, bool check_cu, int32_t (*to_int)(PyObject*) = as_int)
      : q(token_major(a[0], "q")), k(token_major(a[1], "k")), v(token_major(a[2], "v")),
        cu(check_cu ? index_array(a[3], at::kInt, "cu_seqlens") : tensor(a[3], "cu_seqlens")),
        batch(size32(cu.numel() - 1)), tokens(size32(q.size(0))), longest(to_int(a[4])), n_q(size32(q.size(1))),
        n_kv(size32(k.size(1))), d(size32(q.size(2))), causal(truth(a[5])), scale((float)real(a[6])) {}
};

PyObject* py_attn_varlen_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("attn_varlen_fwd", n, 10, [&] {
    const Packed p(a, true, whole);
    const at::Tensor out = out_like(a[7], p.q);
    const at::Tensor ws = a[8] == Py_None
                              ? bytes_on(p.q, std::max<size_t>(lib.attn_workspace_bytes(p.batch, p.tokens, p.longest, p.n_q, p.n_kv, p.d), 16))
                              : tensor(a[8], "workspace");
    void* s = stream_handle(a[9]);
    call("hydra_attn_varlen_fwd", [&] {
      return lib.attn_varlen_fwd(p.q.data_ptr(), p.k.data_ptr(), p.v.data_ptr(), out.data_ptr(), p.q.stride(0), p.k.stride(0), p.v.stride(0),
                                 p.cu.const_data_ptr<int32_t>(), p.batch, p.tokens, p.longest, p.n_q, p.n_kv, p.d, p.causal, p.scale,
                                 ws.data_ptr(), ws.nbytes(), s);
    });
    return THPVariable_Wrap(out);
  });
}

PyObject* py_attn_varlen_fwd_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("attn_varlen_fwd_static", n, 9, [&] {
    const Packed p(a, true);
    const at::Tensor& out = tensor(a[7], "out");
    check_out(out, p.q);
    void* s = stream_handle(a[8]);
    call("hydra_attn_varlen_fwd_static", [&] {
      return lib.attn_varlen_fwd_static(p.q.data_ptr(), p.k.data_ptr(), p.v.data_ptr(), out.data_ptr(), p.q.stride(0), p.k.stride(0),
                                        p.v.stride(0), p.cu.const_data_ptr<int32_t>(), p.batch, p.tokens, p.longest, p.n_q, p.n_kv, p.d,
                                        p.causal, p.scale, s);
    });
    return Py_NewRef(a[7]);
  });
}

PyObject* py_attn_build_worklist(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("attn_build_worklist", n, 9, [&] {
    const at::Tensor& cu = index_array(a[0], at::kInt, "cu_seqlens");
    const auto size = a[7] == Py_None ? whole : as_int;
    const int32_t batch = size32(cu.numel() - 1), tokens = size(a[1]), longest = size(a[2]), n_q = whole(a[3]), n_kv = whole(a[4]), d = whole(a[5]);
    const int causal = truth(a[6]);
    const at::Tensor ws = a[7] == Py_None ? bytes_on(cu, std::max<size_t>(lib.attn_workspace_bytes(batch, tokens, longest, n_q, n_kv, d), 16))
                                          : tensor(a[7], "workspace");
    void* s = stream_handle(a[8]);
    call("hydra_attn_build_worklist", [&] {
      return lib.attn_build_worklist(cu.const_data_ptr<int32_t>(), batch, tokens, longest, n_q, n_kv, d, causal, ws.data_ptr(), ws.nbytes(), s);
    });
    return THPVariable_Wrap(ws);
  });
}

// (workgroups_per_cu None: hydra_attn_varlen_fwd_prebuilt, otherwise hydra_attn_varlen_fwd_shared)
PyObject* py_attn_varlen_fwd_prebuilt(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("attn_varlen_fwd_prebuilt", n, 11, [&] {
    const Packed p(a, false);
    const at::Tensor &out = tensor(a[7], "out"), &ws = tensor(a[8], "workspace");
    check_out(out, p.q);
    void* s = stream_handle(a[10]);
    const auto cu = static_cast<const int32_t*>(p.cu.data_ptr());
    if (a[9] == Py_None) {
      call("hydra_attn_varlen_fwd_prebuilt", [&] {
        return lib.attn_varlen_fwd_prebuilt(p.q.data_ptr(), p.k.data_ptr(), p.v.data_ptr(), out.data_ptr(), p.q.stride(0), p.k.stride(0),
                                            p.v.stride(0), cu, p.batch, p.tokens, p.longest, p.n_q, p.n_kv, p.d, p.causal, p.scale, ws.data_ptr(),
                                            ws.nbytes(), s);
      });
    } else {
      const int32_t per_cu = as_int(a[9]);
      call("hydra_attn_varlen_fwd_shared", [&] {
        return lib.attn_varlen_fwd_shared(p.q.data_ptr(), p.k.data_ptr(), p.v.data_ptr(), out.data_ptr(), p.q.stride(0), p.k.stride(0),
                                          p.v.stride(0), cu, p.batch, p.tokens, p.longest, p.n_q, p.n_kv, p.d, p.causal, p.scale, ws.data_ptr(),
                                          ws.nbytes(), per_cu, s);
      });
    }
    return Py_NewRef(a[7]);
  });
}

void check_caches(const at::Tensor& kc, const at::Tensor& vc) {
  if (kc.dim() != 4 || !kc.is_contiguous() || !vc.is_contiguous() || kc.sizes() != vc.sizes())
    raise(PyExc_ValueError, "caches must be contiguous [num_blocks, block_size, n_kv_heads, head_dim] of equal shape");
  if (!is_bf16(kc) || !is_bf16(vc) || !kc.is_cuda()) raise(PyExc_TypeError, "caches must be CUDA bf16 tensors");
}

PyObject* py_kv_cache_write(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("kv_cache_write", n, 6, [&] {
    const at::Tensor &k = token_major(a[0], "k"), &v = token_major(a[1], "v");
    const at::Tensor &kc = tensor(a[2], "k_cache"), &vc = tensor(a[3], "v_cache");
    check_caches(kc, vc);
    const at::Tensor& slots = index_array(a[4], at::kLong, "slot_mapping");
    if (slots.numel() != k.size(0) || kc.size(2) != k.size(1) || kc.size(3) != k.size(2) || v.sizes() != k.sizes())
      raise(PyExc_ValueError, "shape mismatch between k/v, caches and slot_mapping");
    const int32_t tokens = size32(k.size(0)), n_kv = size32(k.size(1)), d = size32(k.size(2)), block = size32(kc.size(1));
    void* s = stream_handle(a[5]);
    call("hydra_kv_cache_write", [&] {
      return lib.kv_cache_write(k.data_ptr(), v.data_ptr(), k.stride(0), v.stride(0), kc.data_ptr(), vc.data_ptr(), slots.const_data_ptr<int64_t>(),
                                tokens, n_kv, d, block, kc.size(0), s);
    });
    return Py_NewRef(Py_None);
  });
}

PyObject* py_attn_paged_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("attn_paged_fwd", n, 12, [&] {
    const at::Tensor& q = token_major(a[0], "q");
    const at::Tensor &kc = tensor(a[1], "k_cache"), &vc = tensor(a[2], "v_cache");
    check_caches(kc, vc);
    const at::Tensor &table = index_array(a[3], at::kInt, "block_tables"), &cu = index_array(a[4], at::kInt, "cu_seqlens_q"),
                     &kv_lens = index_array(a[5], at::kInt, "kv_lens");
    const int64_t batch64 = cu.numel() - 1;
    if (table.dim() != 2 || table.size(0) != batch64 || kv_lens.numel() != batch64 || kc.size(3) != q.size(2))
      raise(PyExc_ValueError, "shape mismatch between q, caches, block_tables, cu_seqlens_q and kv_lens");
    const int32_t batch = size32(batch64), tokens = size32(q.size(0)), longest = as_int(a[6]), n_q = size32(q.size(1)), n_kv = size32(kc.size(2)),
                  d = size32(q.size(2)), block = size32(kc.size(1)), width = size32(table.size(1));
    const float scale = (float)real(a[7]);
    const at::Tensor out = out_like(a[8], q);
    at::Tensor ws;
    if (a[9] != Py_None) {
      ws = tensor(a[9], "workspace");
    } else if (truth(a[10])) {
      const size_t need = lib.attn_paged_workspace_bytes(batch, n_kv, d, width, block);
      if (need) ws = bytes_on(q, need);
    }
    void* s = stream_handle(a[11]);
    call("hydra_attn_paged_fwd", [&] {
      return lib.attn_paged_fwd(q.data_ptr(), out.data_ptr(), q.stride(0), kc.data_ptr(), vc.data_ptr(), table.const_data_ptr<int32_t>(), width,
                                cu.const_data_ptr<int32_t>(), kv_lens.const_data_ptr<int32_t>(), batch, tokens, longest, n_q, n_kv, d, block,
                                kc.size(0), scale, ws.defined() ? ws.data_ptr() : nullptr, ws.defined() ? ws.nbytes() : 0, s);
    });
    return THPVariable_Wrap(out);
  });
}

// rows, cache, slot_mapping of the two image-cache calls
void check_page_cache(const at::Tensor& rows, const at::Tensor& cache, const at::Tensor& slots) {
  if (!is_bf16(rows) || rows.dim() != 2 || !rows.is_cuda() || rows.stride(1) != 1) raise(PyExc_TypeError, "rows must be a CUDA bf16 matrix with contiguous rows");
  if (!is_bf16(cache) || !cache.is_cuda() || !cache.is_contiguous() || cache.dim() < 1 || cache.size(-1) != rows.size(1))
    raise(PyExc_TypeError, "cache must be a contiguous CUDA bf16 tensor [..., row_elems]");
  if (slots.scalar_type() != at::kLong || !slots.is_cuda() || !slots.is_contiguous() || slots.numel() != rows.size(0))
    raise(PyExc_TypeError, "slot_mapping must be a contiguous CUDA int64 tensor with one entry per row");
}
PyObject* py_page_cache_write(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("page_cache_write", n, 4, [&] {
    const at::Tensor &rows = tensor(a[0], "rows"), &cache = tensor(a[1], "cache"), &slots = tensor(a[2], "slot_mapping");
    check_page_cache(rows, cache, slots);
    const int32_t n_rows = size32(rows.size(0)), row = size32(rows.size(1));
    const int64_t num = row ? cache.numel() / row : 0;
    void* s = stream_handle(a[3]);
    call("hydra_page_cache_write", [&] {
      return lib.page_cache_write(rows.data_ptr(), rows.stride(0), cache.data_ptr(), slots.const_data_ptr<int64_t>(), n_rows, row, num, s);
    });
    return Py_NewRef(Py_None);
  });
}
PyObject* py_page_cache_gather(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded("page_cache_gather", n, 4, [&] {
    const at::Tensor &cache = tensor(a[0], "cache"), &slots = tensor(a[1], "slot_mapping"), &rows = tensor(a[2], "rows");
    check_page_cache(rows, cache, slots);
    const int32_t n_rows = size32(rows.size(0)), row = size32(rows.size(1));
    const int64_t num = row ? cache.numel() / row : 0;
    void* s = stream_handle(a[3]);
    call("hydra_page_cache_gather", [&] {
      return lib.page_cache_gather(cache.data_ptr(), slots.const_data_ptr<int64_t>(), rows.data_ptr(), rows.stride(0), n_rows, row, num, s);
    });
    return Py_NewRef(Py_None);
  });
}

// load(path, HydraError): opens the library and looks its entry points up
PyObject* py_load(PyObject*, PyObject* args) {
  const char* path;
  PyObject* error;
  if (!PyArg_ParseTuple(args, "sO", &path, &error)) return nullptr;
  void* h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
  if (!h) {
    PyErr_SetString(PyExc_ImportError, dlerror());
    return nullptr;
  }
  Library l;
  bool all = true;
  auto find = [&](auto& fn, const char* name) {
    fn = reinterpret_cast<std::decay_t<decltype(fn)>>(dlsym(h, name));
    all = all && fn;
  };
  find(l.attn_workspace_bytes, "hydra_attn_workspace_bytes");
  find(l.attn_varlen_fwd, "hydra_attn_varlen_fwd");
  find(l.attn_varlen_fwd_static, "hydra_attn_varlen_fwd_static");
  find(l.attn_build_worklist, "hydra_attn_build_worklist");
  find(l.attn_varlen_fwd_prebuilt, "hydra_attn_varlen_fwd_prebuilt");
  find(l.attn_varlen_fwd_shared, "hydra_attn_varlen_fwd_shared");
  find(l.kv_cache_write, "hydra_kv_cache_write");
  find(l.attn_paged_fwd, "hydra_attn_paged_fwd");
  find(l.attn_paged_workspace_bytes, "hydra_attn_paged_workspace_bytes");
  find(l.page_cache_write, "hydra_page_cache_write");
  find(l.page_cache_gather, "hydra_page_cache_gather");
  if (!all) {
    PyErr_Format(PyExc_ImportError, "%s lacks an entry point of hydra_attn.h", path);
    return nullptr;
  }
  lib = l;
  Py_INCREF(error);
  Py_XDECREF(hydra_error);
  hydra_error = error;
  Py_RETURN_NONE;
}

#define HYDRA_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"load", py_load, METH_VARARGS, nullptr},
                         HYDRA_FAST(attn_varlen_fwd),
                         HYDRA_FAST(attn_varlen_fwd_static),
                         HYDRA_FAST(attn_build_worklist),
                         HYDRA_FAST(attn_varlen_fwd_prebuilt),
                         HYDRA_FAST(kv_cache_write),
                         HYDRA_FAST(attn_paged_fwd),
                         HYDRA_FAST(page_cache_write),
                         HYDRA_FAST(page_cache_gather),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hydra_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hydra_torch() { return PyModule_Create(&module); }
