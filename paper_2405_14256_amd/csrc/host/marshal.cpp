// Argument marshalling of the Python binding in native code: tensors to zc_tensor4, the
// current HIP stream, a scratch buffer of the stream, and the call itself.  Nothing of the
// method happens here, and nothing about a call's tensors is kept.
//
// Why: a decode step at batch 1 is 9 us of GPU work, and describing its tensors through ctypes
// (attribute by attribute, a structure each) took 19 us of the caller's thread; here a tensor
// costs one look at its C++ object.  Steps of one 4096-token prompt issued one after the other:
// 18.5 -> 9.2 us each (the GPU's own time); six launches of a flush at batch 8: 47 -> 34 us.
//
// The library's entry points come in as addresses (bind), so that whichever build of the library
// the binding has loaded is the one that is called.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <map>
#include <tuple>
#include <vector>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "zipcache.h"

namespace {

// ---- entry points, in the order of kNames ---------------------------------------------------
enum Fn {
  kProbe, kAccumulated, kPrefill, kSelect, kQuantize, kQuantizeKV, kDecode, kDecodeStatic, kProbs, kRows, kDequantize,
  kProbeWs, kQuantizeWs, kQuantizeKVWs, kDecodeWs, kFnCount
};
const char* const kNames[kFnCount] = {
    "zc_probe_saliency", "zc_probe_accumulated", "zc_prefill_attention", "zc_select_salient", "zc_quantize_pack",
    "zc_quantize_pack_kv", "zc_decode_attention", "zc_decode_attention_static", "zc_decode_probs", "zc_rows_saliency",
    "zc_dequantize_cache", "zc_probe_saliency_workspace", "zc_quantize_pack_workspace", "zc_quantize_pack_kv_workspace",
    "zc_decode_attention_workspace"};
void* g_fn[kFnCount];

#define ZC_FN(id, name) reinterpret_cast<decltype(&name)>(g_fn[id])

// ---- arguments ---------------------------------------------------------------------------------
struct Bad {};   // a Python exception has been set

const at::Tensor& tensor_of(PyObject* o) {
  if (!THPVariable_Check(o)) { PyErr_Format(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name); throw Bad(); }
  return THPVariable_Unpack(o);
}
void* ptr_of(PyObject* o) { return o == Py_None ? nullptr : tensor_of(o).data_ptr(); }
template <class T> T* ptr_as(PyObject* o) { return static_cast<T*>(ptr_of(o)); }

int64_t int_of(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Bad();
  return v;
}
float float_of(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Bad();
  return (float)v;
}

// A [B, H, L, D] tensor with unit stride on D; `row`: a [B, H, D] one stands for L = 1 too.
zc_tensor4 describe(PyObject* o, bool row = false) {
  const at::Tensor& t = tensor_of(o);
  const auto sz = t.sizes();
  const auto st = t.strides();
  const bool three = row && sz.size() == 3;
  if ((sz.size() != 4 && !three) || st.back() != 1) {
    PyErr_SetString(PyExc_AssertionError, "need a 4-D tensor with contiguous last axis");
    throw Bad();
  }
  zc_tensor4 r;
  r.ptr = t.data_ptr();
  switch (t.scalar_type()) {
    case at::kFloat: r.dtype = ZC_F32; break;
    case at::kHalf: r.dtype = ZC_F16; break;
    case at::kBFloat16: r.dtype = ZC_BF16; break;
    default: PyErr_Format(PyExc_KeyError, "%s", c10::toString(t.scalar_type())); throw Bad();
  }
  r.reserved = 0;
  r.B = sz[0]; r.H = sz[1]; r.sB = st[0]; r.sH = st[1];
  r.L = three ? 1 : sz[2];
  r.D = sz[three ? 2 : 3];
  r.sL = three ? r.D : st[2];
  return r;
}

// The zc_packed behind a ctypes structure, for the duration of a call.
struct Packed {
  Py_buffer view;
  explicit Packed(PyObject* o) {
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Bad();
    if (view.len != (Py_ssize_t)sizeof(zc_packed)) {
      PyBuffer_Release(&view);
      PyErr_SetString(PyExc_TypeError, "expected a zc_packed structure");
      throw Bad();
    }
  }
  Packed(const Packed&) = delete;
  ~Packed() { PyBuffer_Release(&view); }
  zc_packed* get() const { return static_cast<zc_packed*>(view.buf); }
};

// ---- scratch ---------------------------------------------------------------------------------
// One buffer per device, kind of call and stream (calls on different streams may run
// concurrently and must not share scratch memory), used by every call of that kind on that
// stream, in stream order.  A buffer is replaced by one at least half as large again and goes
// back to torch's allocator, which reuses it in the order of the stream - unless a call that used
// it was captured: the graph holds its address, and it is kept.  (So a stream holds less than one and a
// half times its largest request, and what its graphs were captured with.)  All of this runs
// under the interpreter lock.
enum Kind { kScratchProbe, kScratchQuantize, kScratchQuantizeKV, kScratchDecode };
struct Scratch { at::Tensor t; void* ptr = nullptr; size_t bytes = 0; bool captured = false; };
std::map<std::tuple<int, int, void*>, Scratch>* g_scratch;
std::vector<at::Tensor>* g_captured;      // replaced buffers that graphs may hold

// The reference keeps the buffer during the call, whose launch runs without the lock.
Scratch scratch(size_t need, const at::Tensor& like, Kind kind, hipStream_t stream) {
  Scratch& s = (*g_scratch)[std::make_tuple((int)like.device().index(), (int)kind, (void*)stream)];
  if (!s.ptr || s.bytes < need) {
    size_t n = need < 256 ? 256 : need;
    if (s.ptr && n < s.bytes + s.bytes / 2) n = s.bytes + s.bytes / 2;
    at::Tensor t = at::zeros({(int64_t)n}, like.options().dtype(at::kByte));
    if (s.captured) g_captured->push_back(s.t);
    s.ptr = t.data_ptr();
    s.t = std::move(t);
    s.bytes = n;
    s.captured = false;
  }
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
    (void)hipGetLastError();
    s.captured = true;                     // (the default stream beside a capture: taken for one)
  }
  s.captured |= status != hipStreamCaptureStatusNone;
  return s;
}

hipStream_t current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs a launch without the interpreter lock (it may wait for room in the stream's queue).
template <class F> int unlocked(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}

// Every function below returns the library's status as an int.
template <class F> PyObject* guarded(Fn id, Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) return PyErr_Format(PyExc_TypeError, "%s: %zd arguments, expected %zd", kNames[id], n, want);
  if (!g_fn[id]) return PyErr_Format(PyExc_RuntimeError, "%s is not bound", kNames[id]);
  try {
    return PyLong_FromLong(f());
  } catch (const Bad&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

typedef PyObject* const* Args;

// (accumulated, q, k, probe_rows, probe_pos, sm_scale, lse_ext, scores, scores_per_head)
PyObject* probe(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kProbe, n, 9, [&]() -> int {
    const bool acc = PyObject_IsTrue(a[0]) != 0;
    const zc_tensor4 q = describe(a[1]), k = describe(a[2]);
    const auto* rows = ptr_as<const int32_t>(a[3]);
    const at::Tensor& pos = tensor_of(a[4]);
    const auto* posp = static_cast<const int32_t*>(pos.data_ptr());
    const int32_t P = (int32_t)pos.numel();
    const float scale = float_of(a[5]);
    const auto* lse = ptr_as<const float>(a[6]);
    auto* scores = ptr_as<float>(a[7]);
    auto* per_head = ptr_as<float>(a[8]);
    const hipStream_t st = current_stream();
    const Scratch ws = scratch(ZC_FN(kProbeWs, zc_probe_saliency_workspace)(q.B, q.H, k.L, P), tensor_of(a[1]), kScratchProbe, st);
    void* wp = ws.ptr;
    const size_t wn = ws.bytes;
    const auto fn = ZC_FN(acc ? kAccumulated : kProbe, zc_probe_saliency);
    return unlocked([&] { return fn(&q, &k, rows, posp, P, scale, lse, scores, per_head, wp, wn, st); });
  });
}

// (q, k, v, sm_scale, out, lse, probe_pos, lse_probe)
PyObject* prefill(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kPrefill, n, 8, [&]() -> int {
    const zc_tensor4 q = describe(a[0]), k = describe(a[1]), v = describe(a[2]), o = describe(a[4]);
    const float scale = float_of(a[3]);
    auto* lse = ptr_as<float>(a[5]);
    const int32_t P = a[6] == Py_None ? 0 : (int32_t)tensor_of(a[6]).numel();
    const auto* pos = P ? ptr_as<const int32_t>(a[6]) : nullptr;
    auto* lse_probe = P ? ptr_as<float>(a[7]) : nullptr;
    const hipStream_t st = current_stream();
    const auto fn = ZC_FN(kPrefill, zc_prefill_attention);
    return unlocked([&] { return fn(&q, &k, &v, scale, &o, lse, pos, P, lse_probe, st); });
  });
}

// (scores, k, salient_idx, regular_idx, mask)
PyObject* select(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kSelect, n, 5, [&]() -> int {
    const at::Tensor& s = tensor_of(a[0]);
    if (s.dim() != 2) { PyErr_Format(PyExc_ValueError, "scores must be [B, L], got %d dimensions", (int)s.dim()); throw Bad(); }
    const int64_t B = s.size(0), L = s.size(1), k = int_of(a[1]);
    const auto* sp = static_cast<const float*>(s.data_ptr());
    auto *sal = ptr_as<int32_t>(a[2]), *reg = ptr_as<int32_t>(a[3]);
    auto* mask = ptr_as<uint8_t>(a[4]);
    const hipStream_t st = current_stream();
    const auto fn = ZC_FN(kSelect, zc_select_salient);
    return unlocked([&] { return fn(sp, B, L, k, sal, reg, mask, nullptr, 0, st); });
  });
}

struct Lists { int64_t k, n_reg; const int32_t *sal, *reg; };
Lists lists_of(PyObject* sal, PyObject* reg) {
  Lists l;
  l.k = sal == Py_None ? 0 : tensor_of(sal).size(1);
  l.n_reg = reg == Py_None ? 0 : tensor_of(reg).size(1);
  l.sal = l.k ? ptr_as<const int32_t>(sal) : nullptr;
  l.reg = l.n_reg ? ptr_as<const int32_t>(reg) : nullptr;
  return l;
}

// (x, salient_idx, regular_idx, packed, pos_offset)
PyObject* quantize(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kQuantize, n, 5, [&]() -> int {
    const zc_tensor4 x = describe(a[0]);
    const Lists l = lists_of(a[1], a[2]);
    const Packed p(a[3]);
    const int64_t off = int_of(a[4]);
    const hipStream_t st = current_stream();
    const Scratch ws = scratch(ZC_FN(kQuantizeWs, zc_quantize_pack_workspace)(x.B, x.H, l.k + l.n_reg, x.D), tensor_of(a[0]),
                                kScratchQuantize, st);
    void* wp = ws.ptr;
    const size_t wn = ws.bytes;
    const auto fn = ZC_FN(kQuantize, zc_quantize_pack);
    return unlocked([&] { return fn(&x, l.sal, l.k, l.reg, l.n_reg, off, p.get(), wp, wn, st); });
  });
}

// (xk, xv, salient_idx, regular_idx, packedK, packedV, pos_offset)
PyObject* quantize_kv(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kQuantizeKV, n, 7, [&]() -> int {
    const zc_tensor4 xk = describe(a[0]), xv = describe(a[1]);
    const Lists l = lists_of(a[2], a[3]);
    const Packed pk(a[4]), pv(a[5]);
    const int64_t off = int_of(a[6]);
    const hipStream_t st = current_stream();
    const Scratch ws = scratch(ZC_FN(kQuantizeKVWs, zc_quantize_pack_kv_workspace)(xk.B, xk.H, l.k + l.n_reg, xk.D),
                                tensor_of(a[0]), kScratchQuantizeKV, st);
    void* wp = ws.ptr;
    const size_t wn = ws.bytes;
    const auto fn = ZC_FN(kQuantizeKV, zc_quantize_pack_kv);
    return unlocked([&] { return fn(&xk, &xv, l.sal, l.k, l.reg, l.n_reg, off, pk.get(), pv.get(), wp, wn, st); });
  });
}

// (use_static, q, packedK, packedV, tail_k, tail_v, tail_len, sm_scale, out, lse_out)
PyObject* decode(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kDecode, n, 10, [&]() -> int {
    const bool use_static = PyObject_IsTrue(a[0]) != 0;
    const zc_tensor4 q = describe(a[1], true);
    const Packed pk(a[2]), pv(a[3]);
    const int64_t T = int_of(a[6]);
    zc_tensor4 tk, tv;
    if (T) { tk = describe(a[4]); tv = describe(a[5]); }
    const zc_tensor4 *tkp = T ? &tk : nullptr, *tvp = T ? &tv : nullptr;
    const float scale = float_of(a[7]);
    void* out = tensor_of(a[8]).data_ptr();
    auto* lse = ptr_as<float>(a[9]);
    const hipStream_t st = current_stream();
    if (use_static) {
      const auto fn = ZC_FN(kDecodeStatic, zc_decode_attention_static);
      return unlocked([&] { return fn(&q, pk.get(), pv.get(), tkp, tvp, T, scale, out, lse, st); });
    }
    const Scratch ws = scratch(ZC_FN(kDecodeWs, zc_decode_attention_workspace)(q.B, q.H, q.D), tensor_of(a[1]), kScratchDecode, st);
    void* wp = ws.ptr;
    const size_t wn = ws.bytes;
    const auto fn = ZC_FN(kDecode, zc_decode_attention);
    return unlocked([&] { return fn(&q, pk.get(), pv.get(), tkp, tvp, T, scale, out, lse, wp, wn, st); });
  });
}

// (q, packedK, tail_k, tail_len, tail_pos0, lse, probs_out, sm_scale)
PyObject* probs(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kProbs, n, 8, [&]() -> int {
    const at::Tensor& out = tensor_of(a[6]);
    if (out.dim() != 3 || !out.is_contiguous() || out.scalar_type() != at::kFloat) {
      PyErr_SetString(PyExc_AssertionError, "probs_out must be a contiguous float32 [B, Hq, N] tensor");
      throw Bad();
    }
    const zc_tensor4 q = describe(a[0], true);
    const Packed pk(a[1]);
    const int64_t T = int_of(a[3]), pos0 = int_of(a[4]);
    zc_tensor4 tk;
    if (T) tk = describe(a[2]);
    const zc_tensor4* tkp = T ? &tk : nullptr;
    const auto* lse = static_cast<const float*>(tensor_of(a[5]).data_ptr());
    auto* po = static_cast<float*>(out.data_ptr());
    const int64_t N = out.size(2);
    const float scale = float_of(a[7]);
    const hipStream_t st = current_stream();
    const auto fn = ZC_FN(kProbs, zc_decode_probs);
    return unlocked([&] { return fn(&q, pk.get(), tkp, T, pos0, scale, lse, po, N, st); });
  });
}

// (rows, row_len, n_out, normalize, scores)
PyObject* rows_saliency(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kRows, n, 5, [&]() -> int {
    const at::Tensor &rows = tensor_of(a[0]), &len = tensor_of(a[1]);
    if (rows.dim() != 4 || !rows.is_contiguous() || rows.scalar_type() != at::kFloat || len.scalar_type() != at::kInt) {
      PyErr_SetString(PyExc_AssertionError, "rows must be contiguous float32 [P, B, Hq, N], row_len int32");
      throw Bad();
    }
    const auto* rp = static_cast<const float*>(rows.data_ptr());
    const auto* lp = static_cast<const int32_t*>(len.data_ptr());
    const int32_t P = (int32_t)rows.size(0);
    const int64_t B = rows.size(1), H = rows.size(2), N = rows.size(3), n_out = int_of(a[2]);
    const int normalize = PyObject_IsTrue(a[3]) != 0;
    auto* sp = static_cast<float*>(tensor_of(a[4]).data_ptr());
    const hipStream_t st = current_stream();
    const auto fn = ZC_FN(kRows, zc_rows_saliency);
    return unlocked([&] { return fn(rp, lp, P, B, H, N, n_out, normalize, sp, st); });
  });
}

// (packed, out)
PyObject* dequantize(PyObject*, Args a, Py_ssize_t n) {
  return guarded(kDequantize, n, 2, [&]() -> int {
    const Packed p(a[0]);
    const zc_tensor4 o = describe(a[1]);
    const hipStream_t st = current_stream();
    const auto fn = ZC_FN(kDequantize, zc_dequantize_cache);
    return unlocked([&] { return fn(p.get(), &o, st); });
  });
}

// names(): the entry points bind() wants; bind(addresses): their addresses, in that order
PyObject* names(PyObject*, PyObject*) {
  PyObject* t = PyTuple_New(kFnCount);
  for (int i = 0; t && i < kFnCount; ++i) PyTuple_SET_ITEM(t, i, PyUnicode_FromString(kNames[i]));
  return t;
}
PyObject* bind(PyObject*, PyObject* seq) {
  if (!PyTuple_Check(seq) || PyTuple_GET_SIZE(seq) != kFnCount) return PyErr_Format(PyExc_TypeError, "bind: a tuple of %d addresses", (int)kFnCount);
  void* got[kFnCount];
  for (int i = 0; i < kFnCount; ++i) {
    got[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(seq, i));
    if (!got[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "bind: %s has no address", kNames[i]);
  }
  for (int i = 0; i < kFnCount; ++i) g_fn[i] = got[i];
  Py_RETURN_NONE;
}

#define ZC_METHOD(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    {"names", names, METH_NOARGS, nullptr},
    {"bind", bind, METH_O, nullptr},
    ZC_METHOD("probe", probe),
    ZC_METHOD("prefill", prefill),
    ZC_METHOD("select", select),
    ZC_METHOD("quantize", quantize),
    ZC_METHOD("quantize_kv", quantize_kv),
    ZC_METHOD("decode", decode),
    ZC_METHOD("probs", probs),
    ZC_METHOD("rows_saliency", rows_saliency),
    ZC_METHOD("dequantize", dequantize),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_zc_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__zc_host() {
  g_scratch = new std::map<std::tuple<int, int, void*>, Scratch>();   // (neither is freed: tensors must not outlive the allocator at exit)
  g_captured = new std::vector<at::Tensor>();
  return PyModule_Create(&kModule);
}
