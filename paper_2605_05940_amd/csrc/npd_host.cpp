// The argument marshalling of binding.py in native code: the same checks on the same tensors, the same scratch memory and
// the same calls into libnpd (whose entry points arrive as addresses, see `bind`).
//
// Every function returns libnpd's status, or -1 if anything about its arguments is out of the ordinary -- a tensor that is
// not a plain one on the GPU, a type, shape or stride that the call does not take, a number that is not one: nothing has
// been enqueued then, and the caller's Python code, which is the reference for what is accepted, handles the call or raises.
//
// Why: a call of a few hundred positions keeps the GPU busy for 5 us, and reading fifteen tensors' attributes and filling
// the foreign-function call's arguments from Python took as long (MI355X, loss and two reductions, us a pass, marshalled
// from Python / here: 512 x 1,024 20.3 / 12.3, 64 x 151,936 24.8 / 21.1; the GPU alone needs 8.6 and 19.9).
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/zeros.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <vector>

#include "../../include/npd.h"

namespace {

struct Entry {
  decltype(&npd_workspace_bytes) workspace_bytes;
  decltype(&npd_workspace_bytes_preferred) workspace_bytes_preferred;
  decltype(&npd_forward_scratch_bytes) forward_scratch_bytes;
  decltype(&npd_kd_loss_fwd_bwd) kd;
  decltype(&npd_kd_loss_forward) kd_forward;
  decltype(&npd_segment_reduce) segment_reduce;
  decltype(&npd_delta_ifd_score) delta_ifd;
  decltype(&npd_teacher_topk) teacher_topk;
  decltype(&npd_policy_lag) policy_lag;
  decltype(&npd_kept_workspace_bytes) kept_bytes;  // null with a library that has no calls on kept records
  decltype(&npd_kd_loss_fwd_bwd_kept) kd_kept;
};
Entry lib;                            // written by bind() under the interpreter lock, before any call
PyObject* raw_stream = nullptr;       // torch's current raw stream of a device index
PyObject* workspaces = nullptr;       // the buffers it keeps, by device index

struct NotPlain {};                   // thrown by the helpers below: the caller's Python code takes the call

// the tensor behind an argument, nullptr for None
const at::Tensor* tensor(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_CheckExact(o)) throw NotPlain();
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided) throw NotPlain();
  return &t;
}
const at::Tensor& required(PyObject* o) {
  const at::Tensor* t = tensor(o);
  if (!t) throw NotPlain();
  return *t;
}
void* pointer(const at::Tensor* t, at::ScalarType type) {
  if (!t) return nullptr;
  if (t->scalar_type() != type) throw NotPlain();
  return t->data_ptr();
}
// contiguous array of n elements, nullptr if it is absent
void* array(PyObject* o, int64_t n, at::ScalarType type) {
  const at::Tensor* t = tensor(o);
  if (t && (t->numel() != n || !t->is_contiguous())) throw NotPlain();
  return pointer(t, type);
}
template <class T>
T* array_of(PyObject* o, int64_t n, at::ScalarType type) {
  return static_cast<T*>(array(o, n, type));
}
int64_t row_stride(const at::Tensor& t) {
  if (t.dim() != 2 || t.stride(1) != 1) throw NotPlain();
  return t.stride(0);
}
double number(PyObject* o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw NotPlain();
  return x;
}
long whole(PyObject* o) {
  if (!PyLong_Check(o)) throw NotPlain();
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  if (over || x != (long)(int32_t)x) throw NotPlain();
  return x;
}
bool flag(PyObject* o) {
  const int x = PyObject_IsTrue(o);
  if (x < 0) throw NotPlain();
  return x != 0;
}

c10::Device current_device() { return c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice(); }

void* current_stream() {
  PyObject* index = PyLong_FromLong(current_device().index());
  if (!index) throw NotPlain();
  PyObject* r = PyObject_CallOneArg(raw_stream, index);
  Py_DECREF(index);
  if (!r) throw NotPlain();
  void* s = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  if (!s && PyErr_Occurred()) throw NotPlain();
  return s;
}

// Memory for the kernels, whatever mode the caller has on: a tensor made under one may be a fake or a wrapped one without memory,
// and code of the mode would run here.  (No memory: its exception.)
at::Tensor memory(size_t bytes, bool zero) {
  const c10::impl::ForceDispatchKeyGuard plain(c10::DispatchKeySet(c10::DispatchKey::BackendSelect),
                                               c10::default_excluded_set | c10::autograd_dispatch_keyset_with_ADInplaceOrView);
  const auto options = at::TensorOptions().dtype(at::kByte).device(current_device());
  return zero ? at::zeros({(int64_t)bytes}, options) : at::empty({(int64_t)bytes}, options);
}

// scratch of one call: from torch's stream-ordered allocator, reused only behind the call on its stream (no memory: the
// exception leaves the call to the Python code, which knows what runs without)
at::Tensor scratch(size_t bytes) { return memory(bytes, false); }

// Records of the calls that clear none (npd_kd_loss_fwd_bwd_kept): one per device and stream, so that calls on different
// streams share none and a record goes back to the pool of the stream that it was used on.  Written under the interpreter
// lock, the one used last at the end.  At most kRecords of at most kRecordBytes: a call on another stream takes the place of the
// one that has been idle longest (a new record costs a launch that zeroes it, as much as clearing one for the call); calls that
// need more clear a block of their own.
struct Record {
  c10::DeviceIndex device;
  void* stream;
  at::Tensor bytes;
};
constexpr size_t kRecords = 8, kRecordTail = 512;  // (bytes behind the slices' words: 64 words)
constexpr size_t kRecordBytes = (32u << 20) + kRecordTail, kRecordLeast = (1u << 18) + kRecordTail;
// bytes of a record for a call that needs `bytes`: a power of two of words, so that batches that get longer by little do not make
// a new one each
size_t record_bytes(size_t bytes) {
  size_t n = kRecordLeast;
  while (n < bytes) n = 2 * (n - kRecordTail) + kRecordTail;
  return n;
}
std::vector<Record>& records() {
  static auto* all = new std::vector<Record>;  // (not destroyed behind the runtime's own end)
  return *all;
}
// the record of a stream, moved to the end; nullptr: it has none
Record* find_record(c10::DeviceIndex device, void* stream) {
  auto& all = records();
  for (auto x = all.begin(); x != all.end(); ++x) {
    if (x->device != device || x->stream != stream) continue;
    std::rotate(x, x + 1, all.end());
    return &all.back();
  }
  return nullptr;
}
// undefined: none to be had
at::Tensor record_of(size_t bytes, void* stream) {
  const c10::DeviceIndex device = current_device().index();
  const Record* have = find_record(device, stream);
  if (have && (size_t)have->bytes.numel() >= bytes) return have->bytes;
  if (bytes > kRecordBytes) return at::Tensor();
  at::Tensor t;
  try {
    t = memory(record_bytes(bytes), true);
  } catch (const std::exception&) {  // no memory: the call as before
    return at::Tensor();
  }
  auto& all = records();
  if (Record* r = find_record(device, stream)) {  // (looked up anew: an observer of the allocator may have let another thread run)
    r->bytes = t;
  } else {
    if (all.size() >= kRecords) all.erase(all.begin());
    all.push_back(Record{device, stream, t});
  }
  return t;
}
// bytes of the record that a call on `logits` runs on, 0: on none
size_t kept_bytes(const at::Tensor& logits, const npd_kd_desc& d, void* stream) {
  return lib.kept_bytes && logits.get_device() == current_device().index() ? lib.kept_bytes(&d, stream) : 0;
}
PyObject* release(PyObject*, PyObject*) {
  records().clear();
  Py_RETURN_NONE;
}

// A call into libnpd, without the interpreter lock: a launch may wait for room in its queue.
template <class F, class... A>
int call(F f, A... a) {
  PyThreadState* state = PyEval_SaveThread();
  const npd_status st = f(a...);
  PyEval_RestoreThread(state);
  return (int)st;
}

template <class Call>
PyObject* guarded(Call body) {
  try {
    return PyLong_FromLong((long)body());
  } catch (const NotPlain&) {
  } catch (const std::exception&) {  // torch's own: a tensor without memory of its own
  }
  PyErr_Clear();
  return PyLong_FromLong(-1);
}

// (student_logits, loss_mask, teacher_dense, teacher_idx, teacher_val, labels, tau, grad_scale, ce_grad_scale, divergence,
//  skew_alpha, grad_out, kd_tok, nll_tok, teacher_nll_tok, lse_tok, dev_status, workspace, no_workspace)
PyObject* kd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 19) return PyLong_FromLong(-1);
  return guarded([&]() -> int {
    const at::Tensor& s = required(a[0]);
    npd_kd_desc d{};
    d.student_stride = row_stride(s);
    const int64_t T = s.size(0), V = s.size(1);
    if (V > NPD_MAX_VOCAB) throw NotPlain();
    d.n_tokens = T;
    d.vocab = (int32_t)V;
    const at::Tensor *t = tensor(a[2]), *idx = nullptr, *val = nullptr;
    if (t) {
      d.teacher_kind = NPD_TEACHER_DENSE_BF16;
      d.teacher_stride = row_stride(*t);
      if (t->size(0) != T || t->size(1) != V) throw NotPlain();
      if (a[3] != Py_None || a[4] != Py_None) throw NotPlain();
    } else {
      idx = tensor(a[3]);
      val = tensor(a[4]);
      d.teacher_kind = idx ? NPD_TEACHER_TOPK : NPD_TEACHER_NONE;
      if (!idx != !val) throw NotPlain();
      if (idx) {
        if (idx->dim() != 2 || idx->size(0) != T || idx->size(1) > V || !idx->is_contiguous() || !val->is_contiguous() ||
            val->sizes() != idx->sizes())
          throw NotPlain();
        d.topk = (int32_t)idx->size(1);
      }
    }
    d.tau = (float)number(a[6]);
    d.grad_scale = (float)number(a[7]);
    d.ce_grad_scale = (float)number(a[8]);
    const double tau = number(a[6]), ce = number(a[8]);
    d.divergence = (int32_t)whole(a[9]);
    d.skew_alpha = (float)number(a[10]);
    const at::Tensor* g = tensor(a[11]);
    if (!g) {
      d.flags |= NPD_FLAG_FWD_ONLY;
    } else {
      if (row_stride(*g) != d.student_stride || g->size(0) != T || g->size(1) != V) throw NotPlain();
      if (g->data_ptr() == s.data_ptr()) d.flags |= NPD_FLAG_INPLACE_GRAD;
    }
    const bool no_workspace = flag(a[18]);
    if (no_workspace) d.flags |= NPD_FLAG_NO_WORKSPACE;
    const at::Tensor* ws = tensor(a[17]);
    void* const sp = pointer(&s, at::kBFloat16);
    void* const tp = pointer(t, at::kBFloat16);
    int32_t* const ip = static_cast<int32_t*>(pointer(idx, at::kInt));
    float* const vp = static_cast<float*>(pointer(val, at::kFloat));
    int32_t* const labels = array_of<int32_t>(a[5], T, at::kInt);
    uint8_t* const mask = static_cast<uint8_t*>(array(a[1], T, at::kByte));
    void* const gp = pointer(g, at::kBFloat16);
    float* const kd_tok = array_of<float>(a[12], T, at::kFloat);
    float* const nll = array_of<float>(a[13], T, at::kFloat);
    float* const tnll = array_of<float>(a[14], T, at::kFloat);
    float* const lse = array_of<float>(a[15], T, at::kFloat);
    int32_t* const status = static_cast<int32_t*>(pointer(tensor(a[16]), at::kInt));
    void* const stream = current_stream();
    if (!ws && !no_workspace && !g) {
      const size_t need = lib.forward_scratch_bytes(&d);
      if (need) {
        // (first: without memory for it the call runs whole, whatever earlier calls have kept, and so gives the same bits)
        const at::Tensor own = scratch(need);
        if (const size_t bytes = kept_bytes(s, d, stream)) {
          const at::Tensor kept = record_of(bytes, stream);  // (held through the call)
          if (kept.defined())
            return call(lib.kd_kept, &d, sp, tp, ip, vp, labels, mask, nullptr, kd_tok, nll, tnll, lse, status, kept.data_ptr(),
                        (size_t)kept.numel(), stream);
        }
        return call(lib.kd_forward, &d, sp, tp, ip, vp, labels, mask, kd_tok, nll, tnll, lse, status, own.data_ptr(), need, stream);
      }
    }
    const size_t need = !ws && !no_workspace && g ? lib.workspace_bytes(&d) : 0;
    if (need) {
      const size_t want = lib.workspace_bytes_preferred(&d);
      at::Tensor w;  // (held through the call)
      if (const size_t bytes = kept_bytes(s, d, stream)) {
        const at::Tensor kept = record_of(bytes, stream);  // (held through the call)
        if (kept.defined())
          return call(lib.kd_kept, &d, sp, tp, ip, vp, labels, mask, gp, kd_tok, nll, tnll, lse, status, kept.data_ptr(),
                      (size_t)kept.numel(), stream);
        w = scratch(want);  // (calls on other streams, and graphs that are replayed, may use the buffer below meanwhile)
      } else if (!((ce != 0.0 && tau != 1.0) || (((uintptr_t)sp | (uintptr_t)(2 * d.student_stride)) & 15) != 0)) {
        // as binding._workspace
        PyObject* key = PyLong_FromLong(s.get_device());
        PyObject* kept = key ? PyDict_GetItemWithError(workspaces, key) : nullptr;  // borrowed
        Py_XDECREF(key);
        if (!kept || !THPVariable_CheckExact(kept)) throw NotPlain();  // (Python makes it)
        w = THPVariable_Unpack(kept);
        if (!w.is_cuda() || (size_t)w.numel() < need) throw NotPlain();
      }
      if (!w.defined() || (size_t)w.numel() < want) w = scratch(want);
      return call(lib.kd, &d, sp, tp, ip, vp, labels, mask, gp, kd_tok, nll, tnll, lse, status, w.data_ptr(), (size_t)w.nbytes(),
                    stream);
    }
    return call(lib.kd, &d, sp, tp, ip, vp, labels, mask, gp, kd_tok, nll, tnll, lse, status, ws ? ws->data_ptr() : nullptr,
                  ws ? (size_t)ws->numel() * ws->element_size() : 0, stream);
  });
}

// (values, loss_mask, cu_seqlens, seg_sum, seg_count, seg_mean, token_to_sample, dev_status)
PyObject* segment_reduce(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 8) return PyLong_FromLong(-1);
  return guarded([&]() -> int {
    const at::Tensor &mask = required(a[1]), &cu = required(a[2]);
    const int64_t T = mask.numel(), S = cu.numel() - 1;
    if (S < 0 || S > 0x7fffffffLL) throw NotPlain();
    return call(lib.segment_reduce, T, (int32_t)S, array_of<float>(a[0], T, at::kFloat),
                              static_cast<uint8_t*>(pointer(&mask, at::kByte)), static_cast<int32_t*>(pointer(&cu, at::kInt)),
                              array_of<float>(a[3], S, at::kFloat), array_of<int32_t>(a[4], S, at::kInt),
                              array_of<float>(a[5], S, at::kFloat), array_of<int32_t>(a[6], T, at::kInt),
                              static_cast<int32_t*>(pointer(tensor(a[7]), at::kInt)), current_stream());
  });
}

// (mean_nll_student, mean_nll_teacher, seg_count, pair_cond, pair_uncond, lo, hi, flags, ifd_student, ifd_teacher, delta,
//  zone, keep, keep_count)
PyObject* delta_ifd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 14) return PyLong_FromLong(-1);
  return guarded([&]() -> int {
    const at::Tensor &ms = required(a[0]), &mt = required(a[1]), &cnt = required(a[2]), &pc = required(a[3]),
                     &pu = required(a[4]);
    const int64_t S = ms.numel(), P = pc.numel();
    if (mt.numel() != S || cnt.numel() != S || pu.numel() != P || S > 0x7fffffffLL || P > 0x7fffffffLL) throw NotPlain();
    const long flags = whole(a[7]);
    if (flags < 0) throw NotPlain();
    return call(lib.delta_ifd, (int32_t)P, (int32_t)S, static_cast<float*>(pointer(&ms, at::kFloat)),
                         static_cast<float*>(pointer(&mt, at::kFloat)), static_cast<int32_t*>(pointer(&cnt, at::kInt)),
                         static_cast<int32_t*>(pointer(&pc, at::kInt)), static_cast<int32_t*>(pointer(&pu, at::kInt)),
                         (float)number(a[5]), (float)number(a[6]), (uint32_t)flags, array_of<float>(a[8], P, at::kFloat),
                         array_of<float>(a[9], P, at::kFloat), array_of<float>(a[10], P, at::kFloat),
                         array_of<uint8_t>(a[11], P, at::kByte), array_of<uint8_t>(a[12], P, at::kByte),
                         static_cast<int32_t*>(pointer(tensor(a[13]), at::kInt)), current_stream());
  });
}

// (teacher_logits, k, topk_idx, topk_val, loss_mask, log_probs)
PyObject* teacher_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 6) return PyLong_FromLong(-1);
  return guarded([&]() -> int {
    const at::Tensor &t = required(a[0]), &idx = required(a[2]), &val = required(a[3]);
    const int64_t stride = row_stride(t), T = t.size(0), V = t.size(1);
    const long k = whole(a[1]);
    if (V > 0x7fffffffLL) throw NotPlain();
    for (const at::Tensor* o : {&idx, &val})
      if (o->dim() != 2 || o->size(0) != T || o->size(1) != k || !o->is_contiguous()) throw NotPlain();
    return call(lib.teacher_topk, T, (int32_t)V, stride, (int32_t)k, flag(a[5]) ? NPD_TOPK_LOG_PROBS : 0u,
                            pointer(&t, at::kBFloat16), array_of<uint8_t>(a[4], T, at::kByte),
                            static_cast<int32_t*>(pointer(&idx, at::kInt)), static_cast<float*>(pointer(&val, at::kFloat)),
                            current_stream());
  });
}

// (kl_tok, loss_mask, cu_seqlens, epsilon, seg_kl_mean, seg_count, batch_kl_mean, batch_count, lag_exceeded, dev_status)
PyObject* policy_lag(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) return PyLong_FromLong(-1);
  return guarded([&]() -> int {
    const at::Tensor &mask = required(a[1]), &cu = required(a[2]);
    const int64_t T = mask.numel(), S = cu.numel() - 1;
    if (S < 0 || S > 0x7fffffffLL) throw NotPlain();
    return call(lib.policy_lag, T, (int32_t)S, array_of<float>(a[0], T, at::kFloat),
                          static_cast<uint8_t*>(pointer(&mask, at::kByte)), static_cast<int32_t*>(pointer(&cu, at::kInt)),
                          (float)number(a[3]), array_of<float>(a[4], S, at::kFloat), array_of<int32_t>(a[5], S, at::kInt),
                          array_of<float>(a[6], 1, at::kFloat), array_of<int32_t>(a[7], 1, at::kInt),
                          array_of<int32_t>(a[8], 1, at::kInt), static_cast<int32_t*>(pointer(tensor(a[9]), at::kInt)),
                          current_stream());
  });
}

// bind(raw_stream, workspaces, addresses): `addresses` of libnpd's entry points in the order of Entry; 0 for both of the last two:
// a library without them
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *stream, *kept, *addresses;
  if (!PyArg_ParseTuple(args, "OO!O!", &stream, &PyDict_Type, &kept, &PyTuple_Type, &addresses)) return nullptr;
  constexpr int kEntries = 11, kRequired = 9;
  void* p[kEntries];
  if (PyTuple_GET_SIZE(addresses) != kEntries) {
    PyErr_SetString(PyExc_ValueError, "11 addresses");
    return nullptr;
  }
  for (int i = 0; i < kEntries; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (!p[i] && PyErr_Occurred()) return nullptr;
    if (i < kRequired ? !p[i] : !p[i] != !p[kRequired]) {
      PyErr_SetString(PyExc_ValueError, "a null address");
      return nullptr;
    }
  }
  records().clear();  // (another library counts its calls anew: what they left could pass for words of its first ones)
  Py_INCREF(stream);
  Py_INCREF(kept);
  Py_XSETREF(raw_stream, stream);
  Py_XSETREF(workspaces, kept);
  lib.workspace_bytes = reinterpret_cast<decltype(lib.workspace_bytes)>(p[0]);
  lib.workspace_bytes_preferred = reinterpret_cast<decltype(lib.workspace_bytes_preferred)>(p[1]);
  lib.forward_scratch_bytes = reinterpret_cast<decltype(lib.forward_scratch_bytes)>(p[2]);
  lib.kd = reinterpret_cast<decltype(lib.kd)>(p[3]);
  lib.kd_forward = reinterpret_cast<decltype(lib.kd_forward)>(p[4]);
  lib.segment_reduce = reinterpret_cast<decltype(lib.segment_reduce)>(p[5]);
  lib.delta_ifd = reinterpret_cast<decltype(lib.delta_ifd)>(p[6]);
  lib.teacher_topk = reinterpret_cast<decltype(lib.teacher_topk)>(p[7]);
  lib.policy_lag = reinterpret_cast<decltype(lib.policy_lag)>(p[8]);
  lib.kept_bytes = reinterpret_cast<decltype(lib.kept_bytes)>(p[9]);
  lib.kd_kept = reinterpret_cast<decltype(lib.kd_kept)>(p[10]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"kd", reinterpret_cast<PyCFunction>(kd), METH_FASTCALL, nullptr},
    {"segment_reduce", reinterpret_cast<PyCFunction>(segment_reduce), METH_FASTCALL, nullptr},
    {"delta_ifd", reinterpret_cast<PyCFunction>(delta_ifd), METH_FASTCALL, nullptr},
    {"teacher_topk", reinterpret_cast<PyCFunction>(teacher_topk), METH_FASTCALL, nullptr},
    {"policy_lag", reinterpret_cast<PyCFunction>(policy_lag), METH_FASTCALL, nullptr},
    {"release", release, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "npd_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_npd_host() { return PyModule_Create(&module); }
