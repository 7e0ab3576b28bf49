// The binding's per-call work in native code: checks, output allocation, the
// current stream and the C-ABI call.  In Python these took 9-11 us a call,
// more than the kernels of a decode step or of a small layer (128 x 256 x 256,
// quantize X, quantize W, GEMM: 50 us a pass, 28 of them kernels).
//
// Every function takes exactly the calls it can prove ordinary (torch.Tensor
// or Parameter objects of the expected dtype, shape, strides and device, plain
// ints) and returns None for any other, without having done anything: the
// Python code in __init__.py then makes the call or raises the error that
// names what is wrong.  It returns the outputs, or the fp8q_status of a call
// the library refused, as an int.  The GIL is released around the library
// call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cxxabi.h>

#include <cstring>

#include "fp8q.h"

namespace {

// the library's entry points, from the loaded libfp8q.so (see bind)
struct Api {
  decltype(&fp8q_scales_count) scales_count;
  decltype(&fp8q_quantize) quantize;
  decltype(&fp8q_quantize_dual) quantize_dual;
  decltype(&fp8q_gemm_formats) gemm_formats;
  decltype(&fp8q_gemm_grouped) gemm_grouped;
  decltype(&fp8q_gemm_pow2) gemm_pow2;
  decltype(&fp8q_gemm_quantized) gemm_quantized;
  decltype(&fp8q_gemm_splitk_workspace) splitk_workspace;
  decltype(&fp8q_gemm_splitk) gemm_splitk;
  decltype(&fp8q_calibrate_clip_workspace) clip_workspace;
  decltype(&fp8q_calibrate_clip) calibrate_clip;
};
constexpr Py_ssize_t kApiSize = sizeof(Api) / sizeof(void*);

// Not an ordinary call: left to the Python code.
struct NotOrdinary {};
[[noreturn]] void leave() { throw NotOrdinary{}; }

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) leave();
  return THPVariable_Unpack(o);
}

int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) leave();
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) leave();
  return v;
}

double real(PyObject* o) {
  if (!PyFloat_CheckExact(o)) leave();
  return PyFloat_AS_DOUBLE(o);
}

// t is a row-major 2-D tensor of the dtype on the GPU
const at::Tensor& matrix(PyObject* o, at::ScalarType dtype) {
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != dtype || t.dim() != 2 || t.stride(1) != 1) leave();
  return t;
}

// the same with that shape and device, or a new one for None
at::Tensor matrix_or_new(PyObject* o, at::ScalarType dtype, int64_t rows, int64_t cols, c10::Device device) {
  if (o == Py_None) return at::empty({rows, cols}, at::TensorOptions().dtype(dtype).device(device));
  const at::Tensor& t = matrix(o, dtype);
  if (t.size(0) != rows || t.size(1) != cols || t.device() != device) leave();
  return t;
}

// t is a contiguous tensor of the dtype on the device, of n elements or more
const at::Tensor& vector(PyObject* o, at::ScalarType dtype, int64_t n, c10::Device device) {
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != dtype || !t.is_contiguous() ||
      t.device() != device || t.numel() < n)
    leave();
  return t;
}

at::Tensor vector_or_new(PyObject* o, at::ScalarType dtype, int64_t n, c10::Device device) {
  if (o == Py_None) return at::empty({n}, at::TensorOptions().dtype(dtype).device(device));
  return vector(o, dtype, n, device);
}

ihipStream_t* stream_of(const at::Tensor& t) {
  return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.device().index()).stream();
}

// The caller's object, or a new one for an output made here.
PyObject* give(PyObject* given, const at::Tensor& t) {
  if (given == Py_None) return THPVariable_Wrap(t);
  Py_INCREF(given);
  return given;
}

PyObject* pack(std::initializer_list<PyObject*> items) {
  PyObject* r = PyTuple_New((Py_ssize_t)items.size());
  Py_ssize_t i = 0;
  bool ok = r != nullptr;
  for (PyObject* o : items) {
    ok = ok && o;
    if (r) PyTuple_SET_ITEM(r, i++, o);
    else Py_XDECREF(o);
  }
  if (!ok) Py_CLEAR(r);
  return r;
}

// f() with the GIL released; f throws nothing.  Taken back by a call and not
// by a destructor: in a daemon thread that returns while the interpreter shuts
// down, PyEval_RestoreThread ends the thread by unwinding its stack, which a
// destructor (noexcept) would turn into an abort of the process.
template <typename F>
auto unlocked(F&& f) {
  PyThreadState* const s = PyEval_SaveThread();
  const auto r = f();
  PyEval_RestoreThread(s);
  return r;
}

Api* api_of(PyObject* module) { return static_cast<Api*>(PyModule_GetState(module)); }

// f(api, args), with everything it throws turned into "not an ordinary call"
// (the Python code then meets the same condition and reports it), but for the
// unwinding of a thread that ends (see unlocked), which must go on.
template <Py_ssize_t N, typename F>
PyObject* guarded(PyObject* module, PyObject* const* args, Py_ssize_t n, F&& f) {
  const Api* api = api_of(module);
  if (n == N && api->quantize) {
    try {
      return f(*api, args);
    } catch (abi::__forced_unwind&) {
      throw;
    } catch (...) {
      PyErr_Clear();
    }
  }
  Py_RETURN_NONE;
}

// quantize(x, granularity, flags, codes, scales) -> (codes, scales)
PyObject* py_quantize(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<5>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const at::Tensor& x = matrix(a[0], at::kBFloat16);
    const auto g = (fp8q_granularity)integer(a[1]);
    const unsigned flags = (unsigned)integer(a[2]);
    const int64_t rows = x.size(0), cols = x.size(1);
    const int64_t ns = api.scales_count(rows, cols, g, flags & FP8Q_OUT_TRANSPOSED);
    if (ns < 0) leave();
    const bool t = flags & FP8Q_OUT_TRANSPOSED;
    const at::Tensor codes = matrix_or_new(a[3], at::kByte, t ? cols : rows, t ? rows : cols, x.device());
    const at::Tensor scales = vector_or_new(a[4], at::kFloat, ns, x.device());
    const void* xp = x.const_data_ptr();
    uint8_t* cp = codes.mutable_data_ptr<uint8_t>();
    float* sp = scales.mutable_data_ptr<float>();
    ihipStream_t* s = stream_of(x);
    const fp8q_status st = unlocked([&] {
      return api.quantize(xp, rows, cols, x.stride(0), g, flags, cp, codes.stride(0), sp, s);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    return pack({give(a[3], codes), give(a[4], scales)});
  });
}

// quantize_dual(x, flags, codes_r, scales_r, codes_t, scales_t) -> the four
PyObject* py_quantize_dual(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<6>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const at::Tensor& x = matrix(a[0], at::kBFloat16);
    const unsigned flags = (unsigned)integer(a[1]);
    const int64_t rows = x.size(0), cols = x.size(1);
    const int64_t nr = api.scales_count(rows, cols, FP8Q_BLOCK_1x128, 0);
    const int64_t nt = api.scales_count(rows, cols, FP8Q_BLOCK_128x1, FP8Q_OUT_TRANSPOSED);
    if (nr < 0 || nt < 0) leave();
    const at::Tensor cr = matrix_or_new(a[2], at::kByte, rows, cols, x.device());
    const at::Tensor sr = vector_or_new(a[3], at::kFloat, nr, x.device());
    const at::Tensor ct = matrix_or_new(a[4], at::kByte, cols, rows, x.device());
    const at::Tensor sct = vector_or_new(a[5], at::kFloat, nt, x.device());
    const void* xp = x.const_data_ptr();
    uint8_t *crp = cr.mutable_data_ptr<uint8_t>(), *ctp = ct.mutable_data_ptr<uint8_t>();
    float *srp = sr.mutable_data_ptr<float>(), *stp = sct.mutable_data_ptr<float>();
    ihipStream_t* s = stream_of(x);
    const fp8q_status st = unlocked([&] {
      return api.quantize_dual(xp, rows, cols, x.stride(0), flags, crp, cr.stride(0), srp, ctp, ct.stride(0), stp, s);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    return pack({give(a[2], cr), give(a[3], sr), give(a[4], ct), give(a[5], sct)});
  });
}

// The operands shared by the GEMM entry points: a, sa, ga, b, sb, gb.
struct Operands {
  int64_t M, N, K, lda, ldb;
  fp8q_granularity ga, gb;
  const uint8_t *a, *b;
  const float *sa, *sb;
  c10::Device device;
  ihipStream_t* stream;
};

void operand(const Api& api, PyObject* oc, PyObject* os, fp8q_granularity g, c10::Device device, const at::Tensor*& c,
             const uint8_t*& cp, const float*& sp) {
  c = &matrix(oc, at::kByte);
  if (c->device() != device) leave();
  const int64_t ns = api.scales_count(c->size(0), c->size(1), g, 0);
  if (ns < 0) leave();
  cp = c->const_data_ptr<uint8_t>();
  sp = vector(os, at::kFloat, ns, device).const_data_ptr<float>();
}

Operands operands(const Api& api, PyObject* oa, PyObject* osa, fp8q_granularity ga, PyObject* ob, PyObject* osb,
                  fp8q_granularity gb) {
  const at::Tensor *a, *b;
  Operands p{0, 0, 0, 0, 0, ga, gb, nullptr, nullptr, nullptr, nullptr, tensor(oa).device(), nullptr};
  operand(api, oa, osa, ga, p.device, a, p.a, p.sa);
  operand(api, ob, osb, gb, p.device, b, p.b, p.sb);
  p.M = a->size(0);
  p.N = b->size(0);
  p.K = a->size(1);
  if (b->size(1) != p.K) leave();
  p.lda = a->stride(0);
  p.ldb = b->stride(0);
  p.stream = stream_of(*a);
  return p;
}

Operands operands(const Api& api, PyObject* const* a) {
  return operands(api, a[0], a[1], (fp8q_granularity)integer(a[2]), a[3], a[4], (fp8q_granularity)integer(a[5]));
}

// gemm(a, sa, ga, b, sb, gb, formats, out), gemm_pow2(a, .., gb, out) -> out
template <bool POW2>
PyObject* py_gemm(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<POW2 ? 7 : 8>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const Operands p = operands(api, a);
    PyObject* const given = a[POW2 ? 6 : 7];
    const unsigned formats = POW2 ? 0u : (unsigned)integer(a[6]);
    const at::Tensor out = matrix_or_new(given, at::kBFloat16, p.M, p.N, p.device);
    void* cp = out.mutable_data_ptr();
    const fp8q_status st = unlocked([&] {
      return POW2 ? api.gemm_pow2(p.a, p.sa, p.ga, p.lda, p.b, p.sb, p.gb, p.ldb, p.M, p.N, p.K, cp, out.stride(0),
                                p.stream)
                : api.gemm_formats(p.a, p.sa, p.ga, p.lda, p.b, p.sb, p.gb, p.ldb, p.M, p.N, p.K, formats, cp,
                                   out.stride(0), p.stream);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    return give(given, out);
  });
}

// gemm_splitk(a, sa, ga, b, sb, gb, out, workspace) -> out
PyObject* py_gemm_splitk(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<8>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const Operands p = operands(api, a);
    const int64_t need = api.splitk_workspace(p.M, p.N, p.K);
    if (need < 0) leave();
    const at::Tensor& ws = vector(a[7], at::kByte, need, p.device);
    const at::Tensor out = matrix_or_new(a[6], at::kBFloat16, p.M, p.N, p.device);
    void *cp = out.mutable_data_ptr(), *wp = ws.mutable_data_ptr();
    const int64_t bytes = ws.numel();
    const fp8q_status st = unlocked([&] {
      return api.gemm_splitk(p.a, p.sa, p.ga, p.lda, p.b, p.sb, p.gb, p.ldb, p.M, p.N, p.K, cp, out.stride(0), wp, bytes,
                           p.stream);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    return give(a[6], out);
  });
}

// gemm_quantized(a, sa, ga, b, sb, gb, codes, scales) -> (codes, scales)
PyObject* py_gemm_quantized(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<8>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const Operands p = operands(api, a);
    const int64_t ns = api.scales_count(p.M, p.N, FP8Q_BLOCK_1x128, 0);
    if (ns < 0) leave();
    const at::Tensor codes = matrix_or_new(a[6], at::kByte, p.M, p.N, p.device);
    const at::Tensor scales = vector_or_new(a[7], at::kFloat, ns, p.device);
    uint8_t* cp = codes.mutable_data_ptr<uint8_t>();
    float* sp = scales.mutable_data_ptr<float>();
    const fp8q_status st = unlocked([&] {
      return api.gemm_quantized(p.a, p.sa, p.ga, p.lda, p.b, p.sb, p.gb, p.ldb, p.M, p.N, p.K, cp, codes.stride(0), sp,
                              p.stream);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    return pack({give(a[6], codes), give(a[7], scales)});
  });
}

// gemm_grouped([(a, sa, b, sb), ..], ga, gb, outs) -> outs (a list; the
// caller's object when given)
PyObject* py_gemm_grouped(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<4>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    if (!PyList_CheckExact(a[0])) leave();
    const Py_ssize_t count = PyList_GET_SIZE(a[0]);
    const bool given = a[3] != Py_None;
    if (count < 1 || count > FP8Q_MAX_GROUP || (given && (!PyList_CheckExact(a[3]) || PyList_GET_SIZE(a[3]) != count)))
      leave();
    const auto ga = (fp8q_granularity)integer(a[1]), gb = (fp8q_granularity)integer(a[2]);
    fp8q_gemm_problem probs[FP8Q_MAX_GROUP];
    at::Tensor outs[FP8Q_MAX_GROUP];
    int64_t K = 0;
    c10::Device device(c10::DeviceType::CPU);
    ihipStream_t* stream = nullptr;
    for (Py_ssize_t i = 0; i < count; ++i) {
      PyObject* t = PyList_GET_ITEM(a[0], i);
      if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 4) leave();
      const Operands p = operands(api, PyTuple_GET_ITEM(t, 0), PyTuple_GET_ITEM(t, 1), ga, PyTuple_GET_ITEM(t, 2),
                                  PyTuple_GET_ITEM(t, 3), gb);
      if (i == 0) {
        K = p.K;
        device = p.device;
        stream = p.stream;
      } else if (p.K != K || p.device != device) {
        leave();
      }
      outs[i] = matrix_or_new(given ? PyList_GET_ITEM(a[3], i) : Py_None, at::kBFloat16, p.M, p.N, device);
      probs[i] = fp8q_gemm_problem{p.a, p.sa, p.lda, p.b, p.sb, p.ldb, outs[i].mutable_data_ptr(), outs[i].stride(0), p.M, p.N};
    }
    const fp8q_status st = unlocked([&] {
      return api.gemm_grouped(probs, (int)count, ga, gb, K, stream);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    if (given) {
      Py_INCREF(a[3]);
      return a[3];
    }
    PyObject* list = PyList_New(count);
    for (Py_ssize_t i = 0; list && i < count; ++i) {
      PyObject* o = THPVariable_Wrap(outs[i]);
      if (!o) Py_CLEAR(list);
      else PyList_SET_ITEM(list, i, o);
    }
    return list;
  });
}

// calibrate_clip(adv, w_tis, pi_sampler, r_bf16, r_fp8, l_old, h_old, address
// of an fp8q_clip_config, workspace, result, read) -> the result's bytes with
// read (the result itself when reading it failed), else True
PyObject* py_calibrate_clip(PyObject* m, PyObject* const* a, Py_ssize_t n) {
  return guarded<11>(m, a, n, [](const Api& api, PyObject* const* a) -> PyObject* {
    const float* in[5];
    const at::Tensor& adv = tensor(a[0]);
    const int64_t tokens = adv.numel();
    for (int i = 0; i < 5; ++i) {
      const at::Tensor& t = vector(a[i], at::kFloat, tokens, adv.device());
      if (t.numel() != tokens) leave();
      in[i] = t.const_data_ptr<float>();
    }
    const double l_old = real(a[5]), h_old = real(a[6]);
    const auto* config = reinterpret_cast<const fp8q_clip_config*>((uintptr_t)integer(a[7]));
    const int64_t need = api.clip_workspace(tokens);
    if (need < 0) leave();
    const at::Tensor ws = vector_or_new(a[8], at::kByte, need, adv.device());
    constexpr int64_t kResult = sizeof(fp8q_clip_result);
    const at::Tensor result = vector_or_new(a[9], at::kByte, kResult, adv.device());
    void* wp = ws.mutable_data_ptr();
    auto* rp = static_cast<fp8q_clip_result*>(result.mutable_data_ptr());
    const int64_t bytes = ws.numel();
    ihipStream_t* s = stream_of(adv);
    if (a[10] != Py_True && a[10] != Py_False) leave();
    const fp8q_status st = unlocked([&] {
      return api.calibrate_clip(in[0], in[1], in[2], in[3], in[4], tokens, l_old, h_old, config, wp, bytes, rp, s);
    });
    if (st != FP8Q_OK) return PyLong_FromLong(st);
    if (a[10] == Py_False) Py_RETURN_TRUE;
    at::Tensor host;
    const bool read = unlocked([&] {  // the copy waits for the kernels
      try {
        host = result.reshape({-1}).slice(0, 0, kResult).cpu();
        return true;
      } catch (...) {
        return false;
      }
    });
    if (!read) return give(a[9], result);  // the Python code reads it again and reports why
    return PyBytes_FromStringAndSize(static_cast<const char*>(host.const_data_ptr()), kResult);
  });
}

// bind((address, ..)): the entry points of Api, in its order
PyObject* py_bind(PyObject* m, PyObject* addresses) {
  if (!PyTuple_CheckExact(addresses) || PyTuple_GET_SIZE(addresses) != kApiSize) {
    PyErr_SetString(PyExc_ValueError, "bind: a tuple of the entry points' addresses");
    return nullptr;
  }
  void* p[kApiSize];
  for (Py_ssize_t i = 0; i < kApiSize; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: a null address");
      return nullptr;
    }
  }
  std::memcpy(static_cast<void*>(api_of(m)), p, sizeof p);
  Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", py_bind, METH_O, nullptr},
    {"quantize", FAST(py_quantize), nullptr},
    {"quantize_dual", FAST(py_quantize_dual), nullptr},
    {"gemm", FAST(py_gemm<false>), nullptr},
    {"gemm_pow2", FAST(py_gemm<true>), nullptr},
    {"gemm_splitk", FAST(py_gemm_splitk), nullptr},
    {"gemm_quantized", FAST(py_gemm_quantized), nullptr},
    {"gemm_grouped", FAST(py_gemm_grouped), nullptr},
    {"calibrate_clip", FAST(py_calibrate_clip), nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, sizeof(Api), methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  PyObject* m = PyModule_Create(&module);
  if (m) std::memset(PyModule_GetState(m), 0, sizeof(Api));
  return m;
}
