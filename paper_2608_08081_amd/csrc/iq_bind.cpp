// Native argument checks of the Python binding (module _bind).
//
// Each function takes the arguments of one api.py entry point, checks every
// tensor (device, dtype, shape, contiguity) exactly as api.py does, and calls
// the C ABI on the current stream of the tensors' device.  It returns the
// status, or None when it did not call: some argument is not what the call
// takes, or is of a kind that only the general Python path handles (tensor
// subclasses, tensors without storage, missing workspaces).  api.py then runs
// that path, which names the fault or handles the case.  Nothing is kept from
// one call for the next.
//
// Why: ten tensors checked and converted in Python and passed through ctypes
// cost a fused step's call more than its kernels take (32K positions, calls
// back to back with the reset of the length: 24.3 us, now 13.4; decode of one
// head over 1K positions 18.9 and 8.8; compression of 1021 tokens 13.9 and 7.1).
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <initializer_list>

#include "isoquant.h"

namespace {

// The library's functions, set once by bind() when it is loaded.
struct Functions {
  decltype(&iq_compress_kv) compress;
  decltype(&iq_compress_kv_bits) compress_bits;
  decltype(&iq_decode_attention) decode;
  decltype(&iq_decode_attention_bits) decode_bits;
  decltype(&iq_decode_step) step;
  decltype(&iq_decode_step_bits) step_bits;
  decltype(&iq_decode_attention_paged) decode_paged;
  decltype(&iq_decode_step_paged) step_paged;
  decltype(&iq_decode_attention_multi) multi;
  decltype(&iq_decode_attention_multi_bits) multi_bits;
  decltype(&iq_decode_step_multi) step_multi;
  decltype(&iq_decode_attention_rope) rope;
  decltype(&iq_dequantize_kv) dequantize;
} fn;

constexpr auto kF32 = at::kFloat;
constexpr auto kF16 = at::kHalf;
constexpr auto kU8 = at::kByte;
constexpr auto kI32 = at::kInt;

// The arguments of one call; `ok` falls when one of them is not for this path.
struct Args {
  PyObject* const* v;
  int dev = -1;   // the device of the first tensor
  bool ok;

  Args(PyObject* const* values, Py_ssize_t n, Py_ssize_t want) : v(values), ok(n == want) {}

  // Argument i if it is a plain contiguous device tensor on the call's device.
  const at::Tensor* any(int i) {
    if (!ok || !THPVariable_CheckExact(v[i])) return fail();
    const at::Tensor& t = THPVariable_Unpack(v[i]);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.is_contiguous())
      return fail();
    if (dev < 0) dev = t.get_device();
    return t.get_device() == dev ? &t : fail();
  }
  const at::Tensor* fail() {
    ok = false;
    return nullptr;
  }
  // The sizes of tensor i if it has `dims` of them.
  at::IntArrayRef sizes(int i, int64_t dims) {
    static const int64_t none[4] = {0, 0, 0, 0};
    const at::Tensor* t = any(i);
    if (t != nullptr && t->dim() == dims) return t->sizes();
    ok = false;
    return at::IntArrayRef(none, 4);
  }
  void* tensor(int i, at::ScalarType type, std::initializer_list<int64_t> shape) {
    const at::Tensor* t = any(i);
    if (t == nullptr || t->scalar_type() != type || !t->sizes().equals(shape)) {
      ok = false;
      return nullptr;
    }
    return t->data_ptr();
  }
  void* optional(int i, at::ScalarType type, std::initializer_list<int64_t> shape) {
    return v[i] == Py_None ? nullptr : tensor(i, type, shape);
  }
  // A K/V input, fp32 or fp16.
  void* input(int i, std::initializer_list<int64_t> shape, int32_t* dtype) {
    const at::Tensor* t = any(i);
    if (t == nullptr || (t->scalar_type() != kF32 && t->scalar_type() != kF16)) {
      ok = false;
      return nullptr;
    }
    *dtype = t->scalar_type() == kF16 ? IQ_DTYPE_F16 : IQ_DTYPE_F32;
    return tensor(i, t->scalar_type(), shape);
  }
  void* workspace(int i, size_t* bytes) {
    const at::Tensor* t = any(i);
    if (t == nullptr || t->scalar_type() != kU8) {
      ok = false;
      return nullptr;
    }
    *bytes = static_cast<size_t>(t->numel());
    return t->data_ptr();
  }
  int64_t integer(int i) {
    if (!PyLong_CheckExact(v[i])) {
      ok = false;
      return 0;
    }
    int over = 0;
    const long long x = PyLong_AsLongLongAndOverflow(v[i], &over);
    if (over != 0) ok = false;
    return x;
  }
  int64_t integer_or(int i, int64_t missing) { return v[i] == Py_None ? missing : integer(i); }
  float real(int i) {
    if (!PyFloat_CheckExact(v[i]) && !PyLong_CheckExact(v[i])) {
      ok = false;
      return 0.f;
    }
    const double x = PyFloat_AsDouble(v[i]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return static_cast<float>(x);
  }
  hipStream_t stream() const {
    return c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(dev)).stream();
  }
};

// The interpreter lock, given back for a scope; taken again also when an
// exception leaves it.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  Unlocked() = default;
  Unlocked(const Unlocked&) = delete;
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// Runs one entry point: `body` fills its arguments and returns a callable that
// makes the call (used only when every argument is fit).  An exception before
// the call leaves it to the general path; one out of the call is an error: it
// may have launched, so it is not made again.
template <class Body>
PyObject* run(PyObject* const* v, Py_ssize_t n, Py_ssize_t want, Body body) {
  bool called = false;
  try {
    Args a(v, n, want);
    if (!a.ok) Py_RETURN_NONE;
    int status = 0;
    body(a, [&](auto call) {
      if (!a.ok) return;
      const hipStream_t stream = a.stream();
      called = true;
      const Unlocked u;
      status = call(stream);
    });
    if (!called) Py_RETURN_NONE;
    return PyLong_FromLong(status);
  } catch (const std::exception& e) {   // e.g. a tensor without storage
    if (called) {
      PyErr_SetString(PyExc_RuntimeError, e.what());
      return nullptr;
    }
  } catch (...) {
    if (called) {
      PyErr_SetString(PyExc_RuntimeError, "unknown exception");
      return nullptr;
    }
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

template <class T>
T* as(void* p) {
  return static_cast<T*>(p);
}

#define IQ_BIND(name) PyObject* name(PyObject*, PyObject* const* v, Py_ssize_t n)

// (k, v, quats, k_codes, k_norms, v_codes, v_norms, dst_offset, bits)
IQ_BIND(compress) {
  return run(v, n, 9, [](Args& a, auto go) {
    const auto s = a.sizes(0, 4);
    const int64_t b = s[0], h = s[1], t = s[2], cap = a.sizes(3, 4)[2], bits = a.integer(8);
    int32_t d = 0, dv = 0;
    void* k = a.input(0, {b, h, t, IQ_HEAD_DIM}, &d);
    void* x = a.input(1, {b, h, t, IQ_HEAD_DIM}, &dv);
    if (d != dv) a.ok = false;
    void* quats = a.tensor(2, kF32, {h, 32, 2, 4});
    void* kc = a.tensor(3, kU8, {b, h, cap, 16 * bits});
    void* kn = a.tensor(4, kF32, {b, h, cap});
    void* vc = a.tensor(5, kU8, {b, h, cap, 16 * bits});
    void* vn = a.tensor(6, kF32, {b, h, cap});
    const int64_t off = a.integer(7);
    go([&](hipStream_t st) {
      if (bits == 3)
        return fn.compress(k, x, d, b, h, t, IQ_HEAD_DIM, as<float>(quats), as<uint8_t>(kc),
                           as<float>(kn), as<uint8_t>(vc), as<float>(vn), cap, off, st);
      return fn.compress_bits(k, x, d, b, h, t, IQ_HEAD_DIM, as<float>(quats), as<uint8_t>(kc),
                              as<float>(kn), as<uint8_t>(vc), as<float>(vn), cap, off,
                              static_cast<int>(bits), st);
    });
  });
}

// A contiguous cache: k_codes, k_norms, v_codes, v_norms, seq_lens, quats at
// arguments i ..
struct Cache {
  int64_t h = 0, cap = 0;
  void *kc = nullptr, *kn = nullptr, *vc = nullptr, *vn = nullptr, *lens = nullptr,
       *quats = nullptr;
  Cache(Args& a, int i, int64_t b, int64_t bits) {
    const auto s = a.sizes(i, 4);
    h = s[1];
    cap = s[2];
    kc = a.tensor(i, kU8, {b, h, cap, 16 * bits});
    kn = a.tensor(i + 1, kF32, {b, h, cap});
    vc = a.tensor(i + 2, kU8, {b, h, cap, 16 * bits});
    vn = a.tensor(i + 3, kF32, {b, h, cap});
    lens = a.tensor(i + 4, kI32, {b});
    quats = a.tensor(i + 5, kF32, {h, 32, 2, 4});
  }
};

// (q, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, out, workspace, max_seq_len, scale,
//  bits)
IQ_BIND(decode) {
  return run(v, n, 12, [](Args& a, auto go) {
    const auto s = a.sizes(0, 3);
    const int64_t b = s[0], hq = s[1], bits = a.integer(11);
    void* q = a.tensor(0, kF32, {b, hq, IQ_HEAD_DIM});
    const Cache c(a, 1, b, bits);
    void* out = a.tensor(7, kF32, {b, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(8, &bytes);
    const int64_t most = a.integer_or(9, c.cap);
    const float scale = a.real(10);
    go([&](hipStream_t st) {
      if (bits == 3)
        return fn.decode(as<float>(q), as<uint8_t>(c.kc), as<float>(c.kn), as<uint8_t>(c.vc),
                         as<float>(c.vn), as<int32_t>(c.lens), c.cap, most, as<float>(c.quats), b,
                         hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws, bytes, st);
      return fn.decode_bits(as<float>(q), as<uint8_t>(c.kc), as<float>(c.kn), as<uint8_t>(c.vc),
                            as<float>(c.vn), as<int32_t>(c.lens), c.cap, most, as<float>(c.quats),
                            b, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws, bytes,
                            static_cast<int>(bits), st);
    });
  });
}

// (q, k_new, v_new, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, out, workspace,
//  max_seq_len, scale, status, bits)
IQ_BIND(step) {
  return run(v, n, 15, [](Args& a, auto go) {
    const auto s = a.sizes(0, 3);
    const int64_t b = s[0], hq = s[1], bits = a.integer(14);
    void* q = a.tensor(0, kF32, {b, hq, IQ_HEAD_DIM});
    const Cache c(a, 3, b, bits);
    int32_t d = 0, dv = 0;
    void* k = a.input(1, {b, c.h, IQ_HEAD_DIM}, &d);
    void* x = a.input(2, {b, c.h, IQ_HEAD_DIM}, &dv);
    if (d != dv) a.ok = false;
    void* out = a.tensor(9, kF32, {b, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(10, &bytes);
    const int64_t most = a.integer_or(11, c.cap);
    const float scale = a.real(12);
    void* flag = a.optional(13, kI32, {1});
    go([&](hipStream_t st) {
      if (bits == 3)
        return fn.step(as<float>(q), k, x, d, as<uint8_t>(c.kc), as<float>(c.kn),
                       as<uint8_t>(c.vc), as<float>(c.vn), as<int32_t>(c.lens), c.cap, most,
                       as<float>(c.quats), b, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws,
                       bytes, as<int32_t>(flag), st);
      return fn.step_bits(as<float>(q), k, x, d, as<uint8_t>(c.kc), as<float>(c.kn),
                          as<uint8_t>(c.vc), as<float>(c.vn), as<int32_t>(c.lens), c.cap, most,
                          as<float>(c.quats), b, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws,
                          bytes, as<int32_t>(flag), static_cast<int>(bits), st);
    });
  });
}

// Page pools: k_codes, k_norms, v_codes, v_norms, block_tables, seq_lens, quats at i ..
struct Pools {
  int64_t pages = 0, h = 0, page = 0, most = 0;
  void *kc = nullptr, *kn = nullptr, *vc = nullptr, *vn = nullptr, *tab = nullptr,
       *lens = nullptr, *quats = nullptr;
  Pools(Args& a, int i, int64_t b) {
    const auto s = a.sizes(i, 4);
    pages = s[0];
    h = s[1];
    page = s[2];
    kc = a.tensor(i, kU8, {pages, h, page, IQ_RECORD_BYTES});
    kn = a.tensor(i + 1, kF32, {pages, h, page});
    vc = a.tensor(i + 2, kU8, {pages, h, page, IQ_RECORD_BYTES});
    vn = a.tensor(i + 3, kF32, {pages, h, page});
    // (a row for every sequence; more than the batch has are not read)
    const auto ts = a.sizes(i + 4, 2);
    most = ts[1];
    if (ts[0] < b) a.ok = false;
    tab = a.tensor(i + 4, kI32, {ts[0], most});
    lens = a.tensor(i + 5, kI32, {b});
    quats = a.tensor(i + 6, kF32, {h, 32, 2, 4});
  }
};

// (q, k_codes, k_norms, v_codes, v_norms, block_tables, seq_lens, quats, out, workspace,
//  max_seq_len, scale)
IQ_BIND(decode_paged) {
  return run(v, n, 12, [](Args& a, auto go) {
    const auto s = a.sizes(0, 3);
    const int64_t b = s[0], hq = s[1];
    void* q = a.tensor(0, kF32, {b, hq, IQ_HEAD_DIM});
    const Pools c(a, 1, b);
    void* out = a.tensor(8, kF32, {b, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(9, &bytes);
    const int64_t most = a.integer_or(10, c.most * c.page);
    const float scale = a.real(11);
    go([&](hipStream_t st) {
      return fn.decode_paged(as<float>(q), as<uint8_t>(c.kc), as<float>(c.kn), as<uint8_t>(c.vc),
                             as<float>(c.vn), c.page, c.pages, as<int32_t>(c.tab), c.most,
                             as<int32_t>(c.lens), most, as<float>(c.quats), b, hq, c.h,
                             IQ_HEAD_DIM, scale, as<float>(out), ws, bytes, st);
    });
  });
}

// (q, k_new, v_new, k_codes, k_norms, v_codes, v_norms, block_tables, seq_lens, quats, out,
//  workspace, max_seq_len, scale, status)
IQ_BIND(step_paged) {
  return run(v, n, 15, [](Args& a, auto go) {
    const auto s = a.sizes(0, 3);
    const int64_t b = s[0], hq = s[1];
    void* q = a.tensor(0, kF32, {b, hq, IQ_HEAD_DIM});
    const Pools c(a, 3, b);
    int32_t d = 0, dv = 0;
    void* k = a.input(1, {b, c.h, IQ_HEAD_DIM}, &d);
    void* x = a.input(2, {b, c.h, IQ_HEAD_DIM}, &dv);
    if (d != dv) a.ok = false;
    void* out = a.tensor(10, kF32, {b, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(11, &bytes);
    const int64_t most = a.integer_or(12, c.most * c.page);
    const float scale = a.real(13);
    void* flag = a.optional(14, kI32, {1});
    go([&](hipStream_t st) {
      return fn.step_paged(as<float>(q), k, x, d, as<uint8_t>(c.kc), as<float>(c.kn),
                           as<uint8_t>(c.vc), as<float>(c.vn), c.page, c.pages,
                           as<int32_t>(c.tab), c.most, as<int32_t>(c.lens), most,
                           as<float>(c.quats), b, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws,
                           bytes, as<int32_t>(flag), st);
    });
  });
}

// (q, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, out, workspace, max_seq_len, scale,
//  bits), q and out [B][T][H_q][128]
IQ_BIND(multi) {
  return run(v, n, 12, [](Args& a, auto go) {
    const auto s = a.sizes(0, 4);
    const int64_t b = s[0], t = s[1], hq = s[2], bits = a.integer(11);
    void* q = a.tensor(0, kF32, {b, t, hq, IQ_HEAD_DIM});
    const Cache c(a, 1, b, bits);
    void* out = a.tensor(7, kF32, {b, t, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(8, &bytes);
    const int64_t most = a.integer_or(9, c.cap);
    const float scale = a.real(10);
    go([&](hipStream_t st) {
      if (bits == 3)
        return fn.multi(as<float>(q), as<uint8_t>(c.kc), as<float>(c.kn), as<uint8_t>(c.vc),
                        as<float>(c.vn), as<int32_t>(c.lens), c.cap, most, as<float>(c.quats), b,
                        t, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws, bytes, st);
      return fn.multi_bits(as<float>(q), as<uint8_t>(c.kc), as<float>(c.kn), as<uint8_t>(c.vc),
                           as<float>(c.vn), as<int32_t>(c.lens), c.cap, most, as<float>(c.quats),
                           b, t, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out), ws, bytes,
                           static_cast<int>(bits), st);
    });
  });
}

// (q, k_new, v_new, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, out, workspace,
//  max_seq_len, scale, status, bits), with T tokens per sequence
IQ_BIND(step_multi) {
  return run(v, n, 15, [](Args& a, auto go) {
    const auto s = a.sizes(0, 4);
    const int64_t b = s[0], t = s[1], hq = s[2], bits = a.integer(14);
    void* q = a.tensor(0, kF32, {b, t, hq, IQ_HEAD_DIM});
    const Cache c(a, 3, b, bits);
    int32_t d = 0, dv = 0;
    void* k = a.input(1, {b, t, c.h, IQ_HEAD_DIM}, &d);
    void* x = a.input(2, {b, t, c.h, IQ_HEAD_DIM}, &dv);
    if (d != dv) a.ok = false;
    void* out = a.tensor(9, kF32, {b, t, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(10, &bytes);
    const int64_t most = a.integer_or(11, c.cap);
    const float scale = a.real(12);
    void* flag = a.optional(13, kI32, {1});
    go([&](hipStream_t st) {
      return fn.step_multi(as<float>(q), k, x, d, as<uint8_t>(c.kc), as<float>(c.kn),
                           as<uint8_t>(c.vc), as<float>(c.vn), as<int32_t>(c.lens), c.cap, most,
                           as<float>(c.quats), b, t, hq, c.h, IQ_HEAD_DIM, scale, as<float>(out),
                           ws, bytes, as<int32_t>(flag), static_cast<int>(bits), st);
    });
  });
}

// (q, q_rope, k_rope, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, out, workspace,
//  max_seq_len, scale)
IQ_BIND(rope) {
  return run(v, n, 13, [](Args& a, auto go) {
    const auto s = a.sizes(0, 3);
    const int64_t b = s[0], hq = s[1], hr = a.sizes(2, 4)[1];
    void* q = a.tensor(0, kF32, {b, hq, IQ_HEAD_DIM});
    void* qr = a.tensor(1, kF32, {b, hq, 64});
    const Cache c(a, 3, b, 3);
    void* kr = a.tensor(2, kF16, {b, hr, c.cap, 64});
    void* out = a.tensor(9, kF32, {b, hq, IQ_HEAD_DIM});
    size_t bytes = 0;
    void* ws = a.workspace(10, &bytes);
    const int64_t most = a.integer_or(11, c.cap);
    const float scale = a.real(12);
    go([&](hipStream_t st) {
      return fn.rope(as<float>(q), as<float>(qr), as<uint8_t>(c.kc), as<float>(c.kn), kr, hr,
                     as<uint8_t>(c.vc), as<float>(c.vn), as<int32_t>(c.lens), c.cap, most,
                     as<float>(c.quats), b, hq, c.h, IQ_HEAD_DIM, 64, scale, as<float>(out), ws,
                     bytes, st);
    });
  });
}

// (k_codes, k_norms, v_codes, v_norms, quats, n_tokens, src_offset, seq_lens, k_out, v_out)
IQ_BIND(dequantize) {
  return run(v, n, 10, [](Args& a, auto go) {
    const auto s = a.sizes(0, 4);
    const int64_t b = s[0], h = s[1], cap = s[2], off = a.integer(6);
    const int64_t t = a.integer_or(5, cap - off);
    void* kc = a.tensor(0, kU8, {b, h, cap, IQ_RECORD_BYTES});
    void* kn = a.tensor(1, kF32, {b, h, cap});
    void* vc = a.tensor(2, kU8, {b, h, cap, IQ_RECORD_BYTES});
    void* vn = a.tensor(3, kF32, {b, h, cap});
    void* quats = a.tensor(4, kF32, {h, 32, 2, 4});
    void* lens = a.optional(7, kI32, {b});
    int32_t d = 0, dv = 0;
    void* ko = a.input(8, {b, h, t, IQ_HEAD_DIM}, &d);
    void* vo = a.input(9, {b, h, t, IQ_HEAD_DIM}, &dv);
    if (d != dv) a.ok = false;
    go([&](hipStream_t st) {
      return fn.dequantize(as<uint8_t>(kc), as<float>(kn), as<uint8_t>(vc), as<float>(vn),
                           as<float>(quats), as<int32_t>(lens), b, h, t, IQ_HEAD_DIM, cap, off, d,
                           ko, vo, st);
    });
  });
}

template <class F>
bool set(F& f, PyObject* const* v, int i) {
  void* p = PyLong_AsVoidPtr(v[i]);
  if (p == nullptr) return false;
  f = reinterpret_cast<F>(p);
  return true;
}

// bind(addresses of the functions, in the order of Functions)
PyObject* bind(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n == 13 && set(fn.compress, v, 0) && set(fn.compress_bits, v, 1) && set(fn.decode, v, 2) &&
      set(fn.decode_bits, v, 3) && set(fn.step, v, 4) && set(fn.step_bits, v, 5) &&
      set(fn.decode_paged, v, 6) && set(fn.step_paged, v, 7) && set(fn.multi, v, 8) &&
      set(fn.multi_bits, v, 9) && set(fn.step_multi, v, 10) && set(fn.rope, v, 11) &&
      set(fn.dequantize, v, 12))
    Py_RETURN_NONE;
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: 13 function addresses expected");
  return nullptr;
}

#define IQ_METHOD(name)                                                            \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, \
   nullptr}
PyMethodDef methods[] = {IQ_METHOD(bind),         IQ_METHOD(compress),   IQ_METHOD(decode),
                         IQ_METHOD(step),         IQ_METHOD(decode_paged), IQ_METHOD(step_paged),
                         IQ_METHOD(multi),        IQ_METHOD(step_multi), IQ_METHOD(rope),
                         IQ_METHOD(dequantize),   {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind() { return PyModule_Create(&module); }
