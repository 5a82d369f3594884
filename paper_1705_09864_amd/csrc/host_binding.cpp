// The host side of a call from Python, as a CPython extension: tensors in, addresses and sizes
// through the C ABI of include/bmx.h, a tensor out.  binding.py declares the functions (names,
// arguments, defaults) and hands its arguments on in order; nothing here computes.
//
// Why it is native: the kernels of most layers run for 3 to 10 us and a launch takes the HIP
// runtime 2.7 us on the host, but the same steps written in Python (checks of each tensor,
// torch.empty twice, the stream object, ctypes' conversion of 14 arguments) took 10 us a call, more
// than the GPU's share: a loop over 64 x 512 -> 256 ran at 13.1 us a call.  Here they take about 1 us.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>
#include <initializer_list>
#include <optional>
#include <string>

#include "../../include/bmx.h"
#include "lazy_calls.h"

namespace {

PyObject* bmx_error = nullptr;      // binding.BmxError(status, what)
PyObject* str_cuda_stream = nullptr;

[[noreturn]] void raise_value(const char* fmt, const char* what, const char* a = "", const char* b = "") {
  PyErr_Format(PyExc_ValueError, fmt, what, a, b);
  throw python_error();
}

void check_status(int status, const char* what) {
  if (status == BMX_OK) return;
  PyObject* e = PyObject_CallFunction(bmx_error, "is", status, what);
  if (e) {
    PyErr_SetObject(bmx_error, e);
    Py_DECREF(e);
  }
  throw python_error();
}

constexpr auto kF32 = at::kFloat, kI32 = at::kInt, kU64 = at::kLong;

using T = const at::Tensor*;

// The guard in front of the C ABI, which sees only an address: on the GPU, of the element type the
// call reads or writes, unit stride along the last dimension (rows may be further apart), or, with
// `dense`, contiguous.  None gives a null pointer.
T tensor(PyObject* o, at::ScalarType type, const char* what, bool dense = false) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) raise_value("%s: expected a torch tensor, got %s", what, Py_TYPE(o)->tp_name);
  T t = &THPVariable_Unpack(o);
  if (!t->is_cuda()) raise_value("%s: tensor must live on the GPU (device is %s)", what, t->device().str().c_str());
  if (t->scalar_type() != type)
    raise_value("%s: dtype %s, expected %s", what, c10::toString(t->scalar_type()), c10::toString(type));
  if (dense) {
    if (!t->is_contiguous()) raise_value("%s: tensor must be contiguous", what);
  } else if (t->dim() >= 1 && t->numel() > 1 && t->size(-1) > 1 && t->stride(-1) != 1) {
    raise_value("%s: last dimension must have stride 1 (got %s)", what, std::to_string(t->stride(-1)).c_str());
  } else if (t->dim() > 2 && !t->is_contiguous()) {
    raise_value("%s: tensor must be contiguous", what);
  }
  return t;
}

T required(PyObject* o, at::ScalarType type, int dims, const char* what, bool dense = false) {
  T t = tensor(o, type, what, dense);
  if (!t) raise_value("%s: expected a torch tensor, got None%s%s", what);
  if (t->dim() != dims)
    raise_value("%s: expected %s dimensions, got %s", what, std::to_string(dims).c_str(), std::to_string(t->dim()).c_str());
  return t;
}

// A matrix by rows: size(0) of them, whatever dimensions a row has (a packed image [N, H, W, words] is N rows; a
// vector, rows of one element).  Of more than two dimensions only contiguous tensors pass the guard above.
T matrix(PyObject* o, at::ScalarType type, const char* what) {
  T t = tensor(o, type, what);
  if (!t) raise_value("%s: expected a torch tensor, got None%s%s", what);
  if (t->dim() < 2 && (t->dim() < 1 || t->size(0) < 2))
    raise_value("%s: expected rows of a matrix, got %s dimensions%s", what, std::to_string(t->dim()).c_str());
  return t;
}

// A packed image [N, H, W, words]; the words of a single one may be left out.
T packed_image(PyObject* o, const char* what) {
  T t = tensor(o, kU64, what, true);
  if (!t) raise_value("%s: expected a torch tensor, got None%s%s", what);
  if (t->dim() < 3) raise_value("%s: expected a packed image, got %s dimensions%s", what, std::to_string(t->dim()).c_str());
  return t;
}

template <class P>
P* ptr(T t) { return t ? static_cast<P*>(t->data_ptr()) : nullptr; }

// Row stride of a matrix in elements (its row length when it has a single row).
int64_t ld(T t) { return t->size(0) > 1 ? t->stride(0) : std::max<int64_t>(t->dim() == 2 ? t->size(1) : t->numel(), 1); }

int64_t integer(PyObject* o) {
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}
// (an int argument of the C ABI: what does not fit would arrive as another number)
int small(PyObject* o) {
  const int64_t v = integer(o);
  if (v != (int)v) {
    PyErr_SetString(PyExc_OverflowError, "argument does not fit a C int");
    throw python_error();
  }
  return (int)v;
}
int as_int(int64_t v) {
  if (v != (int)v) check_status(BMX_ERR_SHAPE, "bmx");
  return (int)v;
}

// Python's lock is given back while this thread allocates or calls the library: either may wait for the GPU
// (room in a queue, the allocator's hipMalloc), and what the GPU waits for may need the lock (a host callback on the
// stream), as may every other Python thread.  0.04 us each time (a call that launches nothing 0.18 -> 0.22 us).
class Unlocked {
  PyThreadState* const state = PyEval_SaveThread();

 public:
  Unlocked() = default;
  ~Unlocked() { PyEval_RestoreThread(state); }
  Unlocked(const Unlocked&) = delete;
};

// A call of the library without Python's lock; its arguments are read with it.
template <class F, class... A>
void call(const char* what, F f, A... args) {
  int status;
  {
    const Unlocked unlocked;
    status = f(args...);
  }
  check_status(status, what);
}

hipStream_t stream_of(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject* h = PyObject_GetAttr(o, str_cuda_stream);
  if (!h) throw python_error();
  void* s = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (!s && PyErr_Occurred()) throw python_error();
  return (hipStream_t)s;
}

// The caller's output tensor, or a new one.
struct Out {
  at::Tensor made;
  T t = nullptr;
  PyObject* given = nullptr;
  Out(PyObject* o, at::ScalarType type, at::IntArrayRef shape, T like, const char* what, bool dense = false) {
    if (o == Py_None) {
      const Unlocked unlocked;
      made = at::Tensor(at::detail::empty_cuda(shape, type, like->device(), std::nullopt));
      t = &made;
    } else {
      t = dense ? tensor(o, type, what, true) : matrix(o, type, what);
      given = o;
    }
  }
  PyObject* result() {
    if (!given) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
  }
};

// A workspace: the caller's, or memory of the caching allocator held until the launches are enqueued
// (it goes back to the pool of the stream the kernels run on, which orders its next use).
struct Workspace {
  void* p = nullptr;
  size_t bytes = 0;
  bool mine = false;
  Workspace() = default;
  Workspace(const Workspace&) = delete;
  bool given(PyObject* o) {
    if (o == Py_None) return false;
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda() || !THPVariable_Unpack(o).is_contiguous()) {
      PyErr_SetString(PyExc_ValueError, "workspace must be a contiguous GPU tensor");
      throw python_error();
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    bytes = t.nbytes();
    p = bytes ? t.data_ptr() : (void*)16;  // (an empty one is a workspace that is too small, not none)
    return true;
  }
  void allocate(int op, std::initializer_list<int64_t> dims, T like, hipStream_t s) {
    bytes = bmx_workspace_bytes(op, dims.begin(), (int)dims.size());
    if (bytes == 0) return;  // nothing needed, or sizes that the call itself will refuse
    const c10::OptionalDeviceGuard guard(like->device());
    p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, s);
    mine = true;
  }
  ~Workspace() {
    if (mine) c10::hip::HIPCachingAllocator::raw_delete(p);
  }
};

// A call f(args..., workspace, its bytes, stream) whose workspace is allocated only if it asks for one.
template <class F, class... A>
void lazily(const char* what, PyObject* given, int op, std::initializer_list<int64_t> dims, T like, hipStream_t s, F f,
            A... args) {
  Workspace theirs;
  const bool has = theirs.given(given);
  call(what, [&] {
    const int status = f(args..., theirs.p, theirs.bytes, s);
    if (has || status != BMX_ERR_WORKSPACE) return status;
    Workspace ws;
    ws.allocate(op, dims, like, s);
    return f(args..., ws.p, ws.bytes, s);
  });
}

using Args = PyObject* const*;
#define FUNCTION(name, count)                                                    \
  PyObject* name##_(Args a);                                                     \
  PyObject* name(PyObject*, Args a, Py_ssize_t n) {                              \
    HANDLE_TH_ERRORS                                                             \
    if (n != count) {                                                            \
      PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments");     \
      throw python_error();                                                      \
    }                                                                            \
    return name##_(a);                                                           \
    END_HANDLE_TH_ERRORS                                                         \
  }                                                                              \
  PyObject* name##_(Args a)

int64_t words(int64_t k) { return (k + 63) / 64; }
bool truth(PyObject* o) { return o == Py_True || (o != Py_False && PyObject_IsTrue(o) == 1); }

FUNCTION(binarize_pack, 4) {  // x, pack_dim, out, stream
  T x = required(a[0], kF32, 2, "binarize_pack x");
  const int64_t rows = x->size(0), cols = x->size(1);
  const int dim = small(a[1]);
  Out out(a[2], kU64, {dim ? rows : cols, words(dim ? cols : rows)}, x, "binarize_pack out");
  const hipStream_t s = stream_of(a[3]);
  call("bmx_binarize_pack", bmx_binarize_pack, ptr<float>(x), rows, cols, ld(x), dim, ptr<uint64_t>(out.t), ld(out.t), s);
  return out.result();
}

FUNCTION(unpack_pm1, 4) {  // bits, K, out, stream
  T bits = matrix(a[0], kU64, "unpack_pm1 bits");
  const int64_t rows = bits->size(0), K = integer(a[1]);
  Out out(a[2], kF32, {rows, std::max<int64_t>(K, 0)}, bits, "unpack_pm1 out");
  const hipStream_t s = stream_of(a[3]);
  call("bmx_unpack_pm1", bmx_unpack_pm1, ptr<uint64_t>(bits), rows, K, ld(bits), ptr<float>(out.t), ld(out.t), s);
  return out.result();
}

FUNCTION(xnor_gemm, 6) {  // A, B, K, out, stream, count
  T A = matrix(a[0], kU64, "xnor_gemm A"), B = matrix(a[1], kU64, "xnor_gemm B");
  const int64_t M = A->size(0), N = B->size(0);
  Out out(a[3], kI32, {M, N}, A, "xnor_gemm out");
  const bool count = truth(a[5]);
  auto f = count ? bmx_xnor_gemm_count : bmx_xnor_gemm;
  const int K = small(a[2]);
  const hipStream_t s = stream_of(a[4]);
  call(count ? "bmx_xnor_gemm_count" : "bmx_xnor_gemm", f, ptr<uint64_t>(A), ld(A), ptr<uint64_t>(B), ld(B),
       ptr<int32_t>(out.t), ld(out.t), as_int(M), as_int(N), K, s);
  return out.result();
}

FUNCTION(widen_words32, 4) {  // rows32, K, out, stream
  T in = matrix(a[0], kI32, "widen_words32 rows32");
  const int64_t rows = in->size(0), K = integer(a[1]);
  Out out(a[2], kU64, {rows, std::max<int64_t>(words(K), 0)}, in, "widen_words32 out");
  const hipStream_t s = stream_of(a[3]);
  call("bmx_widen_words32", bmx_widen_words32, ptr<uint32_t>(in), rows, K, ld(in), ptr<uint64_t>(out.t), ld(out.t), s);
  return out.result();
}

FUNCTION(xnor_gemm_w32, 6) {  // A32, B32, K, out, workspace, stream
  T A = matrix(a[0], kI32, "xnor_gemm_w32 A"), B = matrix(a[1], kI32, "xnor_gemm_w32 B");
  const int64_t M = A->size(0), N = B->size(0);
  const int K = small(a[2]);
  Out out(a[3], kI32, {M, N}, A, "xnor_gemm_w32 out");
  const hipStream_t s = stream_of(a[5]);
  lazily("bmx_xnor_gemm_w32", a[4], BMX_OP_XNOR_GEMM_W32, {M, N, K}, A, s, bmx_lazy_xnor_gemm_w32, ptr<uint32_t>(A),
         ld(A), ptr<uint32_t>(B), ld(B), ptr<int32_t>(out.t), ld(out.t), as_int(M), as_int(N), K);
  return out.result();
}

FUNCTION(binary_fc, 7) {  // x, Wp, alpha, integer_out, out, workspace, stream
  T x = required(a[0], kF32, 2, "binary_fc x"), W = matrix(a[1], kU64, "binary_fc Wp");
  T alpha = tensor(a[2], kF32, "binary_fc alpha", true);
  const int64_t batch = x->size(0), fin = x->size(1), fout = W->size(0);
  const bool i32 = truth(a[3]);
  Out out(a[4], i32 ? kI32 : kF32, {batch, fout}, x, "binary_fc out");
  const hipStream_t s = stream_of(a[6]);
  lazily("bmx_binary_fc", a[5], BMX_OP_BINARY_FC, {batch, fin, fout}, x, s, bmx_lazy_binary_fc, ptr<float>(x), ld(x),
         ptr<uint64_t>(W), ld(W), ptr<float>(alpha), as_int(batch), as_int(fin), as_int(fout),
         i32 ? ptr<int32_t>(out.t) : nullptr, i32 ? nullptr : ptr<float>(out.t), ld(out.t));
  return out.result();
}

FUNCTION(binary_fc_static, 6) {  // x, Wp, alpha, integer_out, out, stream
  T x = required(a[0], kF32, 2, "binary_fc_static x"), W = matrix(a[1], kU64, "binary_fc_static Wp");
  T alpha = tensor(a[2], kF32, "binary_fc_static alpha", true);
  if (a[4] == Py_None) {
    PyErr_SetString(PyExc_ValueError, "binary_fc_static: pass the output tensor (the call allocates nothing)");
    throw python_error();
  }
  const bool i32 = truth(a[3]);
  T out = matrix(a[4], i32 ? kI32 : kF32, "binary_fc_static out");
  const hipStream_t s = stream_of(a[5]);
  call("bmx_binary_fc_static", bmx_binary_fc_static, ptr<float>(x), ld(x), ptr<uint64_t>(W), ld(W), ptr<float>(alpha),
       as_int(x->size(0)), as_int(x->size(1)), as_int(W->size(0)), i32 ? ptr<int32_t>(out) : nullptr,
       i32 ? nullptr : ptr<float>(out), ld(out), s);
  Py_INCREF(a[4]);
  return a[4];
}

FUNCTION(binary_fc_packed, 8) {  // xp, in_features, Wp, alpha, mode ("f32", "i32", "bits"), out, thr, stream
  T x = matrix(a[0], kU64, "binary_fc_packed xp"), W = matrix(a[2], kU64, "binary_fc_packed Wp");
  T alpha = tensor(a[3], kF32, "binary_fc_packed alpha", true), thr = tensor(a[6], kF32, "binary_fc_packed thr", true);
  const char* mode = PyUnicode_AsUTF8(a[4]);
  if (!mode) throw python_error();
  const bool i32 = !strcmp(mode, "i32"), bits = !strcmp(mode, "bits");
  if (!i32 && !bits && strcmp(mode, "f32")) {
    PyErr_SetObject(PyExc_KeyError, a[4]);
    throw python_error();
  }
  const int64_t batch = x->size(0), fout = W->size(0);
  Out out(a[5], bits ? kU64 : i32 ? kI32 : kF32, {batch, bits ? words(fout) : fout}, x, "binary_fc_packed out");
  const int K = small(a[1]);
  const hipStream_t s = stream_of(a[7]);
  call("bmx_binary_fc_packed", bmx_binary_fc_packed, ptr<uint64_t>(x), ld(x), ptr<uint64_t>(W), ld(W), ptr<float>(alpha),
       as_int(batch), K, as_int(fout), i32 ? ptr<int32_t>(out.t) : nullptr, !i32 && !bits ? ptr<float>(out.t) : nullptr,
       bits ? ptr<uint64_t>(out.t) : nullptr, ptr<float>(thr), ld(out.t), s);
  return out.result();
}

FUNCTION(pack_conv_weights, 2) {  // w, stream
  T w = required(a[0], kF32, 4, "pack_conv_weights w", true);
  const int O = as_int(w->size(0)), C = as_int(w->size(1)), KH = as_int(w->size(2)), KW = as_int(w->size(3));
  const int64_t row = bmx_conv_weight_row_words(C, KH, KW);
  if (row <= 0) check_status(BMX_ERR_UNSUPPORTED, "bmx_conv_weight_row_words");
  Out out(Py_None, kU64, {O, row}, w, "");
  const hipStream_t s = stream_of(a[1]);
  call("bmx_pack_conv_weights", bmx_pack_conv_weights, ptr<float>(w), O, C, KH, KW, ptr<uint64_t>(out.t), s);
  return out.result();
}

int64_t conv_out(int64_t n, int k, int stride, int pad) {
  return std::max<int64_t>(0, stride > 0 ? (n + 2 * pad - k) / stride + 1 : 0);
}

FUNCTION(binary_conv2d, 12) {  // x, Wp, O, KH, KW, stride, pad, alpha, integer_out, out, workspace, stream
  T x = required(a[0], kF32, 4, "binary_conv2d x", true), W = tensor(a[1], kU64, "binary_conv2d Wp", true);
  T alpha = tensor(a[7], kF32, "binary_conv2d alpha", true);
  const int64_t N = x->size(0), C = x->size(1), H = x->size(2), Wd = x->size(3);
  const int O = small(a[2]), KH = small(a[3]), KW = small(a[4]), stride = small(a[5]), pad = small(a[6]);
  const bool i32 = truth(a[8]);
  Out out(a[9], i32 ? kI32 : kF32, {N, std::max(O, 0), conv_out(H, KH, stride, pad), conv_out(Wd, KW, stride, pad)}, x,
          "binary_conv2d out", true);
  const hipStream_t s = stream_of(a[11]);
  lazily("bmx_binary_conv2d", a[10], BMX_OP_BINARY_CONV2D, {N, C, H, Wd, O, KH, KW, stride, pad}, x, s,
         bmx_lazy_binary_conv2d, ptr<float>(x), as_int(N), as_int(C), as_int(H), as_int(Wd), ptr<uint64_t>(W), O, KH, KW,
         stride, pad, ptr<float>(alpha), i32 ? ptr<int32_t>(out.t) : nullptr, i32 ? nullptr : ptr<float>(out.t));
  return out.result();
}

FUNCTION(pack_nchw, 4) {  // x, pad, out, stream
  T x = required(a[0], kF32, 4, "pack_nchw x", true);
  const int64_t N = x->size(0), C = x->size(1), H = x->size(2), Wd = x->size(3);
  const int pad = small(a[1]);
  Out out(a[2], kU64, {N, std::max<int64_t>(H + 2 * pad, 0), std::max<int64_t>(Wd + 2 * pad, 0), words(C)}, x,
          "pack_nchw out", true);
  const hipStream_t s = stream_of(a[3]);
  call("bmx_pack_nchw", bmx_pack_nchw, ptr<float>(x), as_int(N), as_int(C), as_int(H), as_int(Wd), pad,
       ptr<uint64_t>(out.t), s);
  return out.result();
}

FUNCTION(binary_conv2d_packed, 12) {  // xp, C, Wp, O, KH, KW, stride, pad, alpha, integer_out, out, stream
  T x = packed_image(a[0], "binary_conv2d_packed xp"), W = tensor(a[2], kU64, "binary_conv2d_packed Wp", true);
  T alpha = tensor(a[8], kF32, "binary_conv2d_packed alpha", true);
  const int C = small(a[1]), O = small(a[3]), KH = small(a[4]), KW = small(a[5]), stride = small(a[6]), pad = small(a[7]);
  const int64_t N = x->size(0), H = x->size(1) - 2 * (int64_t)pad, Wd = x->size(2) - 2 * (int64_t)pad;
  const bool i32 = truth(a[9]);
  Out out(a[10], i32 ? kI32 : kF32, {N, std::max(O, 0), conv_out(H, KH, stride, pad), conv_out(Wd, KW, stride, pad)}, x,
          "binary_conv2d_packed out", true);
  const hipStream_t s = stream_of(a[11]);
  call("bmx_binary_conv2d_packed", bmx_binary_conv2d_packed, ptr<uint64_t>(x), as_int(N), C, as_int(H), as_int(Wd),
       ptr<uint64_t>(W), O, KH, KW, stride, pad, ptr<float>(alpha), i32 ? ptr<int32_t>(out.t) : nullptr,
       i32 ? nullptr : ptr<float>(out.t), s);
  return out.result();
}

// xp, C, Wp, O, KH, KW, stride, pad, alpha, thr, out_pad, out, workspace, stream
FUNCTION(binary_conv2d_bits, 14) {
  T x = packed_image(a[0], "binary_conv2d_bits xp"), W = tensor(a[2], kU64, "binary_conv2d_bits Wp", true);
  T alpha = tensor(a[8], kF32, "binary_conv2d_bits alpha", true), thr = tensor(a[9], kF32, "binary_conv2d_bits thr", true);
  const int C = small(a[1]), O = small(a[3]), KH = small(a[4]), KW = small(a[5]), stride = small(a[6]), pad = small(a[7]);
  const int opad = small(a[10]);
  const int64_t N = x->size(0), H = x->size(1) - 2 * (int64_t)pad, Wd = x->size(2) - 2 * (int64_t)pad;
  const int64_t ho = conv_out(H, KH, stride, pad) + 2 * (int64_t)opad, wo = conv_out(Wd, KW, stride, pad) + 2 * (int64_t)opad;
  Out out(a[11], kU64, {N, std::max<int64_t>(ho, 0), std::max<int64_t>(wo, 0), std::max<int64_t>(words(O), 0)}, x,
          "binary_conv2d_bits out", true);
  const hipStream_t s = stream_of(a[13]);
  lazily("bmx_binary_conv2d_bits", a[12], BMX_OP_BINARY_CONV2D_BITS, {N, C, H, Wd, O, KH, KW, stride, pad, opad}, x, s,
         bmx_lazy_binary_conv2d_bits, ptr<uint64_t>(x), as_int(N), C, as_int(H), as_int(Wd), ptr<uint64_t>(W), O, KH, KW,
         stride, pad, ptr<float>(alpha), ptr<float>(thr), ptr<uint64_t>(out.t), opad);
  return out.result();
}

// a, w, bits_a, bits_w, want_int, want_float, out_int, out_float, workspace, stream -> (int, float)
FUNCTION(quant_gemm, 10) {
  T x = required(a[0], kF32, 2, "quant_gemm a"), w = matrix(a[1], kF32, "quant_gemm w");
  const int64_t M = x->size(0), K = x->size(1), N = w->size(0);
  const int bits_a = small(a[2]), bits_w = small(a[3]);
  std::optional<Out> S, F;
  if (a[6] != Py_None || truth(a[4])) S.emplace(a[6], kI32, at::IntArrayRef({M, N}), x, "quant_gemm out_int");
  if (a[7] != Py_None || truth(a[5])) F.emplace(a[7], kF32, at::IntArrayRef({M, N}), x, "quant_gemm out_float");
  if (!S && !F) check_status(BMX_ERR_NULL, "bmx_quant_gemm");
  const int64_t ldo = ld(S ? S->t : F->t);
  if (S && F && ld(F->t) != ldo) {
    PyErr_SetString(PyExc_ValueError, "quant_gemm: out_int and out_float must share one row stride");
    throw python_error();
  }
  const hipStream_t s = stream_of(a[9]);
  lazily("bmx_quant_gemm", a[8], BMX_OP_QUANT_GEMM, {M, N, K, bits_a, bits_w}, x, s, bmx_lazy_quant_gemm, ptr<float>(x),
         ld(x), bits_a, ptr<float>(w), ld(w), bits_w, as_int(M), as_int(N), as_int(K), S ? ptr<int32_t>(S->t) : nullptr,
         F ? ptr<float>(F->t) : nullptr, ldo);
  PyObject* r = PyTuple_New(2);
  if (!r) throw python_error();
  for (int i = 0; i < 2; ++i) {
    std::optional<Out>& o = i ? F : S;
    PyObject* v = o ? o->result() : nullptr;
    if (!o) Py_INCREF(v = Py_None);
    PyTuple_SET_ITEM(r, i, v);
  }
  return r;
}

FUNCTION(alpha_mean_abs, 2) {  // w, stream
  T w = tensor(a[0], kF32, "alpha_mean_abs w", true);
  if (!w || w->dim() < 1) raise_value("%s: expected a tensor of at least one dimension%s%s", "alpha_mean_abs w");
  const int64_t rows = w->size(0), cols = w->numel() / std::max<int64_t>(rows, 1);
  Out out(Py_None, kF32, {rows}, w, "");
  const hipStream_t s = stream_of(a[1]);
  call("bmx_alpha_mean_abs", bmx_alpha_mean_abs, ptr<float>(w), rows, cols, cols, ptr<float>(out.t), s);
  return out.result();
}

PyObject* set_error(PyObject*, PyObject* cls) {
  Py_INCREF(cls);
  Py_XDECREF(bmx_error);
  bmx_error = cls;
  Py_RETURN_NONE;
}

#define ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(binarize_pack), ENTRY(unpack_pm1), ENTRY(xnor_gemm), ENTRY(widen_words32),
                         ENTRY(xnor_gemm_w32), ENTRY(binary_fc), ENTRY(binary_fc_static), ENTRY(binary_fc_packed),
                         ENTRY(pack_conv_weights), ENTRY(binary_conv2d), ENTRY(pack_nchw), ENTRY(binary_conv2d_packed),
                         ENTRY(binary_conv2d_bits), ENTRY(quant_gemm), ENTRY(alpha_mean_abs),
                         {"set_error", set_error, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bmx_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__bmx_host() {
  str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return str_cuda_stream ? PyModule_Create(&module) : nullptr;
}
