// The host side of the binding's frequent calls: allocation of the outputs and the call of the C entry point, without the
// Python objects in between.  A host-bound program (small operands, the decode stage) spends its time here: a torch.empty takes
// 1.4 us from Python and 0.3 from here, the marshalling of ten arguments through ctypes 0.7; us a call, host-bound, before -> now:
// quantize of 16 x 256 10.3 -> 4.4, dequantize 7.2 -> 3.9, gemm_bf16a of 8 x 4096 x 4096 (two launches) 13.0 -> 6.3.  About 3 us
// of each is a kernel launch.
//
// Every function takes the common case only and returns None for anything else -- another tensor type, layout or dtype, an argument
// that the C entry point refuses -- before it has launched anything; the caller then goes through its general code, which raises.
#include <torch/extension.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <cstdint>
#include "mxp.h"

namespace {

struct Entry {
  decltype(&mxp_quantize) quantize;
  decltype(&mxp_dequantize) dequantize;
  decltype(&mxp_gemm) gemm;
  decltype(&mxp_gemm_workspace_bytes_fmt) gemm_ws;
  decltype(&mxp_gemm_bf16a) bf16a;
  decltype(&mxp_gemm_bf16a_workspace_bytes) bf16a_ws;
  decltype(&mxp_gemm_decode_bf16a) decode_bf16a;
  decltype(&mxp_gemm_w4a16_ws) w4a16;
  decltype(&mxp_gemm_w4a16_workspace_bytes) w4a16_ws;
} lib = {};

// a plain CUDA tensor, or nullptr
const at::Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() ? &t : nullptr;
}
// fp32 / bf16 rows with unit inner stride: the dtype code, or -1
int rows_dtype(const at::Tensor* t) {
  if (!t || t->dim() != 2 || t->stride(1) != 1) return -1;
  return t->scalar_type() == at::kFloat ? MXP_F32 : t->scalar_type() == at::kBFloat16 ? MXP_BF16 : -1;
}
int64_t ld(const at::Tensor& t) { return t.size(0) > 1 ? t.stride(0) : std::max<int64_t>(t.size(1), 1); }
int64_t code_bits(int64_t fmt) { return fmt < MXP_FMT_MXFP6 ? 4 : fmt < MXP_FMT_MXFP8 ? 6 : 8; }

struct Quantized {                                           // (elems, scales, idx), idx possibly None
  const at::Tensor *el = nullptr, *sc = nullptr;
  uint8_t* ix = nullptr;
  bool take(PyObject* q) {
    if (!PyTuple_CheckExact(q) || PyTuple_GET_SIZE(q) != 3) return false;
    el = tensor(PyTuple_GET_ITEM(q, 0));
    sc = tensor(PyTuple_GET_ITEM(q, 1));
    if (!el || !sc || el->dim() != 2 || sc->dim() != 2) return false;
    PyObject* i = PyTuple_GET_ITEM(q, 2);
    if (i == Py_None) return true;
    const at::Tensor* t = tensor(i);
    if (t) ix = static_cast<uint8_t*>(t->data_ptr());
    return t != nullptr;
  }
  const uint8_t* e() const { return static_cast<const uint8_t*>(el->data_ptr()); }
  const uint8_t* s() const { return static_cast<const uint8_t*>(sc->data_ptr()); }
};

at::Tensor bytes(const at::Tensor& like, at::IntArrayRef size) { return at::empty(size, at::TensorOptions().dtype(at::kByte).device(like.device())); }
at::Tensor output(const at::Tensor& like, int64_t M, int64_t N, int64_t d) {
  return at::empty({M, N}, at::TensorOptions().dtype(d == MXP_BF16 ? at::kBFloat16 : at::kFloat).device(like.device()));
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
int64_t integer(PyObject* o) { return PyLong_AsLongLong(o); }

// `n` arguments, those from `first` on integers of 64 bits (a longer one would leave an error set)
bool arguments(PyObject* const* a, Py_ssize_t given, Py_ssize_t n, Py_ssize_t first) {
  if (given != n) return false;
  for (Py_ssize_t i = first; i < n; ++i) {
    int overflow = 0;
    if (!PyLong_CheckExact(a[i]) || (PyLong_AsLongLongAndOverflow(a[i], &overflow), overflow != 0)) return false;
  }
  return true;
}
template <class F>
int unlocked(F&& f) {
  pybind11::gil_scoped_release release;
  return f();
}

PyObject* fast_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void** slots = reinterpret_cast<void**>(&lib);
  if (n != (Py_ssize_t)(sizeof(lib) / sizeof(void*))) {
    PyErr_SetString(PyExc_TypeError, "one address per entry point");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) slots[i] = PyLong_AsVoidPtr(a[i]);
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

PyObject* fast_quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {   // x, fmt
  HANDLE_TH_ERRORS
  const at::Tensor* x = arguments(a, n, 2, 1) ? tensor(a[0]) : nullptr;
  const int dt = rows_dtype(x);
  if (dt < 0) Py_RETURN_NONE;
  const int64_t rows = x->size(0), K = x->size(1), fmt = integer(a[1]);
  if (K % 32 != 0 || fmt < MXP_FMT_MXFP4 || fmt > MXP_FMT_MXFP8P) Py_RETURN_NONE;
  at::Tensor e = bytes(*x, {rows, K * code_bits(fmt) / 8}), s = bytes(*x, {rows, K / 32}), i = bytes(*x, {rows, K / 32});
  if (unlocked([&] {
        return lib.quantize(x->data_ptr(), dt, rows, K, ld(*x), (int)fmt, static_cast<uint8_t*>(e.data_ptr()), static_cast<uint8_t*>(s.data_ptr()),
                            static_cast<uint8_t*>(i.data_ptr()), stream());
      }) != MXP_OK)
    Py_RETURN_NONE;
  PyObject* out = PyTuple_New(3);
  if (!out) return nullptr;
  PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(std::move(e)));
  PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(std::move(s)));
  PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(std::move(i)));
  return out;
  END_HANDLE_TH_ERRORS
}

PyObject* fast_dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {   // q, fmt, dtype code
  HANDLE_TH_ERRORS
  Quantized q;
  if (!arguments(a, n, 3, 1) || !q.take(a[0])) Py_RETURN_NONE;
  const int64_t fmt = integer(a[1]), d = integer(a[2]);
  if (fmt < MXP_FMT_MXFP4 || fmt > MXP_FMT_MXFP8P) Py_RETURN_NONE;
  const int64_t rows = q.el->size(0), K = q.el->size(1) * 8 / code_bits(fmt);
  at::Tensor out = output(*q.el, rows, K, d);
  if (unlocked([&] { return lib.dequantize(q.e(), q.s(), q.ix, (int)fmt, rows, K, out.data_ptr(), (int)d, std::max<int64_t>(K, 1), stream()); }) != MXP_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
  END_HANDLE_TH_ERRORS
}

PyObject* fast_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {   // qa, qb, fmt_a, fmt_b, dtype code
  HANDLE_TH_ERRORS
  Quantized qa, qb;
  if (!arguments(a, n, 5, 2) || !qa.take(a[0]) || !qb.take(a[1])) Py_RETURN_NONE;
  const int64_t fa = integer(a[2]), fb = integer(a[3]), d = integer(a[4]);
  const int64_t M = qa.el->size(0), K = qa.sc->size(1) * 32, N = qb.el->size(0);
  if (qb.sc->size(1) * 32 != K) Py_RETURN_NONE;
  at::Tensor out = output(*qa.el, M, N, d);
  at::Tensor ws = bytes(*qa.el, {std::max<int64_t>((int64_t)lib.gemm_ws(M, N, K, (int)fa, (int)fb), 16)});
  if (unlocked([&] {
        return lib.gemm(M, N, K, qa.e(), qa.s(), qa.ix, (int)fa, qb.e(), qb.s(), qb.ix, (int)fb, out.data_ptr(), (int)d, std::max<int64_t>(N, 1),
                        ws.data_ptr(), (size_t)ws.numel(), stream());
      }) != MXP_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
  END_HANDLE_TH_ERRORS
}

PyObject* fast_gemm_bf16a(PyObject*, PyObject* const* a, Py_ssize_t n) {   // activations, image, fmt_a (not MXFP4++), N, dtype code, image kind
  HANDLE_TH_ERRORS
  if (!arguments(a, n, 6, 2)) Py_RETURN_NONE;
  const at::Tensor *x = tensor(a[0]), *img = tensor(a[1]);
  const int dt = rows_dtype(x);
  if (dt < 0 || !img) Py_RETURN_NONE;
  const int64_t fa = integer(a[2]), N = integer(a[3]), d = integer(a[4]), kind = integer(a[5]), M = x->size(0), K = x->size(1);
  if (N < 0 || K % 32 != 0) Py_RETURN_NONE;
  at::Tensor out = output(*x, M, N, d);
  at::Tensor ws = bytes(*x, {std::max<int64_t>((int64_t)lib.bf16a_ws(M, K), 16)});
  if (unlocked([&] {
        return lib.bf16a(M, N, K, x->data_ptr(), dt, ld(*x), (int)fa, img->data_ptr(), (int)kind, out.data_ptr(), (int)d, std::max<int64_t>(N, 1),
                         ws.data_ptr(), (size_t)ws.numel(), stream());
      }) != MXP_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
  END_HANDLE_TH_ERRORS
}

PyObject* fast_gemm_decode_bf16a(PyObject*, PyObject* const* a, Py_ssize_t n) {   // activations, qw, fmt_a, fmt_w, dtype code
  HANDLE_TH_ERRORS
  Quantized w;
  if (!arguments(a, n, 5, 2) || !w.take(a[1])) Py_RETURN_NONE;
  const at::Tensor* x = tensor(a[0]);
  const int dt = rows_dtype(x);
  if (dt < 0) Py_RETURN_NONE;
  const int64_t fa = integer(a[2]), fw = integer(a[3]), d = integer(a[4]), M = x->size(0), K = x->size(1), N = w.el->size(0);
  if (K % 32 != 0) Py_RETURN_NONE;
  at::Tensor out = output(*x, M, N, d);
  at::Tensor ws = bytes(*x, {std::max<int64_t>((int64_t)lib.bf16a_ws(M, K), 16)});
  if (unlocked([&] {
        return lib.decode_bf16a(M, N, K, x->data_ptr(), dt, ld(*x), (int)fa, w.e(), w.s(), w.ix, (int)fw, out.data_ptr(), (int)d, std::max<int64_t>(N, 1),
                                ws.data_ptr(), (size_t)ws.numel(), stream());
      }) != MXP_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
  END_HANDLE_TH_ERRORS
}

PyObject* fast_gemm_w4a16(PyObject*, PyObject* const* a, Py_ssize_t n) {   // activations, qw, fmt_w, dtype code
  HANDLE_TH_ERRORS
  Quantized w;
  if (!arguments(a, n, 4, 2) || !w.take(a[1])) Py_RETURN_NONE;
  const at::Tensor* x = tensor(a[0]);
  const int dt = rows_dtype(x);
  if (dt < 0) Py_RETURN_NONE;
  const int64_t fw = integer(a[2]), d = integer(a[3]), M = x->size(0), K = x->size(1), N = w.el->size(0);
  if (w.sc->size(1) * 32 != K) Py_RETURN_NONE;
  at::Tensor out = output(*x, M, N, d), ws;
  const int64_t need = (int64_t)lib.w4a16_ws(M, N, K, (int)fw);
  if (need > 0) {
    try {
      ws = bytes(*x, {need});
    } catch (const c10::OutOfMemoryError&) {                 // room that the call can do without
      ws = at::Tensor();
    }
  }
  if (unlocked([&] {
        return lib.w4a16(M, N, K, x->data_ptr(), dt, ld(*x), w.e(), w.s(), w.ix, (int)fw, out.data_ptr(), (int)d, std::max<int64_t>(N, 1),
                         ws.defined() ? ws.data_ptr() : nullptr, ws.defined() ? (size_t)need : 0, stream());
      }) != MXP_OK)
    Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(out));
  END_HANDLE_TH_ERRORS
}

#define MXP_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fast_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MXP_METHOD(init),      MXP_METHOD(quantize),          MXP_METHOD(dequantize), MXP_METHOD(gemm),
                         MXP_METHOD(gemm_bf16a), MXP_METHOD(gemm_decode_bf16a), MXP_METHOD(gemm_w4a16), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mxp_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mxp_binding() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", MXP_TORCH_VERSION) != 0) Py_CLEAR(m);   // of the headers it was compiled with
  return m;
}
