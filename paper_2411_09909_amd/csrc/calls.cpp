// The calls of a serving loop - casts and products into buffers that the caller keeps - without the interpreter and ctypes
// between torch and the C ABI: tensors are taken apart here, and the call made, in 0.3 us instead of 1.8 to 2.9 (a kernel
// launch through the runtime takes 2.3 to 2.9 us itself; a cast and a product of 64 x 1024 x 1024 among others: 11.3 -> 8.2 us, of
// which the kernels and the gaps between them are 6.5).
// Every function returns the status of the C call, or None for arguments that it does not take as they are (buffers to be
// allocated, anything that is not a plain tensor on the GPU, wrong dimensions); binding.py then goes its general way, which
// also says what is wrong with them.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include "../../include/amxfp4.h"

namespace {

// Entry points by address, from the library that binding.py has loaded (bind()).
struct {
  decltype(&amxfp4_quantize) quantize;
  decltype(&amxfp4_quantize_scaled) quantize_scaled;
  decltype(&amxfp4_quantize_batched) quantize_batched;
  decltype(&amxfp4_tensor_scale) tensor_scale;
  decltype(&amxfp4_gemm) gemm;
  decltype(&amxfp4_gemm_scaled) gemm_scaled;
  decltype(&amxfp4_gemm_prepared) gemm_prepared;
  decltype(&amxfp4_attention) attention;
  decltype(&amxfp4_attention_merged) attention_merged;
  decltype(&amxfp4_attention_decode) attention_decode;
} entry;
constexpr const char* kEntries[] = {"amxfp4_quantize", "amxfp4_quantize_scaled", "amxfp4_quantize_batched", "amxfp4_tensor_scale",
                                    "amxfp4_gemm", "amxfp4_gemm_scaled", "amxfp4_gemm_prepared", "amxfp4_attention",
                                    "amxfp4_attention_merged", "amxfp4_attention_decode"};
constexpr size_t kNumEntries = sizeof(kEntries) / sizeof(kEntries[0]);
static_assert(sizeof(entry) == kNumEntries * sizeof(void*), "one name per entry point");

// A plain tensor (torch.Tensor or Parameter itself, no subclass with ways of its own) on the GPU, or null.
const at::Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() ? &t : nullptr;
}

// The first n arguments from `from` on as such tensors; contiguous: all of them.
bool tensors(PyObject* const* args, int from, int n, const at::Tensor** out, bool contiguous) {
  for (int i = 0; i < n; ++i)
    if (!(out[i] = tensor(args[from + i])) || (contiguous && !out[i]->is_contiguous())) return false;
  return true;
}

uint8_t* bytes(const at::Tensor* t) { return static_cast<uint8_t*>(t->data_ptr()); }
size_t size_of(const at::Tensor* t) { return (size_t)t->numel() * t->element_size(); }

// a tensor-scale pair: a contiguous float32 tensor of two elements or more
const at::Tensor* pair(PyObject* o) {
  const at::Tensor* t = tensor(o);
  return t && t->scalar_type() == at::kFloat && t->numel() >= 2 && t->is_contiguous() ? t : nullptr;
}

// The format, out of its ctypes structure (the class given to bind(), or one derived from it: other structures and bytes of the
// same size are no formats).
PyTypeObject* format_type = nullptr;
bool format(PyObject* o, amx_format_t& f) {
  if (!format_type || !PyObject_TypeCheck(o, format_type)) return false;
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = view.len == (Py_ssize_t)sizeof(f);
  if (ok) memcpy(&f, view.buf, sizeof(f));
  PyBuffer_Release(&view);
  return ok;
}

// Runs the C call with the interpreter released, on the current stream of the current device.
template <class Call>
PyObject* run(Call call) {
  int status;
  void* stream = c10::hip::getCurrentHIPStream().stream();
  Py_BEGIN_ALLOW_THREADS;
  status = call(stream);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(status);
}

// quantize(fmt, x, along_rows, codes, scales, tensor_pair or None)
PyObject* quantize(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor *x, *out[2], *p = nullptr;
  if (n != 6 || !format(args[0], f) || !(x = tensor(args[1])) || x->dim() != 2 || x->element_size() != 2 ||
      !tensors(args, 3, 2, out, false) || (args[5] != Py_None && !(p = pair(args[5]))))
    Py_RETURN_NONE;
  const int r = args[2] == Py_True ? 0 : 1;  // the dimension of x that holds the rows
  const int64_t rows = x->size(r), K = x->size(1 - r), row_stride = x->stride(r), k_stride = x->stride(1 - r);
  const void* from = x->data_ptr();
  uint8_t *codes = bytes(out[0]), *scales = bytes(out[1]);
  const float* ratio = p ? static_cast<const float*>(p->data_ptr()) : nullptr;
  return run([&](void* s) {
    return ratio ? entry.quantize_scaled(&f, from, rows, K, row_stride, k_stride, ratio, codes, scales, s)
                 : entry.quantize(&f, from, rows, K, row_stride, k_stride, codes, scales, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// quantize_batched(fmt, x, along_rows, codes, scales)
PyObject* quantize_batched(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor *x, *out[2];
  if (n != 5 || !format(args[0], f) || !(x = tensor(args[1])) || x->dim() != 3 || x->element_size() != 2 ||
      !tensors(args, 3, 2, out, false))
    Py_RETURN_NONE;
  const int r = args[2] == Py_True ? 1 : 2;
  const int64_t batch = x->size(0), batch_stride = x->stride(0), rows = x->size(r), K = x->size(3 - r);
  const int64_t row_stride = x->stride(r), k_stride = x->stride(3 - r);
  const void* from = x->data_ptr();
  uint8_t *codes = bytes(out[0]), *scales = bytes(out[1]);
  return run([&](void* s) {
    return entry.quantize_batched(&f, from, batch, batch_stride, rows, K, row_stride, k_stride, codes, scales, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// tensor_scale(x, out)
PyObject* tensor_scale(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  const at::Tensor *x, *out;
  if (n != 2 || !(x = tensor(args[0])) || !(out = tensor(args[1])) || x->dim() != 2 || x->element_size() != 2 || x->stride(1) != 1)
    Py_RETURN_NONE;
  const void* from = x->data_ptr();
  float* to = static_cast<float*>(out->data_ptr());
  return run([&](void* s) { return entry.tensor_scale(from, x->size(0), x->size(1), x->stride(0), to, s); });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// gemm(fmt, a_codes, a_scales, b_codes, b_scales, out, workspace, a_pair or None, b_pair or None)
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor *t[4], *to[2], *pa = nullptr, *pb = nullptr;
  if (n != 9 || !format(args[0], f) || !tensors(args, 1, 4, t, true) || !tensors(args, 5, 2, to, false)) Py_RETURN_NONE;
  const bool scaled = args[7] != Py_None || args[8] != Py_None;
  if (scaled && (!(pa = pair(args[7])) || !(pb = pair(args[8])))) Py_RETURN_NONE;
  if ((t[0]->dim() != 2 && t[0]->dim() != 3) || t[2]->dim() < 2 || to[0]->dim() < 2) Py_RETURN_NONE;
  const int64_t batch = t[0]->dim() == 3 ? t[0]->size(0) : 1, M = t[0]->size(-2), K = t[0]->size(-1) * 2, N = t[2]->size(-2);
  const int64_t ldc = to[0]->stride(-2);
  uint8_t *ac = bytes(t[0]), *as = bytes(t[1]), *bc = bytes(t[2]), *bs = bytes(t[3]), *ws = bytes(to[1]);
  float *c = static_cast<float*>(to[0]->data_ptr()), *ra = nullptr, *rb = nullptr;
  if (scaled) ra = static_cast<float*>(pa->data_ptr()), rb = static_cast<float*>(pb->data_ptr());
  const size_t ws_bytes = size_of(to[1]);
  return run([&](void* s) {
    return scaled ? entry.gemm_scaled(&f, M, N, K, ac, as, ra, bc, bs, rb, c, ldc, batch, ws, ws_bytes, s)
                  : entry.gemm(&f, M, N, K, ac, as, bc, bs, c, ldc, batch, ws, ws_bytes, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// gemm_prepared(fmt, a_codes, a_scales, b_codes, b_scales, prepared, out, workspace)
PyObject* gemm_prepared(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor* t[7];
  if (n != 8 || !format(args[0], f) || !tensors(args, 1, 7, t, false)) Py_RETURN_NONE;
  if (t[0]->dim() != 2 || t[2]->dim() < 1 || t[5]->dim() < 2) Py_RETURN_NONE;
  const int64_t M = t[0]->size(0), K = t[0]->size(1) * 2, N = t[2]->size(0), ldc = t[5]->stride(-2);
  uint8_t *ac = bytes(t[0]), *as = bytes(t[1]), *bc = bytes(t[2]), *bs = bytes(t[3]), *ws = bytes(t[6]);
  const size_t prepared_bytes = size_of(t[4]), ws_bytes = size_of(t[6]);
  void* prepared = prepared_bytes ? t[4]->data_ptr() : nullptr;
  float* c = static_cast<float*>(t[5]->data_ptr());
  return run([&](void* s) {
    return entry.gemm_prepared(&f, M, N, K, ac, as, bc, bs, prepared, prepared_bytes, c, ldc, ws, ws_bytes, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// q_codes [Hq, Sq, D/2], .., k_codes [Hkv, Sk, D/2], .., v_codes [Hkv, D, Sk/2], ..: whether the shapes go together
bool heads(const at::Tensor* const* t) {
  return t[0]->dim() == 3 && t[2]->dim() == 3 && t[4]->dim() == 3 && t[2]->size(2) == t[0]->size(2) && t[4]->size(0) == t[2]->size(0) &&
         t[4]->size(1) == 2 * t[0]->size(2) && t[4]->size(2) == t[2]->size(1) / 2;
}

// attention(fmt, q_codes, q_scales, k_codes, k_scales, v_codes, v_scales, scale, causal, out, workspace, merged)
PyObject* attention(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor *t[6], *to[2];
  if (n != 12 || !format(args[0], f) || !tensors(args, 1, 6, t, true) || !heads(t) || !tensors(args, 9, 2, to, false) ||
      !PyFloat_CheckExact(args[7]))
    Py_RETURN_NONE;
  const bool merged = args[11] == Py_True, causal = args[8] == Py_True;
  if (!to[0]->is_contiguous() || to[0]->scalar_type() != (merged ? at::kBFloat16 : at::kFloat)) Py_RETURN_NONE;
  const int64_t Hq = t[0]->size(0), Sq = t[0]->size(1), D = t[0]->size(2) * 2, Hkv = t[2]->size(0), Sk = t[2]->size(1);
  uint8_t* p[6];
  for (int i = 0; i < 6; ++i) p[i] = bytes(t[i]);
  const float scale = (float)PyFloat_AS_DOUBLE(args[7]);
  float* out = static_cast<float*>(to[0]->data_ptr());
  uint8_t* ws = bytes(to[1]);
  const size_t ws_bytes = size_of(to[1]);
  return run([&](void* s) {
    return merged ? entry.attention_merged(&f, Hq, Hkv, Sq, Sk, D, p[0], p[1], p[2], p[3], p[4], p[5], scale, causal,
                                           reinterpret_cast<uint16_t*>(out), ws, ws_bytes, s)
                  : entry.attention(&f, Hq, Hkv, Sq, Sk, D, p[0], p[1], p[2], p[3], p[4], p[5], scale, causal, out, ws, ws_bytes, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// attention_decode(fmt, q_codes, q_scales, k_codes, k_scales, v_codes, v_scales, scale, causal, key_splits, out, workspace)
PyObject* attention_decode(PyObject*, PyObject* const* args, Py_ssize_t n) try {
  amx_format_t f;
  const at::Tensor *t[6], *to[2];
  if (n != 12 || !format(args[0], f) || !tensors(args, 1, 6, t, true) || !heads(t) || !tensors(args, 10, 2, to, false) ||
      !PyFloat_CheckExact(args[7]) || !PyLong_CheckExact(args[9]))
    Py_RETURN_NONE;
  const long long splits = PyLong_AsLongLong(args[9]);
  if (splits == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const int64_t Hq = t[0]->size(0), Sq = t[0]->size(1), D = t[0]->size(2) * 2, Hkv = t[2]->size(0), Sk = t[2]->size(1);
  uint8_t* p[6];
  for (int i = 0; i < 6; ++i) p[i] = bytes(t[i]);
  const float scale = (float)PyFloat_AS_DOUBLE(args[7]);
  const bool causal = args[8] == Py_True;
  float* out = static_cast<float*>(to[0]->data_ptr());
  uint8_t* ws = bytes(to[1]);
  const size_t ws_bytes = size_of(to[1]);
  return run([&](void* s) {
    return entry.attention_decode(&f, Hq, Hkv, Sq, Sk, D, p[0], p[1], p[2], p[3], p[4], p[5], scale, causal, splits, out, ws, ws_bytes, s);
  });
} catch (const std::exception&) {
  Py_RETURN_NONE;
}

// bind(class of the formats, address of each of `entries`)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* address[kNumEntries];
  if (n != (Py_ssize_t)kNumEntries + 1 || !PyType_Check(args[0]))
    return PyErr_Format(PyExc_TypeError, "bind: a class and %zu addresses", kNumEntries);
  for (size_t i = 0; i < kNumEntries; ++i) {
    address[i] = PyLong_AsVoidPtr(args[i + 1]);
    if (!address[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "bind: %s is null", kEntries[i]);
  }
  memcpy(&entry, address, sizeof(address));
  Py_INCREF(args[0]);
  PyTypeObject* before = format_type;
  format_type = reinterpret_cast<PyTypeObject*>(args[0]);
  Py_XDECREF(before);
  Py_RETURN_NONE;
}

#define CALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {CALL(quantize), CALL(quantize_batched), CALL(tensor_scale), CALL(gemm), CALL(gemm_prepared),
                          CALL(attention), CALL(attention_decode), CALL(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  PyObject* m = PyModule_Create(&kModule);
  PyObject* names = m ? PyTuple_New(kNumEntries) : nullptr;
  for (size_t i = 0; names && i < kNumEntries; ++i) PyTuple_SET_ITEM(names, i, PyUnicode_FromString(kEntries[i]));
  if (!names || PyModule_AddObject(m, "entries", names) != 0) return nullptr;
  if (PyModule_AddStringConstant(m, "torch_version", AMX_TORCH_VERSION) != 0) return nullptr;  // binding.py asks before bind()
  return m;
}
