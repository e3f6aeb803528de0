// The argument marshalling of binding.py's calls in native code: a CPython module whose Calls objects hold the
// entry points of one loaded libquest.so and call them with the pointers, sizes and strides of torch tensors.
//
// A call from Python through ctypes spends 2.5 to 3 us of its 5 on reading tensors' attributes one by one and converting
// the arguments, more than the launch itself; here both take 0.3 us.  Only the ordinary call is taken: exact tensors
// (no subclass, no active torch-function mode), plain Python numbers in the range of their C type,
// sizes of the expected rank.  For anything else a method returns None, nothing having been called, and binding.py goes the
// general way, which also is the one that raises for what is wrong.
#include <Python.h>

#include <string.h>

#include <limits>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/quest.h"

namespace {

struct Entries {
    decltype(&quest_hadamard_quantize) quantize;
    decltype(&quest_hadamard_quantize_pair) quantize_pair;
    decltype(&quest_hadamard_quantize_fp4) quantize_fp4;
    decltype(&quest_hadamard_quantize_fp4_pair) quantize_fp4_pair;
    decltype(&quest_lowbit_gemm) lowbit_gemm;
    decltype(&quest_lowbit_gemm_fp4) lowbit_gemm_fp4;
    decltype(&quest_trust_backward) trust_backward;
    decltype(&quest_trust_backward_pair) trust_backward_pair;
    decltype(&quest_grad_gemm) grad_gemm;
    decltype(&quest_grad_gemm_fp4) grad_gemm_fp4;
    decltype(&quest_weight_only_gemm) weight_only_gemm;
};
constexpr Py_ssize_t kEntries = sizeof(Entries) / sizeof(void *);

struct Calls {
    PyObject_HEAD
    Entries entry;
};

// Reads the arguments one after another; `plain` stays true while each is what the quick way takes.
class Reader {
public:
    Reader(PyObject *const *args, Py_ssize_t count, Py_ssize_t expected) : args_(args), plain(count == expected) {}

    int64_t integer(int64_t low, int64_t high)
    {
        PyObject *o = next();
        if (!plain || !PyLong_CheckExact(o))
            return refuse();
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        return overflow || v < low || v > high ? refuse() : v;
    }
    int32_t i32() { return (int32_t)integer(std::numeric_limits<int32_t>::min(), std::numeric_limits<int32_t>::max()); }
    int64_t i64() { return integer(std::numeric_limits<int64_t>::min(), std::numeric_limits<int64_t>::max()); }
    float f32()
    {
        PyObject *o = next();
        if (!plain || !PyFloat_CheckExact(o)) {
            refuse();
            return 0.0f;
        }
        return (float)PyFloat_AS_DOUBLE(o);
    }
    const at::Tensor *tensor()
    {
        PyObject *o = next();
        if (!plain || !THPVariable_CheckExact(o) || at::impl::torch_function_mode_enabled()) {
            refuse();
            return nullptr;
        }
        return &THPVariable_Unpack(o);
    }
    // a tensor of two dimensions, the second one contiguous or not (the entry points take row pitches only)
    const at::Tensor *matrix()
    {
        const at::Tensor *t = tensor();
        if (t && t->dim() != 2) {
            refuse();
            return nullptr;
        }
        return t;
    }
    const at::Tensor *tensor_or_none()
    {
        if (plain && args_[at_] == Py_None) {
            ++at_;
            return nullptr;
        }
        return tensor();
    }
    quest_dtype dtype(const at::Tensor *t)
    {
        if (t && t->scalar_type() == at::kBFloat16)
            return QUEST_BF16;
        if (!t || t->scalar_type() != at::kFloat)
            refuse();
        return QUEST_F32;
    }
    int64_t size(const at::Tensor *t, int64_t dim) { return t && dim < t->dim() ? t->size(dim) : refuse(); }
    int64_t stride(const at::Tensor *t, int64_t dim) { return t && dim < t->dim() ? t->stride(dim) : refuse(); }
    PyObject *object() { return next(); }
    void require(bool condition)
    {
        if (!condition)
            refuse();
    }

private:
    PyObject *next() { return plain ? args_[at_++] : nullptr; }
    int64_t refuse()
    {
        plain = false;
        return 0;
    }

    PyObject *const *args_;
    Py_ssize_t at_ = 0;

public:
    bool plain;
};

template <typename T = uint8_t>
T *pointer(const at::Tensor *t)
{
    return t ? static_cast<T *>(t->data_ptr()) : nullptr;
}

int64_t bytes(const at::Tensor *t)
{
    return t ? t->numel() * t->element_size() : 0;
}

// The call itself on the stream that `ask_stream` returns the handle of, without the interpreter lock; its status as a number
template <typename Call>
PyObject *enqueue(PyObject *ask_stream, Call &&call)
{
    PyObject *handle = PyObject_CallNoArgs(ask_stream);
    if (!handle)
        return nullptr;
    void *stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!stream && PyErr_Occurred())
        return nullptr;
    quest_status status;
    Py_BEGIN_ALLOW_THREADS
    status = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

#define QUEST_ENTRY()                                              \
    const Entries &entry = reinterpret_cast<Calls *>(self)->entry; \
    HANDLE_TH_ERRORS
#define QUEST_PLAIN_OR_NONE(READER) \
    if (!(READER).plain)            \
        Py_RETURN_NONE;

// Arguments of the methods in brackets; `stream`: a callable that returns the stream's handle
// (x, had_block, bits, alpha, outer_trust, codes, scales, mask, xh_out, stream)
PyObject *hadamard_quantize(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 10);
    const at::Tensor *x = r.matrix();
    const int32_t block = r.i32(), bits = r.i32();
    const float alpha = r.f32(), outer = r.f32();
    const at::Tensor *codes = r.tensor(), *scales = r.tensor(), *mask = r.tensor_or_none(), *xh = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const quest_dtype dtype = r.dtype(x);
    QUEST_PLAIN_OR_NONE(r)
    void *px = pointer(x);
    uint8_t *pc = pointer(codes), *pm = pointer(mask);
    float *ps = pointer<float>(scales), *ph = pointer<float>(xh);
    const int64_t rows = x->size(0), cols = x->size(1), ld = x->stride(0);
    return enqueue(ask_stream, [&](void *stream) { return entry.quantize(px, dtype, rows, cols, ld, block, bits, alpha, outer, pc, ps, pm, ph, stream); });
    END_HANDLE_TH_ERRORS
}

// (x, had_block, alpha, codes, scales, mask, xh_out, stream)
PyObject *hadamard_quantize_fp4(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 8);
    const at::Tensor *x = r.matrix();
    const int32_t block = r.i32();
    const float alpha = r.f32();
    const at::Tensor *codes = r.tensor(), *scales = r.tensor(), *mask = r.tensor_or_none(), *xh = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const quest_dtype dtype = r.dtype(x);
    QUEST_PLAIN_OR_NONE(r)
    void *px = pointer(x);
    uint8_t *pc = pointer(codes), *pm = pointer(mask);
    float *ps = pointer<float>(scales), *ph = pointer<float>(xh);
    const int64_t rows = x->size(0), cols = x->size(1), ld = x->stride(0);
    return enqueue(ask_stream, [&](void *stream) { return entry.quantize_fp4(px, dtype, rows, cols, ld, block, alpha, pc, ps, pm, ph, stream); });
    END_HANDLE_TH_ERRORS
}

// (x, w, had_block, bits, alpha, outer_trust, x_codes, x_scales, x_mask, w_codes, w_scales, w_mask, stream); with E2M1 without
// bits and outer_trust
template <bool FP4>
PyObject *hadamard_quantize_pair(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, FP4 ? 11 : 13);
    const at::Tensor *x = r.matrix(), *w = r.matrix();
    const int32_t block = r.i32(), bits = FP4 ? 4 : r.i32();
    const float alpha = r.f32(), outer = FP4 ? -1.0f : r.f32();
    const at::Tensor *x_codes = r.tensor(), *x_scales = r.tensor(), *x_mask = r.tensor_or_none();
    const at::Tensor *w_codes = r.tensor(), *w_scales = r.tensor(), *w_mask = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const quest_dtype dtype = r.dtype(x);
    r.require(r.plain && x->size(1) == w->size(1) && x->scalar_type() == w->scalar_type());
    QUEST_PLAIN_OR_NONE(r)
    void *px = pointer(x), *pw = pointer(w);
    uint8_t *xc = pointer(x_codes), *xm = pointer(x_mask), *wc = pointer(w_codes), *wm = pointer(w_mask);
    float *xs = pointer<float>(x_scales), *ws = pointer<float>(w_scales);
    const int64_t cols = x->size(1), rows_x = x->size(0), rows_w = w->size(0), ld_x = x->stride(0), ld_w = w->stride(0);
    return enqueue(ask_stream, [&](void *stream) {
        return FP4 ? entry.quantize_fp4_pair(px, rows_x, ld_x, xc, xs, xm, pw, rows_w, ld_w, wc, ws, wm, dtype, cols, block,
                                             alpha, stream)
                   : entry.quantize_pair(px, rows_x, ld_x, xc, xs, xm, pw, rows_w, ld_w, wc, ws, wm, dtype, cols, block, bits,
                                         alpha, outer, stream);
    });
    END_HANDLE_TH_ERRORS
}

// (a_codes, a_scales, b_codes, b_scales, K, bits, y, acc_out, workspace, stream)
PyObject *lowbit_gemm(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 10);
    const at::Tensor *a = r.tensor(), *a_scales = r.tensor(), *b = r.tensor(), *b_scales = r.tensor();
    const int64_t K = r.i64();
    const int32_t bits = r.i32();
    const at::Tensor *y = r.tensor_or_none(), *acc = r.tensor_or_none(), *workspace = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const int64_t M = r.size(a, 0), N = r.size(b, 0), ld_y = y ? r.stride(y, 0) : N;
    QUEST_PLAIN_OR_NONE(r)
    uint8_t *pa = pointer(a), *pb = pointer(b);
    float *sa = pointer<float>(a_scales), *sb = pointer<float>(b_scales);
    void *py = pointer(y), *pws = pointer(workspace);
    int32_t *pacc = pointer<int32_t>(acc);
    const int64_t scratch = bytes(workspace);
    return enqueue(ask_stream, [&](void *stream) { return entry.lowbit_gemm(pa, sa, M, pb, sb, N, K, bits, py, ld_y, pacc, pws, scratch, stream); });
    END_HANDLE_TH_ERRORS
}

// (a_codes, a_scales, b_codes, b_scales, K, y, acc_out, stream)
PyObject *lowbit_gemm_fp4(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 8);
    const at::Tensor *a = r.tensor(), *a_scales = r.tensor(), *b = r.tensor(), *b_scales = r.tensor();
    const int64_t K = r.i64();
    const at::Tensor *y = r.tensor_or_none(), *acc = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const int64_t M = r.size(a, 0), N = r.size(b, 0), ld_y = y ? r.stride(y, 0) : N;
    QUEST_PLAIN_OR_NONE(r)
    uint8_t *pa = pointer(a), *pb = pointer(b);
    float *sa = pointer<float>(a_scales), *sb = pointer<float>(b_scales), *pacc = pointer<float>(acc);
    void *py = pointer(y);
    return enqueue(ask_stream, [&](void *stream) { return entry.lowbit_gemm_fp4(pa, sa, M, pb, sb, N, K, py, ld_y, pacc, stream); });
    END_HANDLE_TH_ERRORS
}

// (g, mask, had_block, out, stream)
PyObject *trust_backward(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 5);
    const at::Tensor *g = r.matrix(), *mask = r.tensor_or_none();
    const int32_t block = r.i32();
    const at::Tensor *out = r.tensor();
    PyObject *ask_stream = r.object();
    const quest_dtype g_dtype = r.dtype(g), out_dtype = r.dtype(out);
    QUEST_PLAIN_OR_NONE(r)
    void *pg = pointer(g), *po = pointer(out);
    uint8_t *pm = pointer(mask);
    const int64_t rows = g->size(0), cols = g->size(1);
    return enqueue(ask_stream, [&](void *stream) { return entry.trust_backward(pg, g_dtype, pm, rows, cols, block, po, out_dtype, stream); });
    END_HANDLE_TH_ERRORS
}

// (g_x, mask_x, g_w, mask_w, had_block, out_x, out_w, stream)
PyObject *trust_backward_pair(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 8);
    const at::Tensor *gx = r.matrix(), *mask_x = r.tensor_or_none(), *gw = r.matrix(), *mask_w = r.tensor_or_none();
    const int32_t block = r.i32();
    const at::Tensor *out_x = r.tensor(), *out_w = r.tensor();
    PyObject *ask_stream = r.object();
    const quest_dtype g_dtype = r.dtype(gx), out_dtype = r.dtype(out_x);
    r.require(r.plain && gx->size(1) == gw->size(1) && gx->scalar_type() == gw->scalar_type() &&
              out_x->scalar_type() == out_w->scalar_type());
    QUEST_PLAIN_OR_NONE(r)
    void *px = pointer(gx), *pw = pointer(gw), *ox = pointer(out_x), *ow = pointer(out_w);
    uint8_t *mx = pointer(mask_x), *mw = pointer(mask_w);
    const int64_t rows_x = gx->size(0), rows_w = gw->size(0), cols = gx->size(1);
    return enqueue(ask_stream, [&](void *stream) {
        return entry.trust_backward_pair(px, mx, rows_x, ox, pw, mw, rows_w, ow, g_dtype, cols, block, out_dtype, stream);
    });
    END_HANDLE_TH_ERRORS
}

// (which, dy, q_codes, q_scales, bits, M, N, K, out, workspace, stream); with E2M1 without bits
template <bool FP4>
PyObject *grad_gemm(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, FP4 ? 10 : 11);
    const int32_t which = r.i32();
    const at::Tensor *dy = r.tensor(), *codes = r.tensor(), *scales = r.tensor();
    const int32_t bits = FP4 ? 4 : r.i32();
    const int64_t M = r.i64(), N = r.i64(), K = r.i64();
    const at::Tensor *out = r.tensor(), *workspace = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    QUEST_PLAIN_OR_NONE(r)
    void *pdy = pointer(dy), *po = pointer(out), *pws = pointer(workspace);
    uint8_t *pc = pointer(codes);
    float *ps = pointer<float>(scales);
    const int64_t scratch = bytes(workspace);
    return enqueue(ask_stream, [&](void *stream) {
        return FP4 ? entry.grad_gemm_fp4(which, pdy, pc, ps, M, N, K, po, pws, scratch, stream)
                   : entry.grad_gemm(which, pdy, pc, ps, bits, M, N, K, po, pws, scratch, stream);
    });
    END_HANDLE_TH_ERRORS
}

// (x, w_codes, w_scales, bits, y, workspace, stream)
PyObject *weight_only_gemm(PyObject *self, PyObject *const *args, Py_ssize_t count)
{
    QUEST_ENTRY()
    Reader r(args, count, 7);
    const at::Tensor *x = r.matrix(), *codes = r.tensor(), *scales = r.tensor();
    const int32_t bits = r.i32();
    const at::Tensor *y = r.tensor(), *workspace = r.tensor_or_none();
    PyObject *ask_stream = r.object();
    const int64_t N = r.size(codes, 0);
    QUEST_PLAIN_OR_NONE(r)
    void *px = pointer(x), *py = pointer(y), *pws = pointer(workspace);
    uint8_t *pc = pointer(codes);
    float *ps = pointer<float>(scales);
    const int64_t M = x->size(0), K = x->size(1), scratch = bytes(workspace);
    return enqueue(ask_stream, [&](void *stream) { return entry.weight_only_gemm(px, pc, ps, bits, M, N, K, py, pws, scratch, stream); });
    END_HANDLE_TH_ERRORS
}

#undef QUEST_ENTRY
#undef QUEST_PLAIN_OR_NONE

// Calls(addresses of the entry points in the order of Entries)
PyObject *new_calls(PyTypeObject *type, PyObject *args, PyObject *)
{
    if (PyTuple_GET_SIZE(args) != kEntries) {
        PyErr_SetString(PyExc_TypeError, "one address for each entry point");
        return nullptr;
    }
    auto *self = reinterpret_cast<Calls *>(type->tp_alloc(type, 0));
    if (!self)
        return nullptr;
    void *address[kEntries];
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        address[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(args, i));
        if (!address[i]) {
            if (!PyErr_Occurred())
                PyErr_SetString(PyExc_ValueError, "null entry point");
            Py_DECREF(self);
            return nullptr;
        }
    }
    memcpy(&self->entry, address, sizeof(Entries));
    return reinterpret_cast<PyObject *>(self);
}

#define QUEST_METHOD(NAME, FUNCTION) {NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(FUNCTION)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {QUEST_METHOD("hadamard_quantize", hadamard_quantize),
                         QUEST_METHOD("hadamard_quantize_pair", hadamard_quantize_pair<false>),
                         QUEST_METHOD("hadamard_quantize_fp4", hadamard_quantize_fp4),
                         QUEST_METHOD("hadamard_quantize_fp4_pair", hadamard_quantize_pair<true>),
                         QUEST_METHOD("lowbit_gemm", lowbit_gemm),
                         QUEST_METHOD("lowbit_gemm_fp4", lowbit_gemm_fp4),
                         QUEST_METHOD("trust_backward", trust_backward),
                         QUEST_METHOD("trust_backward_pair", trust_backward_pair),
                         QUEST_METHOD("grad_gemm", grad_gemm<false>),
                         QUEST_METHOD("grad_gemm_fp4", grad_gemm<true>),
                         QUEST_METHOD("weight_only_gemm", weight_only_gemm),
                         {nullptr, nullptr, 0, nullptr}};
#undef QUEST_METHOD

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0) "quest_python.Calls", sizeof(Calls)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "quest_python", nullptr, -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_quest_python(void)
{
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_methods = methods;
    calls_type.tp_new = new_calls;
    if (PyType_Ready(&calls_type) < 0)
        return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m)
        return nullptr;
    if (PyModule_AddStringConstant(m, "TORCH_BUILD", QUEST_TORCH_BUILD) < 0) {   // binding.py compares it
        Py_DECREF(m);
        return nullptr;
    }
    Py_INCREF(&calls_type);
    if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject *>(&calls_type)) < 0) {
        Py_DECREF(&calls_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
