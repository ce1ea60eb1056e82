// The per-call half of the Python binding in C++: the launches of the hot path as Python callables.
//
// A pass over a small layer is a handful of kernels of 3 - 6 us, and marshalled through ctypes a call took 9 - 10 us of
// host time (argument checks 4, conversion of the C arguments 2, current stream 1.3, launch 2 - 3), so small batches ran at
// the speed of the interpreter.  The same checks, in the same order and with the same messages, take well under a
// microsecond here.  No arithmetic, no allocation but the outputs that the caller leaves out, no state but the table
// of entry points, which is filled once from the loaded libptq4vm.so.
#include <ATen/ATen.h>
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "../../include/ptq4vm.h"

namespace {

struct Raised {};  // a Python exception is set

[[noreturn]] void raise(PyObject *type, const std::string &text) {
    PyErr_SetString(type, text.c_str());
    throw Raised{};
}

// ---------------------------------------------------------------------------------- entry points of the library
#define PTQ4VM_HOT_ENTRIES(X)                                                                                      \
    X(quantize_pts) X(quantize_dynamic) X(quantize_pts_offset) X(quantize_pts_a4) X(quantize_pts_a4_e2m3)          \
    X(w8a8_linear) X(w8a8_linear_offset) X(w4a4_linear) X(w4a4_linear_e2m3) X(w8a8_linear_fused)                   \
    X(w8a8_linear_offset_fused) X(w4a4_linear_fused) X(f16_linear)

struct Entries {
#define X(name) decltype(&ptq4vm_##name) name = nullptr;
    PTQ4VM_HOT_ENTRIES(X)
#undef X
} entry;
bool bound = false;
PyObject *load_library = nullptr;  // binding._load_entries(): calls bind() below, raises if the library is missing
PyObject *raise_status = nullptr;  // binding.check(status)

void need_library() {
    if (bound) return;
    PyObject *r = PyObject_CallNoArgs(load_library);
    if (!r) throw Raised{};
    Py_DECREF(r);
}

void check(int status) {
    if (status == PTQ4VM_OK) return;
    PyObject *r = PyObject_CallFunction(raise_status, "i", status);
    Py_XDECREF(r);
    throw Raised{};
}

// Calls f(current stream) without the interpreter lock (a launch waits when its queue is full) and raises for its status.
template <typename F>
void launch(F &&f) {
    void *const stream = static_cast<void *>(c10::hip::getCurrentHIPStream().stream());
    PyThreadState *const state = PyEval_SaveThread();
    const int status = f(stream);
    PyEval_RestoreThread(state);
    check(status);
}

// ---------------------------------------------------------------------------------- arguments
const char *dtype_name(at::ScalarType t) {
    switch (t) {
        case at::kHalf: return "torch.float16";
        case at::kChar: return "torch.int8";
        case at::kByte: return "torch.uint8";
        case at::kInt: return "torch.int32";
        default: return "torch.float32";
    }
}

bool given(PyObject *o) { return o && o != Py_None; }

const at::Tensor *tensor(PyObject *o) { return o && THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

struct Matrix {
    int64_t rows, cols, ld;
    void *data;
};

Matrix matrix(PyObject *o, at::ScalarType dtype, const char *name) {
    const at::Tensor *t = tensor(o);
    if (!t || !t->is_cuda() || t->scalar_type() != dtype || t->dim() != 2 || (t->size(1) > 1 && t->stride(1) != 1))
        raise(PyExc_TypeError, std::string(name) + ": expected a 2-D CUDA tensor of " + dtype_name(dtype) + " with unit inner stride");
    const int64_t rows = t->size(0), cols = t->size(1), pitch = t->stride(0);
    return {rows, cols, rows > 1 ? pitch : std::max(pitch, cols), t->data_ptr()};
}

// A matrix that the kernels write rows x cols elements of.  A larger one (a buffer of the largest batch) is taken too; the
// C boundary sees a pointer and a pitch only, so a smaller one has to be refused here.
Matrix written(PyObject *o, at::ScalarType dtype, int64_t rows, int64_t cols, const char *name) {
    const Matrix m = matrix(o, dtype, name);
    if (m.rows < rows || m.cols < cols)
        raise(PyExc_ValueError, std::string(name) + ": expected at least " + std::to_string(rows) + " x " + std::to_string(cols) + " elements, got " +
                                    std::to_string(m.rows) + " x " + std::to_string(m.cols));
    return m;
}

void *vector(PyObject *o, at::ScalarType dtype, int64_t n, const char *name, bool optional = false) {
    if (!given(o)) {
        if (optional) return nullptr;
        raise(PyExc_TypeError, std::string(name) + " is required");
    }
    const at::Tensor *t = tensor(o);
    if (!t || !t->is_cuda() || t->scalar_type() != dtype || t->dim() != 1 || t->size(0) != n || !t->is_contiguous())
        raise(PyExc_TypeError, std::string(name) + ": expected a contiguous CUDA vector of " + std::to_string(n) + " x " + dtype_name(dtype));
    return t->data_ptr();
}

void *accumulators(PyObject *o, int64_t M, int64_t N) {
    if (!given(o)) return nullptr;
    const at::Tensor *t = tensor(o);
    if (!t || !t->is_cuda() || t->scalar_type() != at::kInt || t->dim() != 2 || t->size(0) != M || t->size(1) != N || !t->is_contiguous())
        raise(PyExc_TypeError, "acc_out: expected a dense CUDA int32 [M, N] tensor");
    return t->data_ptr();
}

int64_t integer(PyObject *o) {
    const int64_t v = PyLong_Check(o) ? PyLong_AsLongLong(o) : [&] {
        PyObject *i = PyNumber_Index(o);
        if (!i) throw Raised{};
        const int64_t w = PyLong_AsLongLong(i);
        Py_DECREF(i);
        return w;
    }();
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

int64_t e2m3_blocks(int64_t K) { return (K + 127) / 128; }

struct Container {
    int64_t pitch;
    void *data;
};

Container container(PyObject *o, int64_t rows, int64_t K, const char *name) {
    const at::Tensor *t = tensor(o);
    if (!t || !t->is_cuda() || t->scalar_type() != at::kByte || t->dim() != 3)
        raise(PyExc_TypeError, std::string(name) + ": expected a CUDA uint8 tensor [blocks, rows, 96]");
    const int64_t blocks = e2m3_blocks(K);
    if (t->size(0) != blocks || t->size(1) != rows || t->size(2) != 96 || t->stride(2) != 1 || (rows > 1 && t->stride(1) != 96))
        raise(PyExc_ValueError, std::string(name) + ": expected shape (" + std::to_string(blocks) + ", " + std::to_string(rows) +
                                    ", 96) with dense 96-byte blocks");
    return {blocks > 1 ? t->stride(0) : std::max<int64_t>(t->stride(0), 96 * rows), t->data_ptr()};
}

// An output: the caller's tensor (a new reference to it) or a fresh one on the device of `like`.
PyObject *output(PyObject *o, at::IntArrayRef shape, at::ScalarType dtype, PyObject *like) {
    if (given(o)) {
        Py_INCREF(o);
        return o;
    }
    PyObject *w = THPVariable_Wrap(at::empty(shape, THPVariable_Unpack(like).options().dtype(dtype)));
    if (!w) throw Raised{};
    return w;
}

struct Owned {  // releases the output when a later step raises
    PyObject *o;
    explicit Owned(PyObject *p) : o(p) {}
    Owned(const Owned &) = delete;
    ~Owned() { Py_XDECREF(o); }
    PyObject *release() {
        PyObject *p = o;
        o = nullptr;
        return p;
    }
};

const float *floats(void *p) { return static_cast<const float *>(p); }
const int8_t *codes(const Matrix &m) { return static_cast<const int8_t *>(m.data); }
const uint8_t *bytes(void *p) { return static_cast<const uint8_t *>(p); }
const int32_t *ints(void *p) { return static_cast<const int32_t *>(p); }

// M == B * L, in exact arithmetic
bool is_product(int64_t M, int64_t B, int64_t L) {
    int64_t p;
    return !__builtin_mul_overflow(B, L, &p) && p == M;
}
void same_rows(int64_t M, int64_t B, int64_t L) {
    if (!is_product(M, B, L)) raise(PyExc_ValueError, "x must have B*L rows");
}
void same_shape(bool ok) {
    if (!ok) raise(PyExc_ValueError, "shape mismatch");
}

// ---------------------------------------------------------------------------------- the calls
using Args = PyObject *const *;

PyObject *quantize_pts(Args a) {  // x inv_m s_tok B L xq
    const Matrix x = matrix(a[0], at::kHalf, "x");
    const int64_t B = integer(a[3]), L = integer(a[4]);
    same_rows(x.rows, B, L);
    void *inv_m = vector(a[1], at::kFloat, x.cols, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok");
    Owned out(output(a[5], {x.rows, x.cols}, at::kChar, a[0]));
    const Matrix xq = written(out.o, at::kChar, x.rows, x.cols, "xq");
    launch([&](void *s) { return entry.quantize_pts(x.data, floats(inv_m), floats(s_tok), static_cast<int8_t *>(xq.data), B, L, x.cols, x.ld, xq.ld, s); });
    return out.release();
}

PyObject *quantize_pts_offset(Args a) {  // x inv_m s_tok z_tok B L xq
    const Matrix x = matrix(a[0], at::kHalf, "x");
    const int64_t B = integer(a[4]), L = integer(a[5]);
    same_rows(x.rows, B, L);
    void *inv_m = vector(a[1], at::kFloat, x.cols, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok"),
         *z_tok = vector(a[3], at::kInt, L, "z_tok");
    Owned out(output(a[6], {x.rows, x.cols}, at::kChar, a[0]));
    const Matrix xq = written(out.o, at::kChar, x.rows, x.cols, "xq");
    launch([&](void *s) { return entry.quantize_pts_offset(x.data, floats(inv_m), floats(s_tok), ints(z_tok), static_cast<int8_t *>(xq.data), B, L, x.cols,
                                    x.ld, xq.ld, s); });
    return out.release();
}

PyObject *quantize_pts_a4(Args a) {  // x inv_m s_tok B L xq4
    const Matrix x = matrix(a[0], at::kHalf, "x");
    const int64_t B = integer(a[3]), L = integer(a[4]);
    same_rows(x.rows, B, L);
    void *inv_m = vector(a[1], at::kFloat, x.cols, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok");
    Owned out(output(a[5], {x.rows, x.cols / 2}, at::kByte, a[0]));
    const Matrix xq = written(out.o, at::kByte, x.rows, x.cols / 2, "xq4");
    launch([&](void *s) { return entry.quantize_pts_a4(x.data, floats(inv_m), floats(s_tok), static_cast<uint8_t *>(xq.data), B, L, x.cols, x.ld, xq.ld, s); });
    return out.release();
}

PyObject *quantize_pts_a4_e2m3(Args a) {  // x inv_m s_tok B L xq6
    const Matrix x = matrix(a[0], at::kHalf, "x");
    const int64_t B = integer(a[3]), L = integer(a[4]);
    same_rows(x.rows, B, L);
    void *inv_m = vector(a[1], at::kFloat, x.cols, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok");
    Owned out(output(a[5], {e2m3_blocks(x.cols), x.rows, 96}, at::kByte, a[0]));
    const Container xq = container(out.o, x.rows, x.cols, "xq6");
    launch([&](void *s) { return entry.quantize_pts_a4_e2m3(x.data, floats(inv_m), floats(s_tok), static_cast<uint8_t *>(xq.data), B, L, x.cols, x.ld, xq.pitch,
                                     s); });
    return out.release();
}

PyObject *quantize_dynamic(Args a) {  // x inv_m xq s_row
    const Matrix x = matrix(a[0], at::kHalf, "x");
    void *inv_m = vector(a[1], at::kFloat, x.cols, "inv_m", true);
    Owned out(output(a[2], {x.rows, x.cols}, at::kChar, a[0]));
    const Matrix xq = written(out.o, at::kChar, x.rows, x.cols, "xq");
    Owned steps(output(a[3], {x.rows}, at::kFloat, a[0]));
    void *s_row = vector(steps.o, at::kFloat, x.rows, "s_row");
    launch([&](void *s) { return entry.quantize_dynamic(x.data, floats(inv_m), static_cast<int8_t *>(xq.data), static_cast<float *>(s_row), x.rows, x.cols, x.ld,
                                 xq.ld, s); });
    PyObject *pair = PyTuple_Pack(2, out.o, steps.o);
    if (!pair) throw Raised{};
    return pair;
}

PyObject *w8a8_linear(Args a) {  // xq wq s_tok s_w bias B L y acc_out
    const Matrix xq = matrix(a[0], at::kChar, "xq"), wq = matrix(a[1], at::kChar, "wq");
    const int64_t B = integer(a[5]), L = integer(a[6]), M = xq.rows, N = wq.rows;
    same_shape(xq.cols == wq.cols && is_product(M, B, L));
    void *s_tok = vector(a[2], at::kFloat, L, "s_tok"), *s_w = vector(a[3], at::kFloat, N, "s_w"), *bias = vector(a[4], at::kHalf, N, "bias", true);
    Owned out(output(a[7], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[8], M, N);
    launch([&](void *s) { return entry.w8a8_linear(codes(xq), codes(wq), floats(s_tok), floats(s_w), bias, y.data, static_cast<int32_t *>(acc), B, L, xq.cols, N,
                            xq.ld, wq.ld, y.ld, s); });
    return out.release();
}

PyObject *w8a8_linear_offset(Args a) {  // xq wq s_tok z_tok rowsum s_w bias B L y acc_out
    const Matrix xq = matrix(a[0], at::kChar, "xq"), wq = matrix(a[1], at::kChar, "wq");
    const int64_t B = integer(a[7]), L = integer(a[8]), M = xq.rows, N = wq.rows;
    same_shape(xq.cols == wq.cols && is_product(M, B, L));
    void *s_tok = vector(a[2], at::kFloat, L, "s_tok"), *z_tok = vector(a[3], at::kInt, L, "z_tok"),
         *rowsum = vector(a[4], at::kInt, N, "rowsum"), *s_w = vector(a[5], at::kFloat, N, "s_w"),
         *bias = vector(a[6], at::kHalf, N, "bias", true);
    Owned out(output(a[9], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[10], M, N);
    launch([&](void *s) { return entry.w8a8_linear_offset(codes(xq), codes(wq), floats(s_tok), ints(z_tok), ints(rowsum), floats(s_w), bias, y.data,
                                   static_cast<int32_t *>(acc), B, L, xq.cols, N, xq.ld, wq.ld, y.ld, s); });
    return out.release();
}

PyObject *w4a4_linear(Args a) {  // xq4 wq4 s_tok s_w bias B L y acc_out
    const Matrix xq = matrix(a[0], at::kByte, "xq4"), wq = matrix(a[1], at::kByte, "wq4");
    const int64_t B = integer(a[5]), L = integer(a[6]), M = xq.rows, N = wq.rows;
    same_shape(xq.cols == wq.cols && is_product(M, B, L));
    void *s_tok = vector(a[2], at::kFloat, L, "s_tok"), *s_w = vector(a[3], at::kFloat, N, "s_w"), *bias = vector(a[4], at::kHalf, N, "bias", true);
    Owned out(output(a[7], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[8], M, N);
    launch([&](void *s) { return entry.w4a4_linear(bytes(xq.data), bytes(wq.data), floats(s_tok), floats(s_w), bias, y.data, static_cast<int32_t *>(acc), B, L,
                            2 * xq.cols, N, xq.ld, wq.ld, y.ld, s); });
    return out.release();
}

PyObject *w4a4_linear_e2m3(Args a) {  // xq6 wq6 s_tok s_w bias B L K y acc_out
    const int64_t B = integer(a[5]), L = integer(a[6]), K = integer(a[7]);
    int64_t M;
    if (__builtin_mul_overflow(B, L, &M)) raise(PyExc_ValueError, "xq6: B*L is out of range");
    const Container xq = container(a[0], M, K, "xq6");
    const at::Tensor *w = tensor(a[1]);
    if (!w || w->dim() != 3) raise(PyExc_TypeError, "wq6: expected a CUDA uint8 tensor [blocks, N, 96]");
    const int64_t N = w->size(1);
    const Container wq = container(a[1], N, K, "wq6");
    void *s_tok = vector(a[2], at::kFloat, L, "s_tok"), *s_w = vector(a[3], at::kFloat, N, "s_w"), *bias = vector(a[4], at::kHalf, N, "bias", true);
    Owned out(output(a[8], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[9], M, N);
    launch([&](void *s) { return entry.w4a4_linear_e2m3(bytes(xq.data), bytes(wq.data), floats(s_tok), floats(s_w), bias, y.data, static_cast<int32_t *>(acc), B, L,
                                 K, N, xq.pitch, wq.pitch, y.ld, s); });
    return out.release();
}

struct CodesOut {
    int64_t ld = 0;
    int8_t *data = nullptr;
};
CodesOut codes_out(PyObject *o, int64_t M, int64_t K) {
    if (!given(o)) return {};
    const Matrix m = matrix(o, at::kChar, "xq_out");
    if (m.rows != M || m.cols != K) raise(PyExc_ValueError, "xq_out must be [B*L, K]");
    return {m.ld, static_cast<int8_t *>(m.data)};
}

PyObject *w8a8_linear_fused(Args a) {  // x inv_m s_tok wq s_w bias B L y acc_out xq_out
    const Matrix x = matrix(a[0], at::kHalf, "x"), wq = matrix(a[3], at::kChar, "wq");
    const int64_t B = integer(a[6]), L = integer(a[7]), M = x.rows, K = x.cols, N = wq.rows;
    same_shape(K == wq.cols && is_product(M, B, L));
    void *inv_m = vector(a[1], at::kFloat, K, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok"),
         *s_w = vector(a[4], at::kFloat, N, "s_w"), *bias = vector(a[5], at::kHalf, N, "bias", true);
    Owned out(output(a[8], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[9], M, N);
    const CodesOut xq = codes_out(a[10], M, K);
    launch([&](void *s) { return entry.w8a8_linear_fused(x.data, floats(inv_m), floats(s_tok), codes(wq), floats(s_w), bias, y.data, static_cast<int32_t *>(acc),
                                  xq.data, B, L, K, N, x.ld, wq.ld, y.ld, xq.ld, s); });
    return out.release();
}

PyObject *w8a8_linear_offset_fused(Args a) {  // x inv_m s_tok z_tok wq rowsum s_w bias B L y acc_out xq_out
    const Matrix x = matrix(a[0], at::kHalf, "x"), wq = matrix(a[4], at::kChar, "wq");
    const int64_t B = integer(a[8]), L = integer(a[9]), M = x.rows, K = x.cols, N = wq.rows;
    same_shape(K == wq.cols && is_product(M, B, L));
    void *inv_m = vector(a[1], at::kFloat, K, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok"),
         *z_tok = vector(a[3], at::kInt, L, "z_tok"), *rowsum = vector(a[5], at::kInt, N, "rowsum"),
         *s_w = vector(a[6], at::kFloat, N, "s_w"), *bias = vector(a[7], at::kHalf, N, "bias", true);
    Owned out(output(a[10], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[11], M, N);
    const CodesOut xq = codes_out(a[12], M, K);
    launch([&](void *s) { return entry.w8a8_linear_offset_fused(x.data, floats(inv_m), floats(s_tok), ints(z_tok), codes(wq), ints(rowsum), floats(s_w), bias, y.data,
                                         static_cast<int32_t *>(acc), xq.data, B, L, K, N, x.ld, wq.ld, y.ld, xq.ld, s); });
    return out.release();
}

PyObject *w4a4_linear_fused(Args a) {  // x inv_m s_tok wq4 s_w bias B L y acc_out xq_out
    const Matrix x = matrix(a[0], at::kHalf, "x"), wq = matrix(a[3], at::kByte, "wq4");
    const int64_t B = integer(a[6]), L = integer(a[7]), M = x.rows, K = x.cols, N = wq.rows;
    same_shape(K == 2 * wq.cols && is_product(M, B, L));
    void *inv_m = vector(a[1], at::kFloat, K, "inv_m", true), *s_tok = vector(a[2], at::kFloat, L, "s_tok"),
         *s_w = vector(a[4], at::kFloat, N, "s_w"), *bias = vector(a[5], at::kHalf, N, "bias", true);
    Owned out(output(a[8], {M, N}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, M, N, "y");
    void *acc = accumulators(a[9], M, N);
    const CodesOut xq = codes_out(a[10], M, K);
    launch([&](void *s) { return entry.w4a4_linear_fused(x.data, floats(inv_m), floats(s_tok), bytes(wq.data), floats(s_w), bias, y.data, static_cast<int32_t *>(acc),
                                  xq.data, B, L, K, N, x.ld, wq.ld, y.ld, xq.ld, s); });
    return out.release();
}

PyObject *f16_linear(Args a) {  // x w bias y
    const Matrix x = matrix(a[0], at::kHalf, "x"), w = matrix(a[1], at::kHalf, "w");
    same_shape(x.cols == w.cols);
    void *bias = vector(a[2], at::kHalf, w.rows, "bias", true);
    Owned out(output(a[3], {x.rows, w.rows}, at::kHalf, a[0]));
    const Matrix y = written(out.o, at::kHalf, x.rows, w.rows, "y");
    launch([&](void *s) { return entry.f16_linear(x.data, w.data, bias, y.data, x.rows, x.cols, w.rows, x.ld, w.ld, y.ld, s); });
    return out.release();
}

// ---------------------------------------------------------------------------------- Python signatures
constexpr int kMaxParams = 13;

struct Signature {
    const char *function;
    int required, total;
    const char *names[kMaxParams];
    PyObject *interned[kMaxParams];
};

// Python's calling convention: positional arguments, then keywords; missing optional ones stay null.
void parse(const Signature &sig, Args args, Py_ssize_t nargs, PyObject *kwnames, PyObject **out) {
    if (nargs > sig.total)
        raise(PyExc_TypeError, std::string(sig.function) + "() takes at most " + std::to_string(sig.total) + " arguments (" + std::to_string(nargs) + " given)");
    for (Py_ssize_t i = 0; i < nargs; i++) out[i] = args[i];
    for (int i = (int)nargs; i < sig.total; i++) out[i] = nullptr;
    const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < n_kw; k++) {
        PyObject *name = PyTuple_GET_ITEM(kwnames, k);
        int at = -1;
        for (int i = 0; i < sig.total && at < 0; i++)
            if (sig.interned[i] == name) at = i;
        for (int i = 0; i < sig.total && at < 0; i++)
            if (PyUnicode_CompareWithASCIIString(name, sig.names[i]) == 0) at = i;
        if (at < 0) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", sig.function, name);
            throw Raised{};
        }
        if (out[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", sig.function, name);
            throw Raised{};
        }
        out[at] = args[nargs + k];
    }
    for (int i = 0; i < sig.required; i++)
        if (!out[i]) raise(PyExc_TypeError, std::string(sig.function) + "() missing required argument: '" + sig.names[i] + "'");
}

// Inside a catch block: the exception as torch raises it (torch.OutOfMemoryError).  Apart from the call itself, because
// torch's macros set up a warning handler on the way in, 0.2 us a call.
PyObject *raise_as_torch() {
    HANDLE_TH_ERRORS
    throw;
    END_HANDLE_TH_ERRORS
}

template <PyObject *(*CALL)(Args), Signature *SIG>
PyObject *call(PyObject *, Args args, Py_ssize_t nargs, PyObject *kwnames) {
    try {
        PyObject *a[kMaxParams];
        parse(*SIG, args, nargs, kwnames, a);
        need_library();
        return CALL(a);
    } catch (const Raised &) {
        return nullptr;
    } catch (...) {  // an output that could not be allocated
        return raise_as_torch();
    }
}

#define SIG(name, required, total, ...) Signature sig_##name = {#name, required, total, {__VA_ARGS__}, {}};
SIG(quantize_pts, 5, 6, "x", "inv_m", "s_tok", "B", "L", "xq")
SIG(quantize_dynamic, 2, 4, "x", "inv_m", "xq", "s_row")
SIG(quantize_pts_offset, 6, 7, "x", "inv_m", "s_tok", "z_tok", "B", "L", "xq")
SIG(quantize_pts_a4, 5, 6, "x", "inv_m", "s_tok", "B", "L", "xq4")
SIG(quantize_pts_a4_e2m3, 5, 6, "x", "inv_m", "s_tok", "B", "L", "xq6")
SIG(w8a8_linear, 7, 9, "xq", "wq", "s_tok", "s_w", "bias", "B", "L", "y", "acc_out")
SIG(w8a8_linear_offset, 9, 11, "xq", "wq", "s_tok", "z_tok", "rowsum", "s_w", "bias", "B", "L", "y", "acc_out")
SIG(w4a4_linear, 7, 9, "xq4", "wq4", "s_tok", "s_w", "bias", "B", "L", "y", "acc_out")
SIG(w4a4_linear_e2m3, 8, 10, "xq6", "wq6", "s_tok", "s_w", "bias", "B", "L", "K", "y", "acc_out")
SIG(w8a8_linear_fused, 8, 11, "x", "inv_m", "s_tok", "wq", "s_w", "bias", "B", "L", "y", "acc_out", "xq_out")
SIG(w8a8_linear_offset_fused, 10, 13, "x", "inv_m", "s_tok", "z_tok", "wq", "rowsum", "s_w", "bias", "B", "L", "y", "acc_out", "xq_out")
SIG(w4a4_linear_fused, 8, 11, "x", "inv_m", "s_tok", "wq4", "s_w", "bias", "B", "L", "y", "acc_out", "xq_out")
SIG(f16_linear, 3, 4, "x", "w", "bias", "y")
#undef SIG

// bind({name: address of ptq4vm_<name>}): the entry points of the loaded library
PyObject *bind(PyObject *, PyObject *table) {
#define X(name)                                                                                        \
    {                                                                                                  \
        PyObject *v = PyDict_GetItemString(table, #name);                                              \
        if (!v) return PyErr_Format(PyExc_KeyError, "ptq4vm_%s", #name);                               \
        entry.name = reinterpret_cast<decltype(&ptq4vm_##name)>(PyLong_AsVoidPtr(v));                  \
        if (!entry.name) return PyErr_Format(PyExc_ValueError, "ptq4vm_%s: no address", #name);        \
    }
    PTQ4VM_HOT_ENTRIES(X)
#undef X
    bound = true;
    Py_RETURN_NONE;
}

// setup(load_library, raise_status): the two Python callbacks
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *load, *status;
    if (!PyArg_ParseTuple(args, "OO", &load, &status)) return nullptr;
    Py_INCREF(load);
    Py_INCREF(status);
    Py_XSETREF(load_library, load);
    Py_XSETREF(raise_status, status);
    Py_RETURN_NONE;
}

#define FAST(name, doc) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call<name, &sig_##name>)), METH_FASTCALL | METH_KEYWORDS, doc}
PyMethodDef methods[] = {
    FAST(quantize_pts, "quantize_pts(x, inv_m, s_tok, B, L, xq=None)\n--\n\nptq4vm_quantize_pts: xq int8 [B*L, K]."),
    FAST(quantize_dynamic, "quantize_dynamic(x, inv_m, xq=None, s_row=None)\n--\n\nptq4vm_quantize_dynamic: (xq int8 [M, K], s_row f32 [M])."),
    FAST(quantize_pts_offset, "quantize_pts_offset(x, inv_m, s_tok, z_tok, B, L, xq=None)\n--\n\n"
                              "ptq4vm_quantize_pts_offset: xq int8 [B*L, K] with the per-token zero offset z_tok (int32 [L])."),
    FAST(quantize_pts_a4, "quantize_pts_a4(x, inv_m, s_tok, B, L, xq4=None)\n--\n\n"
                          "ptq4vm_quantize_pts_a4: xq4 uint8 [B*L, K/2], two 4-bit codes per byte."),
    FAST(quantize_pts_a4_e2m3, "quantize_pts_a4_e2m3(x, inv_m, s_tok, B, L, xq6=None)\n--\n\n"
                               "ptq4vm_quantize_pts_a4_e2m3: xq6 uint8 [e2m3_blocks(K), B*L, 96], 4-bit codes as E2M3 patterns, block-major."),
    FAST(w8a8_linear, "w8a8_linear(xq, wq, s_tok, s_w, bias, B, L, y=None, acc_out=None)\n--\n\n"
                      "ptq4vm_w8a8_linear: y fp16 [B*L, N]; acc_out (int32 [B*L, N], dense) is filled if given."),
    FAST(w8a8_linear_offset, "w8a8_linear_offset(xq, wq, s_tok, z_tok, rowsum, s_w, bias, B, L, y=None, acc_out=None)\n--\n\n"
                             "ptq4vm_w8a8_linear_offset: y fp16 [B*L, N] with the zero-offset correction in the epilogue."),
    FAST(w4a4_linear, "w4a4_linear(xq4, wq4, s_tok, s_w, bias, B, L, y=None, acc_out=None)\n--\n\n"
                      "ptq4vm_w4a4_linear: y fp16 [B*L, N] from packed 4-bit operands."),
    FAST(w4a4_linear_e2m3, "w4a4_linear_e2m3(xq6, wq6, s_tok, s_w, bias, B, L, K, y=None, acc_out=None)\n--\n\n"
                           "ptq4vm_w4a4_linear_e2m3: y fp16 [B*L, N] from operands in the block-major E2M3 container (K codes per row)."),
    FAST(w8a8_linear_fused, "w8a8_linear_fused(x, inv_m, s_tok, wq, s_w, bias, B, L, y=None, acc_out=None, xq_out=None)\n--\n\n"
                            "ptq4vm_w8a8_linear_fused: y fp16 [B*L, N] from fp16 activations; acc_out / xq_out are filled if given."),
    FAST(w8a8_linear_offset_fused,
         "w8a8_linear_offset_fused(x, inv_m, s_tok, z_tok, wq, rowsum, s_w, bias, B, L, y=None, acc_out=None, xq_out=None)\n--\n\n"
         "ptq4vm_w8a8_linear_offset_fused: y fp16 [B*L, N] from fp16 activations, per-token steps and zero offsets;\n"
         "acc_out (raw accumulators) / xq_out (codes with the offset in them) are filled if given."),
    FAST(w4a4_linear_fused, "w4a4_linear_fused(x, inv_m, s_tok, wq4, s_w, bias, B, L, y=None, acc_out=None, xq_out=None)\n--\n\n"
                            "ptq4vm_w4a4_linear_fused: y fp16 [B*L, N] from fp16 activations and a packed 4-bit weight [N, K/2];\n"
                            "acc_out / xq_out (int8, one 4-bit code per byte) are filled if given."),
    FAST(f16_linear, "f16_linear(x, w, bias, y=None)\n--\n\nptq4vm_f16_linear: y fp16 [M, N]."),
    {"bind", bind, METH_O, "bind(table)\n--\n\nAddresses of the library's entry points by name, without the ptq4vm_ prefix."},
    {"setup", setup, METH_VARARGS, "setup(load_library, raise_status)\n--\n\nCallbacks: load the library and bind(); raise for a status."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Launches of libptq4vm.so as Python callables.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    for (Signature *s : {&sig_quantize_pts, &sig_quantize_dynamic, &sig_quantize_pts_offset, &sig_quantize_pts_a4, &sig_quantize_pts_a4_e2m3,
                         &sig_w8a8_linear, &sig_w8a8_linear_offset, &sig_w4a4_linear, &sig_w4a4_linear_e2m3, &sig_w8a8_linear_fused,
                         &sig_w8a8_linear_offset_fused, &sig_w4a4_linear_fused, &sig_f16_linear})
        for (int i = 0; i < s->total; i++) s->interned[i] = PyUnicode_InternFromString(s->names[i]);
    return PyModule_Create(&module);
}
