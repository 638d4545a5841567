// Native half of the Python binding: argument checks, output allocation and the call into the C boundary for the entry
// points that run once per layer and token.
//
// At decode sizes a layer is two short kernels, about 10 us on the GPU, and marshalling the same call in Python (tensor
// attributes one by one, a ctypes call with fifteen arguments, two torch.empty) took 14 us of host time: the GPU waited
// for the interpreter.  Read straight from the tensor objects the call takes about a third of that, most of it the HIP
// launches.  Nothing here computes: a status other than SALR_OK comes back as the binding's SalrError.
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "salr.h"
#include "salr_internal.hpp"   // the two halves of the encoder

namespace {

PyObject* g_salr_error = nullptr;   // class SalrError(status, where), handed over by the package

enum Kind { kBf16, kU32, kU8 };

// Thrown once a Python error is set.
struct PyFailure {};

[[noreturn]] void fail(PyObject* type, const char* fmt, const char* name) {
    PyErr_Format(type, fmt, name);
    throw PyFailure{};
}

bool dtype_ok(at::ScalarType t, Kind kind) {
    switch (kind) {
        case kBf16: return t == at::kBFloat16 || t == at::kShort || t == at::kUInt16;
        case kU32: return t == at::kInt || t == at::kUInt32;
        default: return t == at::kByte;
    }
}

// A tensor argument; None gives an undefined tensor.
const at::Tensor& tensor_of(PyObject* o, const char* name) {
    static const at::Tensor none;
    if (o == Py_None) return none;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a tensor", name);
    return THPVariable_Unpack(o);
}

template <typename T>
T* device_ptr(const at::Tensor& t, Kind kind, const char* name) {
    if (!t.defined()) return nullptr;
    if (!t.is_cuda()) fail(PyExc_TypeError, "%s must be a CUDA tensor", name);
    if (!dtype_ok(t.scalar_type(), kind)) fail(PyExc_TypeError, "%s: unexpected dtype", name);
    if (!t.is_contiguous()) fail(PyExc_TypeError, "%s must be contiguous", name);
    return t.numel() > 0 ? static_cast<T*>(t.data_ptr()) : nullptr;
}

void need_matrix(const at::Tensor& t, const char* name) {
    if (!t.defined() || t.dim() != 2) fail(PyExc_ValueError, "%s must be a matrix", name);
}

void* stream_of(PyObject* o) {   // None: the current stream; else a stream handle as an integer (0 = default stream)
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    void* p = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) throw PyFailure{};
    return p;
}

at::Tensor empty_on(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
    return at::Tensor(at::detail::empty_cuda(shape, type, like.device(), std::nullopt));
}

void check(salr_status_t st, const char* where) {
    if (st == SALR_OK) return;
    PyObject* e = g_salr_error ? PyObject_CallFunction(g_salr_error, "is", (int)st, where) : nullptr;
    if (e) {
        PyErr_SetObject(g_salr_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s: status %d", where, (int)st);
    }
    throw PyFailure{};
}

struct Gil {   // the launches run without the interpreter's lock
    PyThreadState* s = PyEval_SaveThread();
    ~Gil() { PyEval_RestoreThread(s); }
};

// The weight and adapter arguments that every form of the layer shares.
struct Layer {
    int64_t M, K, N, R;
    const uint32_t* bitmap;
    const uint32_t* offsets;
    const uint16_t* a;
    const uint16_t* b;

    Layer(int64_t m, int64_t k, int64_t n, PyObject* bitmap_o, PyObject* offsets_o, PyObject* a_o, PyObject* b_o)
        : M(m), K(k), N(n) {
        const at::Tensor &bm = tensor_of(bitmap_o, "bitmap"), &ro = tensor_of(offsets_o, "row_offsets");
        const at::Tensor &ta = tensor_of(a_o, "a_cat"), &tb = tensor_of(b_o, "b_cat");
        R = ta.defined() ? (need_matrix(ta, "a_cat"), ta.size(1)) : 0;
        if (!bm.defined() || bm.dim() < 1 || bm.size(0) != N || !ro.defined() || ro.numel() != N + 1)
            fail(PyExc_ValueError, "inconsistent %s", "shapes");
        if (R > 0 && (ta.size(0) != K || !tb.defined() || tb.dim() != 2 || tb.size(0) != R || tb.size(1) != N))
            fail(PyExc_ValueError, "adapter %s", "shapes");
        bitmap = device_ptr<uint32_t>(bm, kU32, "bitmap");
        offsets = device_ptr<uint32_t>(ro, kU32, "row_offsets");
        a = device_ptr<uint16_t>(ta, kBf16, "a_cat");
        b = device_ptr<uint16_t>(tb, kBf16, "b_cat");
    }
};

// The caller's workspace, or one of `need` bytes for the length of the call (torch's allocator hands the memory to later
// work of the same stream only).
struct Workspace {
    at::Tensor own;
    void* ptr = nullptr;
    size_t bytes = 0;

    void given(PyObject* o) {
        const at::Tensor& t = tensor_of(o, "workspace");
        if (!t.defined()) return;
        ptr = t.data_ptr();
        bytes = (size_t)t.numel() * t.element_size();
    }
    void allocate(size_t need, const at::Tensor& like) {
        if (need == 0) return;
        own = empty_on({(int64_t)need}, at::kByte, like);
        ptr = own.data_ptr();
        bytes = need;
    }
    // The size with which the call is fastest, unless the caller's is that large.  The call runs without it: where the allocator
    // has no more, on the caller's workspace or, where that is none, on one of the size the query tells.
    void fastest(size_t want, size_t told, const at::Tensor& like, bool have_given) {
        if (have_given && bytes >= want) return;
        try {
            allocate(want, like);
        } catch (const c10::OutOfMemoryError&) {
            if (have_given) return;
            if (told >= want) throw;
            allocate(told, like);
        }
    }
};

// y of the call: the caller's, or a new [M, N] tensor of x's type
at::Tensor output_of(PyObject* y_o, const at::Tensor& x, int64_t N) {
    if (y_o != Py_None) return tensor_of(y_o, "y");
    if (!x.is_cuda()) fail(PyExc_TypeError, "%s must be a CUDA tensor", "x");
    return empty_on({x.size(0), N}, x.scalar_type(), x);
}

int64_t rows_of(PyObject* bitmap_o) {
    const at::Tensor& t = tensor_of(bitmap_o, "bitmap");
    if (!t.defined() || t.dim() < 1) fail(PyExc_ValueError, "inconsistent %s", "shapes");
    return t.size(0);
}

PyObject* result(PyObject* y_o, at::Tensor&& y) {
    if (y_o != Py_None) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(y));
}

void need_args(Py_ssize_t n, Py_ssize_t want, const char* name) {
    if (n != want) fail(PyExc_TypeError, "%s: wrong number of arguments", name);
}

#define SALR_TRY HANDLE_TH_ERRORS try {
#define SALR_CATCH                        \
    } catch (const PyFailure&) {          \
        return nullptr;                   \
    }                                     \
    END_HANDLE_TH_ERRORS

// linear(form, x, bitmap, values, row_offsets, slice_table, a_cat, b_cat, y, workspace, stream)
//   form  0 plain, 1 with the slice table, 2 two-of-four; y None: allocated and returned, and so is a workspace for the length
//   of the call where the caller's is none or smaller than the fastest path wants
PyObject* py_linear(PyObject*, PyObject* const* v, Py_ssize_t n) {
    SALR_TRY
    need_args(n, 11, "linear");
    const long form = PyLong_AsLong(v[0]);
    const at::Tensor& x = tensor_of(v[1], "x");
    need_matrix(x, "x");
    const at::Tensor& values = tensor_of(v[3], "values");
    at::Tensor y = output_of(v[8], x, v[8] == Py_None ? rows_of(v[2]) : 0);
    need_matrix(y, "y");
    if (y.size(0) != x.size(0)) fail(PyExc_ValueError, "inconsistent %s", "shapes");
    const Layer l(x.size(0), x.size(1), y.size(1), v[2], v[4], v[6], v[7]);
    const uint16_t* xp = device_ptr<uint16_t>(x, kBf16, "x");
    const uint16_t* vp = device_ptr<uint16_t>(values, kBf16, "values");
    uint16_t* yp = device_ptr<uint16_t>(y, kBf16, "y");
    const uint32_t* table = nullptr;
    if (form == 1) {
        const at::Tensor& st = tensor_of(v[5], "slice_table");
        if (!st.defined() || st.numel() != l.N * 16) fail(PyExc_ValueError, "inconsistent %s", "shapes");
        table = device_ptr<uint32_t>(st, kU32, "slice_table");
    }
    Workspace ws;
    ws.given(v[9]);
    if (v[8] == Py_None) {   // (a call that brings its y allocates nothing)
        // Less than the query tells is the caller's choice of the path without a decoded weight.
        const size_t told = form == 2 ? salr_linear_2of4_workspace_bytes(l.M, l.K, l.N, l.R) : salr_linear_workspace_bytes(l.M, l.K, l.N, l.R);
        if (v[9] == Py_None || ws.bytes >= told)
            ws.fastest(form == 2 ? salr_linear_2of4_workspace_bytes_fastest(l.M, l.K, l.N, l.R)
                                 : salr_linear_workspace_bytes_fastest(l.M, l.K, l.N, l.R),
                       told, x, v[9] != Py_None);
    }
    void* stream = stream_of(v[10]);
    salr_status_t st;
    {
        Gil release;
        st = form == 1   ? salr_sparse_lowrank_linear_prepared(xp, l.M, l.K, l.N, l.bitmap, vp, l.offsets, table, l.a, l.b, l.R, yp,
                                                               ws.ptr, ws.bytes, stream)
             : form == 2 ? salr_sparse_lowrank_linear_2of4(xp, l.M, l.K, l.N, l.bitmap, vp, l.offsets, l.a, l.b, l.R, yp, ws.ptr,
                                                           ws.bytes, stream)
                         : salr_sparse_lowrank_linear(xp, l.M, l.K, l.N, l.bitmap, vp, l.offsets, l.a, l.b, l.R, yp, ws.ptr, ws.bytes,
                                                      stream);
    }
    check(st, form == 1 ? "salr_sparse_lowrank_linear_prepared" : form == 2 ? "salr_sparse_lowrank_linear_2of4" : "salr_sparse_lowrank_linear");
    return result(v[8], std::move(y));
    SALR_CATCH
}

// qsalr_linear(x, bitmap, codes, scales, row_offsets, nnz, a_cat, b_cat, y, workspace, stream)
PyObject* py_qsalr_linear(PyObject*, PyObject* const* v, Py_ssize_t n) {
    SALR_TRY
    need_args(n, 11, "qsalr_linear");
    const at::Tensor& x = tensor_of(v[0], "x");
    need_matrix(x, "x");
    const int64_t nnz = PyLong_AsLongLong(v[5]);
    if (nnz == -1 && PyErr_Occurred()) throw PyFailure{};
    at::Tensor y = output_of(v[8], x, v[8] == Py_None ? rows_of(v[1]) : 0);
    need_matrix(y, "y");
    if (y.size(0) != x.size(0)) fail(PyExc_ValueError, "inconsistent %s", "shapes");
    const Layer l(x.size(0), x.size(1), y.size(1), v[1], v[4], v[6], v[7]);
    const uint16_t* xp = device_ptr<uint16_t>(x, kBf16, "x");
    const uint8_t* cp = device_ptr<uint8_t>(tensor_of(v[2], "codes"), kU8, "codes");
    const uint16_t* sp = device_ptr<uint16_t>(tensor_of(v[3], "scales"), kBf16, "scales");
    uint16_t* yp = device_ptr<uint16_t>(y, kBf16, "y");
    Workspace ws;
    ws.given(v[9]);
    if (v[9] == Py_None && v[8] == Py_None) {
        const size_t told = salr_qsalr_linear_workspace_bytes(l.M, l.K, l.N, l.R, nnz);
        const size_t want = salr_qsalr_linear_workspace_bytes_fastest(l.M, l.K, l.N, l.R, nnz);
        ws.fastest(want < 256 ? 256 : want, told < 256 ? 256 : told, x, false);
    }
    void* stream = stream_of(v[10]);
    salr_status_t st;
    {
        Gil release;
        st = salr_qsalr_linear(xp, l.M, l.K, l.N, l.bitmap, cp, sp, l.offsets, nnz, l.a, l.b, l.R, yp, ws.ptr, ws.bytes, stream);
    }
    check(st, "salr_qsalr_linear");
    return result(v[8], std::move(y));
    SALR_CATCH
}

// linear_backward(x, dy, bitmap, values, row_offsets, a_cat, b_cat, need_dx, need_dadb) -> (dx, da, db)
PyObject* py_linear_backward(PyObject*, PyObject* const* v, Py_ssize_t n) {
    SALR_TRY
    need_args(n, 9, "linear_backward");
    const at::Tensor &x = tensor_of(v[0], "x"), &dy = tensor_of(v[1], "dy"), &bm = tensor_of(v[2], "bitmap");
    need_matrix(dy, "dy");
    need_matrix(bm, "bitmap");
    const Layer l(dy.size(0), bm.size(1) * 32, dy.size(1), v[2], v[4], v[5], v[6]);
    const bool need_dx = PyObject_IsTrue(v[7]) == 1, need_g = PyObject_IsTrue(v[8]) == 1 && l.R > 0;
    if (x.defined() && (x.dim() != 2 || x.size(0) != l.M || x.size(1) != l.K)) fail(PyExc_ValueError, "%s must be [M, K]", "x");
    const uint16_t* xp = device_ptr<uint16_t>(x, kBf16, "x");
    const uint16_t* dyp = device_ptr<uint16_t>(dy, kBf16, "dy");
    const uint16_t* vp = device_ptr<uint16_t>(tensor_of(v[3], "values"), kBf16, "values");
    if (!dy.is_cuda()) fail(PyExc_TypeError, "%s must be a CUDA tensor", "dy");
    at::Tensor dx, da, db;
    if (need_dx) dx = empty_on({l.M, l.K}, dy.scalar_type(), dy);
    if (need_g) {
        da = empty_on({l.K, l.R}, dy.scalar_type(), dy);
        db = empty_on({l.R, l.N}, dy.scalar_type(), dy);
    }
    Workspace ws;
    const size_t need = salr_linear_backward_workspace_bytes(l.M, l.K, l.N, l.R, need_dx, need_g);
    ws.allocate(need < 256 ? 256 : need, dy);
    void* stream = stream_of(Py_None);
    uint16_t *dxp = device_ptr<uint16_t>(dx, kBf16, "dx"), *dap = device_ptr<uint16_t>(da, kBf16, "da"),
             *dbp = device_ptr<uint16_t>(db, kBf16, "db");
    salr_status_t st;
    {
        Gil release;
        st = salr_sparse_lowrank_linear_backward(xp, dyp, l.M, l.K, l.N, l.bitmap, vp, l.offsets, l.a, l.b, l.R, dxp, dap, dbp, ws.ptr,
                                                 ws.bytes, stream);
    }
    check(st, "salr_sparse_lowrank_linear_backward");
    PyObject* out = PyTuple_New(3);
    at::Tensor* grads[3] = {&dx, &da, &db};
    for (int i = 0; i < 3; ++i) {
        if (!grads[i]->defined()) Py_INCREF(Py_None);
        PyTuple_SET_ITEM(out, i, grads[i]->defined() ? THPVariable_Wrap(*grads[i]) : Py_None);
    }
    return out;
    SALR_CATCH
}

int64_t int_of(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFailure{};
    return v;
}

// A packed-values buffer of nnz elements whose storage is whole 16-byte vectors.
at::Tensor values_alloc(int64_t nnz, const at::Tensor& like) {
    const int64_t padded = (nnz + 7) / 8 * 8;
    return empty_on({padded < 8 ? 8 : padded}, at::kShort, like).narrow(0, 0, nnz);
}

// mask(w, n_keep, m_group, per_row) -> pruned copy; per_row: n_keep per row, m_group unused
PyObject* py_mask(PyObject*, PyObject* const* v, Py_ssize_t n) {
    SALR_TRY
    need_args(n, 4, "mask");
    const at::Tensor& w = tensor_of(v[0], "w");
    need_matrix(w, "w");
    const uint16_t* wp = device_ptr<uint16_t>(w, kBf16, "w");
    const int64_t keep = int_of(v[1]), group = int_of(v[2]);
    const bool per_row = PyObject_IsTrue(v[3]) == 1;
    if (!w.is_cuda()) fail(PyExc_TypeError, "%s must be a CUDA tensor", "w");
    at::Tensor out = empty_on(w.sizes(), w.scalar_type(), w);
    uint16_t* op = device_ptr<uint16_t>(out, kBf16, "w_hat");
    void* stream = stream_of(Py_None);
    salr_status_t st;
    {
        Gil release;
        st = per_row ? salr_magnitude_mask_rows(wp, w.size(0), w.size(1), keep, op, stream)
                        : salr_magnitude_mask_nm(wp, w.size(0), w.size(1), keep, group, op, stream);
    }
    check(st, per_row ? "salr_magnitude_mask_rows" : "salr_magnitude_mask_nm");
    return THPVariable_Wrap(std::move(out));
    SALR_CATCH
}

// encode(w) -> (bitmap, values, row_offsets).  `values` can only be sized once the nonzeros are counted: the encoder's
// first half leaves their number in pinned memory, the host waits for it once, and the second half follows.
PyObject* py_encode(PyObject*, PyObject* w_o) {
    SALR_TRY
    const at::Tensor& w = tensor_of(w_o, "w_dense");
    need_matrix(w, "w_dense");
    const uint16_t* wp = device_ptr<uint16_t>(w, kBf16, "w_dense");
    const int64_t rows = w.size(0), cols = w.size(1);
    if (!w.is_cuda()) fail(PyExc_TypeError, "%s must be a CUDA tensor", "w_dense");
    if (rows > 0x7FFFFFFFLL || cols > 0x7FFFFFFFLL - 31 || (cols > 0 && rows > 0xFFFFFFFFLL / cols)) check(SALR_ERR_SHAPE, "salr_encode_bitmap");
    at::Tensor bitmap = empty_on({rows, (cols + 31) / 32}, at::kInt, w), offsets = empty_on({rows + 1}, at::kInt, w);
    uint32_t *bp = device_ptr<uint32_t>(bitmap, kU32, "bitmap"), *rp = device_ptr<uint32_t>(offsets, kU32, "row_offsets");
    at::Tensor count = at::empty({1}, at::TensorOptions().dtype(at::kInt).pinned_memory(true));
    uint32_t* nnz_host = static_cast<uint32_t*>(count.data_ptr());
    hipStream_t stream = static_cast<hipStream_t>(stream_of(Py_None));
    hipError_t e;
    {
        Gil release;
        e = salr::launch_encode_index(wp, rows, cols, bp, rp, nnz_host, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
    }
    check(e == hipSuccess ? SALR_OK : SALR_ERR_HIP, "salr_encode_bitmap");
    const int64_t nnz = *static_cast<volatile uint32_t*>(nnz_host);
    at::Tensor values = values_alloc(nnz, w);
    e = nnz > 0 ? salr::launch_encode_values(wp, rows, cols, bp, rp, static_cast<uint16_t*>(values.data_ptr()), nnz, stream) : hipSuccess;
    check(e == hipSuccess ? SALR_OK : SALR_ERR_HIP, "salr_encode_bitmap");
    return Py_BuildValue("NNN", THPVariable_Wrap(std::move(bitmap)), THPVariable_Wrap(std::move(values)), THPVariable_Wrap(std::move(offsets)));
    SALR_CATCH
}

// decode(bitmap, values, row_offsets, rows, cols) -> [rows, cols] int16
PyObject* py_decode(PyObject*, PyObject* const* v, Py_ssize_t n) {
    SALR_TRY
    need_args(n, 5, "decode");
    const at::Tensor& bm = tensor_of(v[0], "bitmap");
    const uint32_t* bp = device_ptr<uint32_t>(bm, kU32, "bitmap");
    const uint16_t* vp = device_ptr<uint16_t>(tensor_of(v[1], "values"), kBf16, "values");
    const uint32_t* rp = device_ptr<uint32_t>(tensor_of(v[2], "row_offsets"), kU32, "row_offsets");
    const int64_t rows = int_of(v[3]), cols = int_of(v[4]);
    if (!bm.defined()) fail(PyExc_TypeError, "%s must be a tensor", "bitmap");
    at::Tensor out = empty_on({rows, cols}, at::kShort, bm);
    uint16_t* op = device_ptr<uint16_t>(out, kBf16, "w_dense_out");
    void* stream = stream_of(Py_None);
    salr_status_t st;
    {
        Gil release;
        st = salr_decode(bp, vp, rp, rows, cols, op, stream);
    }
    check(st, "salr_decode");
    return THPVariable_Wrap(std::move(out));
    SALR_CATCH
}

PyObject* py_set_error(PyObject*, PyObject* cls) {
    Py_XINCREF(cls);
    Py_XSETREF(g_salr_error, cls);
    Py_RETURN_NONE;
}

#define SALR_FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(fn)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    SALR_FAST("linear", py_linear),
    SALR_FAST("qsalr_linear", py_qsalr_linear),
    SALR_FAST("linear_backward", py_linear_backward),
    SALR_FAST("mask", py_mask),
    SALR_FAST("decode", py_decode),
    {"encode", py_encode, METH_O, nullptr},
    {"set_error", py_set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_salr_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__salr_binding() { return PyModule_Create(&kModule); }
