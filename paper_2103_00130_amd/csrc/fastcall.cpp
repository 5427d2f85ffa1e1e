// The two calls that a serving loop makes for every layer and every lookup, marshalled natively: the operands of
// abft_gemm_u8s8s32_checked and abft_eb_u8_checked are unpacked from torch tensors here and handed to the C ABI, whose
// addresses bind() receives.  What binding.py checks is checked here too, and whatever does not pass - another type, a wrong
// shape, a tensor subclass - is left to it: the function returns None, and the Python code that follows raises what it
// always raised.  A call took 9.3-10 us of host time through ctypes, more than most of the kernels it launches run.
// The interpreter lock is released around the library call, as ctypes does.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/abft_eb.h"
#include "../../include/abft_gemm.h"

namespace {

decltype(&abft_gemm_u8s8s32_checked) g_gemm = nullptr;
decltype(&abft_eb_u8_checked) g_eb = nullptr;
PyObject* g_current_device = nullptr;  // () -> int
PyObject* g_raw_stream = nullptr;      // (device) -> the current stream of that device, as an integer
PyObject* g_cuda_stream = nullptr;     // the attribute name of an explicit stream

struct Leave {};  // "not mine": the caller's Python code takes over

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) throw Leave{};
    return THPVariable_Unpack(o);
}

// a device tensor of the given type, or null for None
const at::Tensor* operand(PyObject* o, at::ScalarType type) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided) throw Leave{};
    return &t;
}
const at::Tensor& needed(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = operand(o, type);
    if (!t) throw Leave{};
    return *t;
}

template <typename T>
T* ptr(const at::Tensor* t) {
    return t ? static_cast<T*>(t->data_ptr()) : nullptr;
}

// leading dimension of a matrix with unit column stride
int64_t leading(const at::Tensor& t) {
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) throw Leave{};
    return t.size(0) > 1 ? t.stride(0) : std::max(t.stride(0), t.size(1));
}

void entries(const at::Tensor* t, int64_t at_least, bool contiguous) {
    if (t && (t->numel() < at_least || (contiguous && !t->is_contiguous()))) throw Leave{};
}

long long integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw Leave{};
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over) throw Leave{};
    return v;
}

void* handle(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw Leave{};
    void* const h = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Leave{};
    }
    return h;
}

void* stream(PyObject* o) {
    PyObject* v = nullptr;
    if (o == Py_None) {
        PyObject* const dev = PyObject_CallNoArgs(g_current_device);
        if (dev) {
            v = PyObject_CallOneArg(g_raw_stream, dev);
            Py_DECREF(dev);
        }
    } else {
        v = PyObject_GetAttr(o, g_cuda_stream);
    }
    if (!v || !PyLong_Check(v)) {
        Py_XDECREF(v);
        PyErr_Clear();
        throw Leave{};
    }
    void* const s = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Leave{};
    }
    return s;
}

// gemm(A, handle, K, N, C, row_flags, err_count, rq, Cq, inj, n_inj, flags, workspace, stream) -> return code, or None.
// rq: an abft_requant_t of the binding (its bytes are the struct), or None
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Py_buffer rq_bytes;
    bool have_rq = false;
    int rc = 0;
    try {
        if (n != 14 || !g_gemm) throw Leave{};
        const at::Tensor& A = needed(a[0], at::kByte);
        const int64_t lda = leading(A), M = A.size(0), K = integer(a[2]), N = integer(a[3]);
        if (A.size(1) != K || M > 0x7fffffff) throw Leave{};
        const at::Tensor *C = operand(a[4], at::kInt), *flags_out = operand(a[5], at::kInt), *count = operand(a[6], at::kInt);
        const at::Tensor *Cq = operand(a[8], at::kByte), *inj = operand(a[9], at::kInt);
        int64_t ldc = 0, ldcq = 0;
        if (C) {
            ldc = leading(*C);
            if (C->size(0) != M || C->size(1) != N) throw Leave{};
        }
        if (Cq) {
            ldcq = leading(*Cq);
            if (Cq->size(0) != M || Cq->size(1) != N) throw Leave{};
        }
        const long long n_inj = integer(a[10]), flags = integer(a[11]);
        if (n_inj < -0x80000000ll || n_inj > 0x7fffffffll || flags < 0 || flags > 0xffffffffll) throw Leave{};
        entries(flags_out, M, false);
        entries(inj, 3 * n_inj, false);
        void* ws = nullptr;
        size_t ws_bytes = 0;
        if (a[12] != Py_None) {
            const at::Tensor& w = tensor(a[12]);
            ws = w.data_ptr();
            ws_bytes = (size_t)w.numel() * w.element_size();
        }
        void* const Bp = handle(a[1]);
        void* const s = stream(a[13]);
        if (a[7] != Py_None) {
            if (PyObject_GetBuffer(a[7], &rq_bytes, PyBUF_SIMPLE) != 0) {
                PyErr_Clear();
                throw Leave{};
            }
            have_rq = true;
            if (rq_bytes.len != (Py_ssize_t)sizeof(abft_requant_t)) throw Leave{};
        }
        const uint8_t* const A_ptr = ptr<uint8_t>(&A);
        int32_t *const C_ptr = ptr<int32_t>(C), *const flags_ptr = ptr<int32_t>(flags_out), *const count_ptr = ptr<int32_t>(count);
        uint8_t* const Cq_ptr = ptr<uint8_t>(Cq);
        const abft_inject_t* const inj_ptr = ptr<abft_inject_t>(inj);
        const abft_requant_t* const rq = have_rq ? static_cast<const abft_requant_t*>(rq_bytes.buf) : nullptr;
        Py_BEGIN_ALLOW_THREADS
        rc = g_gemm(A_ptr, lda, (int)M, static_cast<const abft_packed_b*>(Bp), C_ptr, ldc, flags_ptr, count_ptr, rq, Cq_ptr, ldcq,
                    inj_ptr, (int)n_inj, (uint32_t)flags, ws, ws_bytes, s);
        Py_END_ALLOW_THREADS
    } catch (...) {   // (a tensor without storage throws from data_ptr)
        if (have_rq) PyBuffer_Release(&rq_bytes);
        Py_RETURN_NONE;
    }
    if (have_rq) PyBuffer_Release(&rq_bytes);
    return PyLong_FromLong(rc);
}

// eb(handle, d, indices, offsets, R, bag_flags, weights, rsum, csum, rel_bound, flags, stream) -> return code, or None
PyObject* eb(PyObject*, PyObject* const* a, Py_ssize_t n) {
    int rc = 0;
    try {
        if (n != 12 || !g_eb) throw Leave{};
        const at::Tensor &indices = needed(a[2], at::kLong), &offsets = needed(a[3], at::kLong), &R = needed(a[4], at::kFloat);
        const int64_t n_bags = offsets.numel() - 1, n_indices = indices.numel();
        if (n_bags < 0 || !offsets.is_contiguous() || !indices.is_contiguous()) throw Leave{};
        const int64_t ldr = leading(R);
        if (R.size(0) < n_bags || R.size(1) != integer(a[1])) throw Leave{};
        const at::Tensor *bag_flags = operand(a[5], at::kInt), *weights = operand(a[6], at::kFloat);
        const at::Tensor *rsum = operand(a[7], at::kDouble), *csum = operand(a[8], at::kDouble);
        entries(bag_flags, n_bags, true);
        entries(rsum, n_bags, true);
        entries(csum, n_bags, true);
        if (weights && (weights->numel() != n_indices || !weights->is_contiguous())) throw Leave{};
        if (!PyFloat_CheckExact(a[9])) throw Leave{};
        const double bound = PyFloat_AS_DOUBLE(a[9]);
        const long long flags = integer(a[10]);
        if (flags < 0 || flags > 0xffffffffll) throw Leave{};
        void* const Tp = handle(a[0]);
        void* const s = stream(a[11]);
        const int64_t *const idx_ptr = ptr<int64_t>(&indices), *const off_ptr = ptr<int64_t>(&offsets);
        const float* const w_ptr = ptr<float>(weights);
        float* const R_ptr = ptr<float>(&R);
        int32_t* const f_ptr = ptr<int32_t>(bag_flags);
        double *const rs_ptr = ptr<double>(rsum), *const cs_ptr = ptr<double>(csum);
        Py_BEGIN_ALLOW_THREADS
        rc = g_eb(static_cast<const abft_eb_table*>(Tp), idx_ptr, n_indices, off_ptr, n_bags, w_ptr, R_ptr, ldr, f_ptr, rs_ptr, cs_ptr,
                  bound, (unsigned)flags, s);
        Py_END_ALLOW_THREADS
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

// bind(address of abft_gemm_u8s8s32_checked, address of abft_eb_u8_checked, current_device, raw_stream)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *gemm_at, *eb_at, *device, *raw;
    if (!PyArg_ParseTuple(args, "OOOO", &gemm_at, &eb_at, &device, &raw)) return nullptr;
    void *const g = PyLong_AsVoidPtr(gemm_at), *const e = PyLong_AsVoidPtr(eb_at);
    if (PyErr_Occurred()) return nullptr;
    g_gemm = reinterpret_cast<decltype(g_gemm)>(g);
    g_eb = reinterpret_cast<decltype(g_eb)>(e);
    Py_INCREF(device);
    Py_INCREF(raw);
    Py_XSETREF(g_current_device, device);
    Py_XSETREF(g_raw_stream, raw);
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, "abft_gemm_u8s8s32_checked on torch tensors; None when the operands are not what it takes"},
    {"eb", (PyCFunction)(void (*)(void))eb, METH_FASTCALL, "abft_eb_u8_checked on torch tensors; None when the operands are not what it takes"},
    {"bind", bind, METH_VARARGS, "addresses of the library's functions, and where to ask for the current device and stream"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", "native marshalling of the two calls of a serving loop", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return g_cuda_stream ? PyModule_Create(&g_module) : nullptr;
}
