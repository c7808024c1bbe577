// What a device call of binding.py does before the library's function, without the interpreter: the tensors' types and sizes, the current
// stream, the call.  A Python extension module; binding.py has the same in Python and is what decides.
//
// What bounds an eager call: the host.  Of 4.65 us for spqt_gather and 6.2 for spqt_gemv 2.7 were the launch inside the runtime; five tensors
// with five attribute reads each, the size formulas, ctypes and its structure were the rest.  Here they take 0.3 to 0.6 (a gather and a GEMV,
// 512 x 1024: 11.0 us in Python, 6.8 here; 4 of each on 11001 x 4224, with the GPU's share, 45.7 / 34.3).
//
// Every function returns the library's status, or None where anything is other than what it knows for certain - a tensor that is not plainly a
// dense one of the type asked for, another size, an int or a threshold of another type, a stream given, a torch-function mode, which the Python code's reads of
// the tensors would reach - and then has done nothing.  The caller goes on with the Python code, which accepts or refuses as it always did.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "spqt.h"
#include "spqt_colblock.h"

namespace {

struct NotPlain {};      // anything that the Python code is to look at

// A dense tensor on the GPU, in memory order, of this type.
const at::Tensor &tensor(PyObject *o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) throw NotPlain();
    const at::Tensor &t = THPVariable_Unpack(o);
    const c10::TensorImpl *impl = t.unsafeGetTensorImpl();
    if (!t.defined() || impl->is_python_dispatch() || !impl->has_storage() || t.layout() != at::kStrided || !t.is_cuda() || t.scalar_type() != type ||
        !t.is_contiguous())
        throw NotPlain();
    return t;
}
int64_t whole(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw NotPlain();
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw NotPlain();
    return v;
}
int small(PyObject *o) {
    const int64_t v = whole(o);
    if (v < -(1 << 30) || v > (1 << 30)) throw NotPlain();
    return (int)v;
}
float threshold(PyObject *o) {
    if (!PyFloat_CheckExact(o)) throw NotPlain();
    return (float)PyFloat_AS_DOUBLE(o);
}
void *current_stream(PyObject *o) {
    if (o != Py_None) throw NotPlain();
    return c10::hip::getCurrentHIPStream().stream();
}
template <class F>
F function(PyObject *o) {
    void *p = PyLong_AsVoidPtr(o);
    if (!p) throw NotPlain();
    return reinterpret_cast<F>(p);
}

// The packed matrix: chunks of `chunk` bytes for `high` x `columns` weights.
void *packed_matrix(PyObject *o, int64_t M, int64_t K, int64_t high, int64_t columns, int64_t chunk) {
    const at::Tensor &t = tensor(o, at::kByte);
    if (M <= 0 || M > 1 << 24 || K <= 0 || K > 1 << 24 || K % SPQT_GROUP != 0 || (columns != SPQT_GROUP && columns != SPQT_GROUP / 2)) throw NotPlain();
    if (t.numel() < (M + high - 1) / high * (K / columns) * chunk) throw NotPlain();
    return t.data_ptr();
}

struct Output {
    void *p;
    int64_t n;
    int flags;
};
Output output(PyObject *o) {
    const bool half = THPVariable_CheckExact(o) && THPVariable_Unpack(o).scalar_type() == at::kHalf;
    const at::Tensor &t = tensor(o, half ? at::kHalf : at::kFloat);
    return {t.data_ptr(), t.numel(), half ? SPQT_CFG_Y_FP16 : 0};
}
struct Space {
    void *p = nullptr;
    size_t n = 0;
};
Space workspace(PyObject *o) {
    if (o == Py_None) return {};
    const at::Tensor &t = tensor(o, at::kByte);
    return {t.data_ptr(), (size_t)t.numel()};
}
struct List {
    const int32_t *idx = nullptr, *count = nullptr;
};
List list(PyObject *idx, PyObject *count) {
    if (idx == Py_None) return {};
    return {(const int32_t *)tensor(idx, at::kInt).data_ptr(), (const int32_t *)tensor(count, at::kInt).data_ptr()};
}
// x[K] or x[batch][K]
struct Rows {
    void *p;
    int batch;
    int64_t K;
};
Rows rows(PyObject *o) {
    const at::Tensor &t = tensor(o, at::kHalf);
    if (t.dim() != 1 && t.dim() != 2) throw NotPlain();
    const int64_t batch = t.dim() == 1 ? 1 : t.size(0);
    if (batch < 1 || batch > SPQT_MAX_BATCH) throw NotPlain();
    return {t.data_ptr(), (int)batch, t.size(t.dim() - 1)};
}

template <class Body>
PyObject *guarded(Py_ssize_t given, Py_ssize_t expected, Body body) {
    if (given != expected) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        if (at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        return PyLong_FromLong(body());
    } catch (...) {                       // NotPlain, and whatever torch throws at a tensor without memory
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
// The library's function, with the interpreter free for other threads as ctypes leaves it.
template <class F, class... A>
int call(F f, A... a) {
    PyThreadState *held = PyEval_SaveThread();
    const int rc = f(a...);
    PyEval_RestoreThread(held);
    return rc;
}

// gather(function, x, threshold, idx_out, count_out, stream)
PyObject *gather(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 6, [&]() {
        const Rows x = rows(a[1]);
        const at::Tensor &idx = tensor(a[3], at::kInt), &count = tensor(a[4], at::kInt);
        if (idx.numel() < x.K || count.numel() < 1) throw NotPlain();
        return call(function<decltype(&spqt_gather)>(a[0]), x.p, x.K, x.batch, threshold(a[2]), (int32_t *)idx.data_ptr(), (int32_t *)count.data_ptr(),
                    current_stream(a[5]));
    });
}
// gather_rows(function, x, threshold, idx_out, count_out, x_masked_out, stream)
PyObject *gather_rows(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 7, [&]() {
        const Rows x = rows(a[1]);
        const at::Tensor &idx = tensor(a[3], at::kInt), &count = tensor(a[4], at::kInt), &masked = tensor(a[5], at::kHalf);
        if (idx.numel() < x.K || count.numel() < 1 || masked.numel() != x.batch * x.K) throw NotPlain();
        return call(function<decltype(&spqt_gather_rows)>(a[0]), x.p, x.K, x.batch, threshold(a[2]), (int32_t *)idx.data_ptr(),
                    (int32_t *)count.data_ptr(), masked.data_ptr(), current_stream(a[6]));
    });
}
// The launch configuration of a call: splits and waves, and the flags with the output's type.
spqt_launch_cfg config(PyObject *splits, PyObject *waves, int flags) {
    spqt_launch_cfg c;
    c.splits = small(splits);
    c.waves = small(waves);
    c.flags = flags;
    return c;
}
// gemv(function of spqt_gemv_ex's type, packed, M, K, x, idx, count, y, workspace, stream, group, splits, waves, flags)
PyObject *gemv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 14, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]), group = whole(a[10]);
        void *packed = packed_matrix(a[1], M, K, SPQT_TILE_ROWS, group, 2 * SPQT_TILE_ROWS + 128 * group);
        const Rows x = rows(a[4]);
        const Output y = output(a[7]);
        if (x.K != K || y.n != x.batch * M) throw NotPlain();
        const List l = list(a[5], a[6]);
        const Space ws = workspace(a[8]);
        const spqt_launch_cfg cfg = config(a[11], a[12], small(a[13]) | y.flags);
        return call(function<decltype(&spqt_gemv_ex)>(a[0]), packed, M, K, (int)group, x.p, x.batch, l.idx, l.count, y.p, ws.p, ws.n,
                    current_stream(a[9]), &cfg);
    });
}

// gemv_fused(function, packed, M, K, x, threshold, y, workspace, stream, group, splits, waves, flags)
PyObject *gemv_fused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 13, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]), group = whole(a[9]);
        void *packed = packed_matrix(a[1], M, K, SPQT_TILE_ROWS, group, 2 * SPQT_TILE_ROWS + 128 * group);
        const at::Tensor &x = tensor(a[4], at::kHalf);
        const Output y = output(a[6]);
        if (x.numel() != K || y.n != M) throw NotPlain();
        const Space ws = workspace(a[7]);
        const spqt_launch_cfg cfg = config(a[10], a[11], small(a[12]) | y.flags);
        return call(function<decltype(&spqt_gemv_fused)>(a[0]), packed, M, K, (int)group, x.data_ptr(), threshold(a[5]), y.p, ws.p, ws.n,
                    current_stream(a[8]), &cfg);
    });
}
// gemv_fused_rows(function, packed, M, K, x, threshold, own_sets, y, workspace, stream, group, splits, waves)
PyObject *gemv_fused_rows(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 13, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]), group = whole(a[10]);
        void *packed = packed_matrix(a[1], M, K, SPQT_TILE_ROWS, group, 2 * SPQT_TILE_ROWS + 128 * group);
        const Rows x = rows(a[4]);
        const Output y = output(a[7]);
        if (x.K != K || y.n != x.batch * M || !PyBool_Check(a[6])) throw NotPlain();
        const Space ws = workspace(a[8]);
        const spqt_launch_cfg cfg = config(a[11], a[12], y.flags);
        return call(function<decltype(&spqt_gemv_fused_rows)>(a[0]), packed, M, K, (int)group, x.p, x.batch, threshold(a[5]), (int)(a[6] == Py_True), y.p,
                    ws.p, ws.n, current_stream(a[9]), &cfg);
    });
}
// The column-block layouts, whose rows per block-row and bytes per chunk come with the call.
// cb_gemv(function, packed, M, K, x, idx, count, y, workspace, stream, splits, waves, high, chunk)
PyObject *cb_gemv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 14, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]);
        void *packed = packed_matrix(a[1], M, K, whole(a[12]), SPQT_GROUP, whole(a[13]));
        const Rows x = rows(a[4]);
        const Output y = output(a[7]);
        if (x.K != K || y.n != x.batch * M) throw NotPlain();
        const List l = list(a[5], a[6]);
        const Space ws = workspace(a[8]);
        const spqt_launch_cfg cfg = config(a[10], a[11], y.flags);
        return call(function<decltype(&spqt_cb_gemv)>(a[0]), packed, M, K, x.p, x.batch, l.idx, l.count, y.p, ws.p, ws.n, current_stream(a[9]), &cfg);
    });
}
// cb_gemv_one(the same): the functions that take one activation row
PyObject *cb_gemv_one(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 14, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]);
        void *packed = packed_matrix(a[1], M, K, whole(a[12]), SPQT_GROUP, whole(a[13]));
        const at::Tensor &x = tensor(a[4], at::kHalf);
        const Output y = output(a[7]);
        if (x.numel() != K || y.n != M) throw NotPlain();
        const List l = list(a[5], a[6]);
        const Space ws = workspace(a[8]);
        const spqt_launch_cfg cfg = config(a[10], a[11], y.flags);
        return call(function<decltype(&spqt_cb8_gemv)>(a[0]), packed, M, K, x.data_ptr(), l.idx, l.count, y.p, ws.p, ws.n, current_stream(a[9]), &cfg);
    });
}
// cb_gemv_fused(function, packed, M, K, x, threshold, y, workspace, stream, splits, waves, high, chunk)
PyObject *cb_gemv_fused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded(n, 13, [&]() {
        const int64_t M = whole(a[2]), K = whole(a[3]);
        void *packed = packed_matrix(a[1], M, K, whole(a[11]), SPQT_GROUP, whole(a[12]));
        const at::Tensor &x = tensor(a[4], at::kHalf);
        const Output y = output(a[6]);
        if (x.numel() != K || y.n != M) throw NotPlain();
        const Space ws = workspace(a[7]);
        const spqt_launch_cfg cfg = config(a[9], a[10], y.flags);
        return call(function<decltype(&spqt_cb_gemv_fused)>(a[0]), packed, M, K, x.data_ptr(), threshold(a[5]), y.p, ws.p, ws.n, current_stream(a[8]),
                    &cfg);
    });
}

#define SPQT_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SPQT_METHOD(gather),  SPQT_METHOD(gather_rows), SPQT_METHOD(gemv),         SPQT_METHOD(gemv_fused), SPQT_METHOD(gemv_fused_rows),
                         SPQT_METHOD(cb_gemv), SPQT_METHOD(cb_gemv_one), SPQT_METHOD(cb_gemv_fused), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", "Device calls of binding.py without the interpreter.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
    PyObject *m = PyModule_Create(&module);
    // binding.py uses the module only with the torch whose headers it was compiled against
    if (m && PyModule_AddStringConstant(m, "torch_version", SPQT_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
