// The Python binding's usual call in native code: what binding.py's varlen_attn_fwd, varlen_attn_bwd and varlen_attn_merge do
// between being called and calling the library, for plain tensors that pass every check.  Anything else (a check that fails, a tensor
// subclass, a torch function mode, allocations for another stream) gets NotImplemented, and binding.py goes through its own
// checks, which name the fault.
//
// Why: the attention call on four samples of 246 tokens runs 7 us on the GPU; checks, parameter block, allocations and
// argument conversion in Python took 13 us per call, so that a program that makes such calls waited for its host.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/varlen_attn.h"

namespace {

decltype(&varlen_attn_fwd_workspace_bytes) fwd_workspace_bytes = nullptr;
decltype(&varlen_attn_bwd_workspace_bytes) bwd_workspace_bytes = nullptr;
decltype(&varlen_attn_fwd) attn_fwd = nullptr;
decltype(&varlen_attn_bwd) attn_bwd = nullptr;
decltype(&varlen_attn_merge) attn_merge = nullptr;

bool plain(PyObject* o) { return THPVariable_CheckExact(o); }
bool plain_or_none(PyObject* o) { return o == Py_None || plain(o); }
bool usable(const at::Tensor& t, at::ScalarType type) { return t.is_cuda() && t.scalar_type() == type && t.is_contiguous(); }
// A buffer of the caller's own (or none): the kernels go by its address, so it has to hold what they read or write there.
bool has_room(const at::Tensor& t, at::ScalarType type, int64_t elements) { return usable(t, type) && t.numel() >= elements; }
bool none_or_room(PyObject* o, at::ScalarType type, int64_t elements) {
    return o == Py_None || has_room(THPVariable_Unpack(o), type, elements);
}
bool none_or_scratch(PyObject* o) {  // (of any type: one byte an element is counted on)
    return o == Py_None || (THPVariable_Unpack(o).is_cuda() && THPVariable_Unpack(o).is_contiguous());
}
bool fits(int64_t x) { return x >= 0 && x <= INT32_MAX; }

// total_tokens, head counts and head_dim from q and k, the rest as given; false if something does not fit the block.
bool fill(varlen_attn_params& p, const at::Tensor& q, const at::Tensor& k, const at::Tensor& cu, int causal, double scale,
          long kv_splits, long max_seqlen) {
    if (q.dim() != 3 || k.dim() != 3 || !fits(q.size(0)) || !fits(q.size(1)) || !fits(q.size(2)) || !fits(k.size(1)) ||
        cu.numel() < 1 || !fits(cu.numel()) || kv_splits < INT32_MIN || kv_splits > INT32_MAX || max_seqlen < INT32_MIN ||
        max_seqlen > INT32_MAX)
        return false;
    p = varlen_attn_params{};
    p.total_tokens = (int32_t)q.size(0);
    p.num_seqs = (int32_t)(cu.numel() - 1);
    p.num_q_heads = (int32_t)q.size(1);
    p.num_kv_heads = (int32_t)k.size(1);
    p.head_dim = (int32_t)q.size(2);
    p.causal = causal;
    p.softmax_scale = (float)scale;
    p.max_seqlen = (int32_t)max_seqlen;
    p.kv_splits = (int32_t)kv_splits;
    return true;
}

at::Tensor given_or_like(PyObject* o, const at::Tensor& like) {
    return o == Py_None ? at::empty_like(like) : THPVariable_Unpack(o);
}
at::Tensor workspace_of(PyObject* o, size_t need, const at::Tensor& q) {
    return o == Py_None ? at::empty({(int64_t)(need < 16 ? 16 : need)}, q.options().dtype(at::kByte)) : THPVariable_Unpack(o);
}
bool stream_of(PyObject* o, void*& stream) {  // None: the current stream; else the handle as a number
    if (o == Py_None) {
        stream = (void*)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    stream = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}
// Whether a call that allocates has to leave it to binding.py: its kernels run on another stream than the one whose pool
// at::empty takes memory from (see _Allocating there).
bool elsewhere(PyObject* given, const void* stream, const at::Tensor& q) {
    return given != Py_None && stream != (void*)c10::hip::getCurrentHIPStream(q.device().index()).stream();
}
PyObject* not_implemented() { Py_RETURN_NOTIMPLEMENTED; }
PyObject* object_of(PyObject* given, const at::Tensor& t) { return given == Py_None ? THPVariable_Wrap(t) : (Py_INCREF(given), given); }
PyObject* pair(PyObject* given_a, const at::Tensor& a, PyObject* given_b, const at::Tensor& b) {
    PyObject *x = object_of(given_a, a), *y = x ? object_of(given_b, b) : nullptr;
    PyObject* r = y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return r;
}

// The interpreter's lock is given up from the first allocation, which may have to go to the driver, to the launch's end.
struct WithoutLock {
    PyThreadState* state = PyEval_SaveThread();
    WithoutLock() = default;
    WithoutLock(const WithoutLock&) = delete;
    ~WithoutLock() { PyEval_RestoreThread(state); }
};

// Errors come out as torch's own Python functions raise them: torch.OutOfMemoryError of an allocation, and what a dispatch mode
// raised inside one.
template <typename F>
PyObject* guarded(F f) {
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the five library functions)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) { PyErr_SetString(PyExc_TypeError, "bind takes 5 addresses"); return nullptr; }
    void* f[5];
    for (int i = 0; i < 5; ++i) {
        f[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    fwd_workspace_bytes = (decltype(fwd_workspace_bytes))f[0];
    bwd_workspace_bytes = (decltype(bwd_workspace_bytes))f[1];
    attn_fwd = (decltype(attn_fwd))f[2];
    attn_bwd = (decltype(attn_bwd))f[3];
    attn_merge = (decltype(attn_merge))f[4];
    Py_RETURN_NONE;
}

// fwd(q, k, v, cu_seqlens, causal, scale, out, lse, workspace, stream, kv_splits, max_seqlen) -> (out, lse), a status or
// NotImplemented
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 12 || !attn_fwd) { PyErr_SetString(PyExc_TypeError, "fwd takes 12 arguments, after bind"); return nullptr; }
    for (int i = 0; i < 4; ++i) if (!plain(a[i])) return not_implemented();
    for (int i = 6; i < 9; ++i) if (!plain_or_none(a[i])) return not_implemented();
    if (at::impl::torch_function_mode_enabled()) return not_implemented();
    return guarded([&]() -> PyObject* {
        const at::Tensor &q = THPVariable_Unpack(a[0]), &k = THPVariable_Unpack(a[1]), &v = THPVariable_Unpack(a[2]),
                         &cu = THPVariable_Unpack(a[3]);
        const double scale = PyFloat_AsDouble(a[5]);
        const long splits = PyLong_AsLong(a[10]), longest = PyLong_AsLong(a[11]);
        if (PyErr_Occurred()) { PyErr_Clear(); return not_implemented(); }
        varlen_attn_params p;
        if (!usable(q, at::kBFloat16) || !usable(k, at::kBFloat16) || !usable(v, at::kBFloat16) || !usable(cu, at::kInt) ||
            !fill(p, q, k, cu, a[4] == Py_True, scale, splits, longest) || k.sizes() != v.sizes() || k.size(0) != q.size(0) ||
            k.size(2) != q.size(2) || !none_or_room(a[6], at::kBFloat16, q.numel()) ||
            !none_or_room(a[7], at::kFloat, q.size(0) * q.size(1)) || !none_or_scratch(a[8]))
            return not_implemented();
        void* stream;
        if (!stream_of(a[9], stream)) return nullptr;
        if ((a[6] == Py_None || a[7] == Py_None || a[8] == Py_None) && elsewhere(a[9], stream, q)) return not_implemented();
        at::Tensor out, lse;
        int status;
        {
            WithoutLock free;
            out = given_or_like(a[6], q);
            lse = a[7] == Py_None ? at::empty({q.size(1), q.size(0)}, q.options().dtype(at::kFloat)) : THPVariable_Unpack(a[7]);
            const at::Tensor ws = workspace_of(a[8], a[8] == Py_None ? fwd_workspace_bytes(&p) : 0, q);
            status = attn_fwd(&p, q.data_ptr(), k.data_ptr(), v.data_ptr(), (const int32_t*)cu.data_ptr(), out.data_ptr(),
                              (float*)lse.data_ptr(), ws.data_ptr(), (size_t)ws.numel(), stream);
        }
        return status != VA_OK ? PyLong_FromLong(status) : pair(a[6], out, a[7], lse);
    });
}

// bwd(dout, q, k, v, out, lse, cu_seqlens, causal, scale, dq, dk, dv, workspace, stream, kv_splits, max_seqlen) ->
// (dq, dk, dv), a status or NotImplemented
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 16 || !attn_bwd) { PyErr_SetString(PyExc_TypeError, "bwd takes 16 arguments, after bind"); return nullptr; }
    for (int i = 0; i < 7; ++i) if (!plain(a[i])) return not_implemented();
    for (int i = 9; i < 13; ++i) if (!plain_or_none(a[i])) return not_implemented();
    if (at::impl::torch_function_mode_enabled()) return not_implemented();
    return guarded([&]() -> PyObject* {
        const at::Tensor &dout = THPVariable_Unpack(a[0]), &q = THPVariable_Unpack(a[1]), &k = THPVariable_Unpack(a[2]),
                         &v = THPVariable_Unpack(a[3]), &out = THPVariable_Unpack(a[4]), &lse = THPVariable_Unpack(a[5]),
                         &cu = THPVariable_Unpack(a[6]);
        const double scale = PyFloat_AsDouble(a[8]);
        const long splits = PyLong_AsLong(a[14]), longest = PyLong_AsLong(a[15]);
        if (PyErr_Occurred()) { PyErr_Clear(); return not_implemented(); }
        varlen_attn_params p;
        for (const at::Tensor* t : {&dout, &q, &k, &v, &out})
            if (!usable(*t, at::kBFloat16)) return not_implemented();
        if (!usable(cu, at::kInt) || !fill(p, q, k, cu, a[7] == Py_True, scale, splits, longest) || dout.sizes() != q.sizes() ||
            out.sizes() != q.sizes() || k.sizes() != v.sizes() || k.size(0) != q.size(0) || k.size(2) != q.size(2) ||
            !has_room(lse, at::kFloat, q.size(0) * q.size(1)) || !none_or_room(a[9], at::kBFloat16, q.numel()) ||
            !none_or_room(a[10], at::kBFloat16, k.numel()) || !none_or_room(a[11], at::kBFloat16, k.numel()) ||
            !none_or_scratch(a[12]))
            return not_implemented();
        void* stream;
        if (!stream_of(a[13], stream)) return nullptr;
        for (int i = 9; i < 13; ++i)
            if (a[i] == Py_None && elsewhere(a[13], stream, q)) return not_implemented();
        at::Tensor dq, dk, dv;
        int status;
        {
            WithoutLock free;
            dq = given_or_like(a[9], q);
            dk = given_or_like(a[10], k);
            dv = given_or_like(a[11], v);
            const at::Tensor ws = workspace_of(a[12], a[12] == Py_None ? bwd_workspace_bytes(&p) : 0, q);
            status = attn_bwd(&p, dout.data_ptr(), q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(),
                              (const float*)lse.data_ptr(), (const int32_t*)cu.data_ptr(), dq.data_ptr(), dk.data_ptr(),
                              dv.data_ptr(), ws.data_ptr(), (size_t)ws.numel(), stream);
        }
        if (status != VA_OK) return PyLong_FromLong(status);
        const at::Tensor* grads[3] = {&dq, &dk, &dv};
        PyObject* r = PyTuple_New(3);
        for (int i = 0; r && i < 3; ++i) {
            PyObject* g = object_of(a[9 + i], *grads[i]);
            if (!g) { Py_DECREF(r); return nullptr; }
            PyTuple_SET_ITEM(r, i, g);
        }
        return r;
    });
}

// merge(o_parts, lse_parts, out, lse, stream) -> (out, lse), a status or NotImplemented
PyObject* merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5 || !attn_merge) { PyErr_SetString(PyExc_TypeError, "merge takes 5 arguments, after bind"); return nullptr; }
    if (!plain(a[0]) || !plain(a[1]) || !plain_or_none(a[2]) || !plain_or_none(a[3]) || at::impl::torch_function_mode_enabled())
        return not_implemented();
    return guarded([&]() -> PyObject* {
        const at::Tensor &o = THPVariable_Unpack(a[0]), &l = THPVariable_Unpack(a[1]);
        if (!usable(o, at::kBFloat16) || !usable(l, at::kFloat) || o.dim() != 4 || l.dim() != 3 || l.size(0) != o.size(0) ||
            l.size(1) != o.size(2) || l.size(2) != o.size(1) ||
            !none_or_room(a[2], at::kBFloat16, o.size(1) * o.size(2) * o.size(3)) ||
            !none_or_room(a[3], at::kFloat, o.size(1) * o.size(2)))
            return not_implemented();
        for (int i = 0; i < 4; ++i) if (!fits(o.size(i))) return not_implemented();
        varlen_attn_params p{};
        p.total_tokens = (int32_t)o.size(1);
        p.num_seqs = 1;
        p.num_q_heads = p.num_kv_heads = (int32_t)o.size(2);
        p.head_dim = (int32_t)o.size(3);
        p.softmax_scale = 1.f;
        void* stream;
        if (!stream_of(a[4], stream)) return nullptr;
        if ((a[2] == Py_None || a[3] == Py_None) && elsewhere(a[4], stream, o)) return not_implemented();
        at::Tensor out, lse;
        int status;
        {
            WithoutLock free;
            out = a[2] == Py_None ? at::empty({o.size(1), o.size(2), o.size(3)}, o.options()) : THPVariable_Unpack(a[2]);
            lse = a[3] == Py_None ? at::empty({o.size(2), o.size(1)}, l.options()) : THPVariable_Unpack(a[3]);
            status = attn_merge(&p, (int32_t)o.size(0), o.data_ptr(), (const float*)l.data_ptr(), out.data_ptr(),
                                (float*)lse.data_ptr(), stream);
        }
        return status != VA_OK ? PyLong_FromLong(status) : pair(a[2], out, a[3], lse);
    });
}

PyMethodDef methods[] = {{"bind", (PyCFunction)(void (*)())bind, METH_FASTCALL, nullptr},
                         {"fwd", (PyCFunction)(void (*)())fwd, METH_FASTCALL, nullptr},
                         {"bwd", (PyCFunction)(void (*)())bwd, METH_FASTCALL, nullptr},
                         {"merge", (PyCFunction)(void (*)())merge, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_varlen_attn_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__varlen_attn_host() { return PyModule_Create(&module); }
