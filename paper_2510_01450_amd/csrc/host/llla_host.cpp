// The host side of a forward or decode call from Python, natively: reads the tensors, allocates result and scratch with torch's allocator and
// calls the C ABI.  A call of one head x 128 rows is 8 us on the GPU and took the host 11.5 in Python (ctypes alone 2.3, strides, sizes and
// two allocations the rest); from here such calls follow each other at the GPU's pace, 8.1 us, and a single call ends 5 to 7 us earlier.
//
// It serves the ordinary forms only: plain torch tensors of the right types and shapes on the GPU.  For everything else -- and for every mistake --
// it returns NotImplemented without having done anything, and binding.py's own code takes the call, which words the errors.  A status of the C ABI
// other than 0 comes back as an integer.
#include <Python.h>

#include <ATen/Functions.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "llla.h"

namespace {

using ForwardFn = decltype(&llla_forward_ex);
using DecodeFn = decltype(&llla_decode_path);
using SizeFn = size_t (*)(int, int, int, int, llla_dtype);

constexpr int64_t MAX_DIM = 2147483647;

bool is_tensor(PyObject *o) { return THPVariable_CheckExact(o); }

bool dtype_of(at::ScalarType s, llla_dtype &t)
{
    if (s == at::kFloat) t = LLLA_F32;
    else if (s == at::kBFloat16) t = LLLA_BF16;
    else return false;
    return true;
}

// a [B, H, n, d] tensor on the GPU with unit stride along d
bool rows4(const at::Tensor &t, llla_strides &s)
{
    if (t.dim() != 4 || t.stride(3) != 1) return false;
    s = llla_strides{t.stride(0), t.stride(1), t.stride(2)};
    return true;
}

bool number(PyObject *o, double &v)
{
    if (!PyFloat_CheckExact(o)) return false;
    v = PyFloat_AS_DOUBLE(o);
    return true;
}

bool flag(PyObject *o, int &v)
{
    if (!PyBool_Check(o)) return false;
    v = o == Py_True;
    return true;
}

// dtype of a new result: None is float32
bool result_type(PyObject *o, at::ScalarType &t)
{
    llla_dtype unused;
    if (o == Py_None) t = at::kFloat;
    else if (THPDtype_Check(o)) t = reinterpret_cast<THPDtype *>(o)->scalar_type;
    else return false;
    return dtype_of(t, unused);
}

struct Scratch {
    at::Tensor own;
    void *ptr;
    size_t bytes;
};

// the caller's scratch, or without any `need` bytes from torch's allocator
Scratch scratch(const at::Tensor *given, size_t need, const at::Device &device)
{
    Scratch s;
    if (given == nullptr) {
        s.own = at::empty({(int64_t)(need < 256 ? 256 : need)}, at::TensorOptions().dtype(at::kByte).device(device));
        given = &s.own;
    }
    s.ptr = given->data_ptr();
    s.bytes = (size_t)given->numel() * given->element_size();
    return s;
}

PyObject *not_implemented() { Py_RETURN_NOTIMPLEMENTED; }

// The stream of a call: a handle, or what to call for the current stream's (asked only now that the tensors are known to be on the GPU)
void *stream_of(PyObject *o)
{
    if (PyLong_Check(o)) return PyLong_AsVoidPtr(o);
    PyObject *r = PyObject_CallNoArgs(o);
    if (r == nullptr) return nullptr;
    void *s = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return s;
}

// Other threads go on while torch allocates (which can wait for the GPU, or free what it holds and try again) and while the C ABI is called (a launch
// can wait for room in the queue), as they do where Python makes these calls.  Taken back on the way out, exceptions included.
struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// forward(llla_forward_ex, llla_forward_workspace_bytes, Q, K, V, lam, scale, causal, out_dtype, path, workspace, out, return_stats, stream)
PyObject *forward(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    if (n_args != 14) return not_implemented();
    for (int i = 2; i < 5; ++i)
        if (!is_tensor(a[i])) return not_implemented();
    const at::Tensor &Q = THPVariable_Unpack(a[2]), &K = THPVariable_Unpack(a[3]), &V = THPVariable_Unpack(a[4]);
    llla_dtype in, out = LLLA_F32;
    llla_strides sq, sk, sv, so;
    at::ScalarType out_type;
    double lambda = 0., scale;
    int causal, stats;
    if (!Q.is_cuda() || !K.is_cuda() || !V.is_cuda() || K.scalar_type() != Q.scalar_type() || V.scalar_type() != Q.scalar_type() ||
        !dtype_of(Q.scalar_type(), in) || !rows4(Q, sq) || !rows4(K, sk) || !rows4(V, sv) || K.sizes() != Q.sizes() || V.sizes() != Q.sizes() ||
        !number(a[6], scale) || !flag(a[7], causal) || !result_type(a[8], out_type) || !flag(a[12], stats))
        return not_implemented();
    const int64_t B = Q.size(0), H = Q.size(1), n = Q.size(2), d = Q.size(3);
    if (B > MAX_DIM || H > MAX_DIM || n > MAX_DIM || d > MAX_DIM) return not_implemented();
    const float *lam_rows = nullptr;
    if (is_tensor(a[5])) {
        const at::Tensor &l = THPVariable_Unpack(a[5]);
        if (!l.is_cuda() || l.scalar_type() != at::kFloat || l.dim() != 3 || l.size(0) != B || l.size(1) != H || l.size(2) != n || !l.is_contiguous())
            return not_implemented();
        lam_rows = static_cast<const float *>(l.data_ptr());
    } else if (!number(a[5], lambda)) {
        return not_implemented();
    }
    if (a[11] != Py_None && (!is_tensor(a[11]) || !dtype_of(THPVariable_Unpack(a[11]).scalar_type(), out) || !rows4(THPVariable_Unpack(a[11]), so)))
        return not_implemented();
    const long path = PyLong_AsLong(a[9]);
    if (path < 0) return not_implemented();
    if (a[10] != Py_None && !is_tensor(a[10])) return not_implemented();

    void *stream = stream_of(a[13]);
    if (PyErr_Occurred()) return nullptr;
    const ForwardFn call = reinterpret_cast<ForwardFn>(PyLong_AsVoidPtr(a[0]));
    const SizeFn size = reinterpret_cast<SizeFn>(PyLong_AsVoidPtr(a[1]));
    const at::Tensor *given = a[10] == Py_None ? nullptr : &THPVariable_Unpack(a[10]);
    at::Tensor O, rho, delta;
    if (a[11] != Py_None) O = THPVariable_Unpack(a[11]);
    llla_status st;
    {
        WithoutGil released;
        const at::TensorOptions options = at::TensorOptions().device(Q.device()).dtype(at::kFloat);
        if (!O.defined()) {
            O = at::empty({B, H, n, d}, options.dtype(out_type));
            dtype_of(out_type, out);
            so = llla_strides{O.stride(0), O.stride(1), O.stride(2)};
        }
        if (stats) {
            rho = at::empty({B, H, n, d}, options);
            delta = at::empty({B, H, n}, options);
        }
        const Scratch ws = scratch(given, given ? 0 : size((int)B, (int)H, (int)n, (int)d, in), Q.device());
        st = call(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), sq, sk, sv, so, (int)B, (int)H, (int)n, (int)d, in, out, causal, (float)lambda,
                  lam_rows, (float)scale, stats ? static_cast<float *>(rho.data_ptr()) : nullptr,
                  stats ? static_cast<float *>(delta.data_ptr()) : nullptr, (llla_path)path, ws.ptr, ws.bytes, stream);
    }
    if (st != LLLA_OK) return PyLong_FromLong(st);
    PyObject *result;
    if (a[11] != Py_None) {
        Py_INCREF(a[11]);
        result = a[11];
    } else {
        result = THPVariable_Wrap(O);
    }
    if (!stats || result == nullptr) return result;
    PyObject *t = PyTuple_New(3);
    PyTuple_SET_ITEM(t, 0, result);
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(rho));
    PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(delta));
    return t;
    END_HANDLE_TH_ERRORS
}

// decode(llla_decode_path, llla_decode_workspace_bytes, q, Kc, Vc, lam, scale, seqlens, out_dtype, path, workspace, out, stream)
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    if (n_args != 13) return not_implemented();
    for (int i = 2; i < 5; ++i)
        if (!is_tensor(a[i])) return not_implemented();
    const at::Tensor &q = THPVariable_Unpack(a[2]), &K = THPVariable_Unpack(a[3]), &V = THPVariable_Unpack(a[4]);
    llla_dtype in, out = LLLA_F32;
    llla_strides sk, sv;
    at::ScalarType out_type;
    double lambda, scale;
    if (!q.is_cuda() || !K.is_cuda() || !V.is_cuda() || K.scalar_type() != q.scalar_type() || V.scalar_type() != q.scalar_type() ||
        !dtype_of(q.scalar_type(), in) || !rows4(K, sk) || !rows4(V, sv) || V.sizes() != K.sizes() || !number(a[5], lambda) || !number(a[6], scale) ||
        !result_type(a[8], out_type))
        return not_implemented();
    const int64_t B = K.size(0), H = K.size(1), n = K.size(2), d = K.size(3);
    if (B > MAX_DIM || H > MAX_DIM || n > MAX_DIM || d > MAX_DIM) return not_implemented();
    if (q.dim() != 3 || q.size(0) != B || q.size(1) != H || q.size(2) != d || !q.is_contiguous()) return not_implemented();
    const int32_t *lens = nullptr;
    if (a[7] != Py_None) {
        if (!is_tensor(a[7])) return not_implemented();
        const at::Tensor &l = THPVariable_Unpack(a[7]);
        if (l.scalar_type() != at::kInt || !l.is_cuda() || l.numel() != B) return not_implemented();
        lens = static_cast<const int32_t *>(l.data_ptr());
    }
    if (a[11] != Py_None && (!is_tensor(a[11]) || !dtype_of(THPVariable_Unpack(a[11]).scalar_type(), out))) return not_implemented();
    const long path = PyLong_AsLong(a[9]);
    if (path < 0) return not_implemented();
    if (a[10] != Py_None && !is_tensor(a[10])) return not_implemented();

    void *stream = stream_of(a[12]);
    if (PyErr_Occurred()) return nullptr;
    const DecodeFn call = reinterpret_cast<DecodeFn>(PyLong_AsVoidPtr(a[0]));
    const SizeFn size = reinterpret_cast<SizeFn>(PyLong_AsVoidPtr(a[1]));
    const at::Tensor *given = a[10] == Py_None ? nullptr : &THPVariable_Unpack(a[10]);
    at::Tensor o;
    if (a[11] != Py_None) o = THPVariable_Unpack(a[11]);
    llla_status st;
    {
        WithoutGil released;
        if (!o.defined()) {
            o = at::empty({B, H, d}, at::TensorOptions().device(q.device()).dtype(out_type));
            dtype_of(out_type, out);
        }
        const Scratch ws = scratch(given, given ? 0 : size((int)B, (int)H, (int)n, (int)d, in), q.device());
        st = call(q.data_ptr(), K.data_ptr(), V.data_ptr(), o.data_ptr(), sk, sv, lens, (int)B, (int)H, (int)n, (int)d, in, out, (float)lambda, (float)scale,
                  (llla_path)path, ws.ptr, ws.bytes, stream);
    }
    if (st != LLLA_OK) return PyLong_FromLong(st);
    if (a[11] != Py_None) {
        Py_INCREF(a[11]);
        return a[11];
    }
    return THPVariable_Wrap(o);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(forward)), METH_FASTCALL, nullptr},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(decode)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "llla_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_llla_host() { return PyModule_Create(&module); }
