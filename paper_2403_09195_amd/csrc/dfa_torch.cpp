// The host side of one dfa_forward or dfa_backward call on torch tensors, in native code: checks, allocation of the results and the workspace, the
// current stream.  Small launches wait for their host side: one 256^2 image took 10.9 us a call in Python and ctypes (two
// torch.empty 3.5 us, marshalling 2.3, the ctypes call's own conversions 1) around 2.4 us of launch and 6.6 us on the GPU; its backward
// 16.0 (four torch.empty, six checked tensors), 9.1 this way, which is the GPU's time (forward and backward 21.0 / 15.8).
//
// Only the ordinary call goes this way: 4-d GPU tensors of one dtype with contiguous last dimension, lists of Python integers.  Anything else
// is handed back (None) to binding.forward or binding.backward, which converts it or names what is wrong with it.
#include <Python.h>
#include <pybind11/pybind11.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include "../../include/dfa.h"

namespace {

using ForwardAlloc = decltype(&dfa_forward_alloc);
using Backward = decltype(&dfa_backward);
ForwardAlloc g_forward = nullptr;
Backward g_backward = nullptr;

constexpr int kMaxOffsets = 1024;

// A Python list or tuple; the items are borrowed.
struct Sequence {
    PyObject** items = nullptr;
    Py_ssize_t n = -1;
    explicit Sequence(PyObject* o) {
        if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) {
            items = PySequence_Fast_ITEMS(o);
            n = PySequence_Fast_GET_SIZE(o);
        }
    }
};

bool as_int32(PyObject* o, int32_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || x != (int32_t)x) return false;
    *out = (int32_t)x;
    return true;
}

// What the workspace callback needs, and what it leaves: the tensor lives until the call has enqueued its launches.
// (Allocated on the current stream: the allocator gives its memory to later work of this stream only.)
struct Workspace {
    const at::TensorOptions options;
    at::Tensor tensor;
    std::exception_ptr error;
};
void* allocate(void* context, size_t bytes) {
    Workspace* w = static_cast<Workspace*>(context);
    try {
        w->tensor = at::empty({(int64_t)bytes}, w->options);
        return w->tensor.data_ptr();
    } catch (...) {
        w->error = std::current_exception();
        return nullptr;
    }
}

// What both calls take, as the library reads it.
struct Call {
    const at::Tensor* t[3];                    // q, k, v
    dfa_strides_t s[3];
    dfa_dtype_t dtype;
    int64_t B, N, H, D;
    dfa_branch_t branches[DFA_MAX_BRANCHES];
    int32_t nb;
    float scale;
    int32_t table[kMaxOffsets];
    const int32_t* offsets;                    // table or NULL
};

// Reads q, k, v and branches, scale, head_offsets; false: not the ordinary call.
bool read_call(PyObject* const* qkv, PyObject* const* rest, Call* c) {
    for (int i = 0; i < 3; ++i) {
        if (!THPVariable_CheckExact(qkv[i])) return false;
        c->t[i] = &THPVariable_Unpack(qkv[i]);
        if (!c->t[i]->is_cuda() || c->t[i]->dim() != 4 || c->t[i]->stride(3) != 1) return false;
        c->s[i] = dfa_strides_t{c->t[i]->stride(0), c->t[i]->stride(1), c->t[i]->stride(2)};
    }
    const at::Tensor& q = *c->t[0];
    const at::ScalarType type = q.scalar_type();
    if (type != at::kBFloat16 && type != at::kFloat) return false;
    c->dtype = type == at::kFloat ? DFA_F32 : DFA_BF16;
    for (int i = 1; i < 3; ++i) {              // nor less than q, which the kernels would read past (the binding refuses it)
        if (c->t[i]->scalar_type() != type) return false;
        for (int d = 0; d < 4; ++d)
            if (c->t[i]->size(d) < q.size(d)) return false;
    }
    c->B = q.size(0), c->N = q.size(1), c->H = q.size(2), c->D = q.size(3);
    if (c->B > INT32_MAX || c->N > INT32_MAX || c->H > INT32_MAX || c->D > INT32_MAX) return false;

    const Sequence list(rest[0]);
    if (list.n < 1 || list.n > DFA_MAX_BRANCHES) return false;
    c->nb = (int32_t)list.n;
    for (Py_ssize_t i = 0; i < list.n; ++i) {
        const Sequence pair(list.items[i]);
        if (pair.n != 2 || !as_int32(pair.items[0], &c->branches[i].w) || !as_int32(pair.items[1], &c->branches[i].r)) return false;
    }
    if (!PyFloat_CheckExact(rest[1])) return false;
    c->scale = (float)PyFloat_AS_DOUBLE(rest[1]);

    c->offsets = nullptr;
    if (rest[2] != Py_None) {
        const Sequence rows(rest[2]);
        if (rows.n != list.n || list.n * c->H > kMaxOffsets) return false;
        for (Py_ssize_t i = 0; i < rows.n; ++i) {
            const Sequence row(rows.items[i]);
            if (row.n != c->H) return false;
            for (Py_ssize_t h = 0; h < row.n; ++h)
                if (!as_int32(row.items[h], &c->table[i * c->H + h])) return false;
        }
        c->offsets = c->table;
    }
    return true;
}

// Whether contiguous t, read as a contiguous array of the n sizes `want`, has the elements of t[:want[0], :want[1], ...]; with another number of
// dimensions, as many elements in this order.  (The kernels would read past the end of less.)
bool holds(const at::Tensor& t, const int64_t* want, int64_t n) {
    int64_t stride = 1;
    bool same = t.dim() == n;
    for (int64_t d = n - 1; d >= 0; --d) {
        same = same && t.size(d) >= want[d] && (want[d] == 1 || t.stride(d) == stride);
        stride *= want[d];
    }
    return t.dim() == n ? same : t.numel() >= stride;
}

// A tuple of tensors, which are given up.
template <size_t n>
PyObject* as_tuple(at::Tensor (&t)[n]) {
    PyObject* const tuple = PyTuple_New((Py_ssize_t)n);
    if (!tuple) return nullptr;
    for (size_t i = 0; i < n; ++i) {
        PyObject* const o = THPVariable_Wrap(std::move(t[i]));
        if (!o) {
            Py_DECREF(tuple);
            return nullptr;
        }
        PyTuple_SET_ITEM(tuple, (Py_ssize_t)i, o);
    }
    return tuple;
}

// forward(q, k, v, branches, scale, head_offsets) -> (out, lse), a negative status, or None
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    Call c;
    if (nargs != 6 || !g_forward || !read_call(args, args + 3, &c)) Py_RETURN_NONE;
    const at::Tensor& q = *c.t[0];
    at::Tensor res[2] = {at::empty({c.B, c.N, c.H, c.D}, q.options()), at::empty({c.B, c.H, c.N}, q.options().dtype(at::kFloat))};
    Workspace ws{q.options().dtype(at::kByte), at::Tensor(), nullptr};
    const void *const qp = q.data_ptr(), *const kp = c.t[1]->data_ptr(), *const vp = c.t[2]->data_ptr();
    int rc;
    {
        // Other threads run meanwhile: a shape's first call builds and uploads its plan, a dropped plan waits for the device, a
        // launch may wait for the queue.  (No Python object is touched; the workspace callback needs none either.)
        pybind11::gil_scoped_release release;
        rc = g_forward(qp, kp, vp, c.s[0], c.s[1], c.s[2], (int32_t)c.B, (int32_t)c.H, (int32_t)c.N, (int32_t)c.D, c.dtype, c.scale, c.branches, c.nb,
                       c.offsets, res[0].data_ptr(), res[1].data_ptr<float>(), allocate, &ws, c10::hip::getCurrentHIPStream().stream());
    }
    if (ws.error) std::rethrow_exception(ws.error);
    if (rc != DFA_OK) return PyLong_FromLong(rc);
    return as_tuple(res);
    END_HANDLE_TH_ERRORS
}

// backward(q, k, v, out, lse, dout, branches, scale, head_offsets) -> (dq, dk, dv), a negative status, or None
PyObject* backward(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    Call c;
    if (nargs != 9 || !g_backward || !read_call(args, args + 6, &c)) Py_RETURN_NONE;
    const at::Tensor& q = *c.t[0];
    const at::Tensor* x[3];                    // out, lse, dout
    const int64_t rows[4] = {c.B, c.N, c.H, c.D}, stats[3] = {c.B, c.H, c.N};
    for (int i = 0; i < 3; ++i) {
        if (!THPVariable_CheckExact(args[3 + i])) Py_RETURN_NONE;
        x[i] = &THPVariable_Unpack(args[3 + i]);
        if (!x[i]->is_cuda() || !x[i]->is_contiguous() || x[i]->scalar_type() != (i == 1 ? at::kFloat : q.scalar_type())) Py_RETURN_NONE;
        if (!(i == 1 ? holds(*x[i], stats, 3) : holds(*x[i], rows, 4))) Py_RETURN_NONE;
    }
    at::Tensor res[3];
    for (at::Tensor& r : res) r = at::empty({c.B, c.N, c.H, c.D}, q.options());
    // (allocated on the current stream: the allocator gives its memory to later work of this stream only)
    at::Tensor delta = at::empty({2, c.B, c.H, c.N}, q.options().dtype(at::kFloat));
    const void *const qp = q.data_ptr(), *const kp = c.t[1]->data_ptr(), *const vp = c.t[2]->data_ptr();
    int rc;
    {
        pybind11::gil_scoped_release release;  // as in forward
        rc = g_backward(qp, kp, vp, x[0]->data_ptr(), x[1]->data_ptr<float>(), x[2]->data_ptr(), c.s[0], c.s[1], c.s[2], (int32_t)c.B, (int32_t)c.H,
                        (int32_t)c.N, (int32_t)c.D, c.dtype, c.scale, c.branches, c.nb, c.offsets, delta.data_ptr<float>(), res[0].data_ptr(),
                        res[1].data_ptr(), res[2].data_ptr(), c10::hip::getCurrentHIPStream().stream());
    }
    if (rc != DFA_OK) return PyLong_FromLong(rc);
    return as_tuple(res);
    END_HANDLE_TH_ERRORS
}

// bind(addresses of dfa_forward_alloc and dfa_backward in the loaded libdfa.so)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 2) {
        PyErr_SetString(PyExc_TypeError, "bind takes two addresses");
        return nullptr;
    }
    g_forward = reinterpret_cast<ForwardAlloc>(PyLong_AsVoidPtr(args[0]));
    g_backward = reinterpret_cast<Backward>(PyLong_AsVoidPtr(args[1]));
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(backward)), METH_FASTCALL, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_dfa_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dfa_torch() { return PyModule_Create(&g_module); }
