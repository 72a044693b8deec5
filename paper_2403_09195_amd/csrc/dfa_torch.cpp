// The host side of one dfa_forward call on torch tensors, in native code: checks, allocation of out, lse and workspace, the
// current stream.  Small launches wait for their host side: one 256^2 image took 10.9 us a call in Python and ctypes (two
// torch.empty 3.5 us, marshalling 2.3, the ctypes call's own conversions 1) around 2.4 us of launch and 6.6 us on the GPU.
//
// Only the ordinary call goes this way: 4-d GPU tensors of one dtype with contiguous last dimension, lists of Python integers.  Anything else
// is handed back (None) to binding.forward, which converts it or names what is wrong with it.
#include <Python.h>
#include <pybind11/pybind11.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include "../../include/dfa.h"

namespace {

using ForwardAlloc = decltype(&dfa_forward_alloc);
ForwardAlloc g_forward = nullptr;

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

// forward(q, k, v, branches, scale, head_offsets) -> (out, lse), a negative status, or None
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 6 || !g_forward) Py_RETURN_NONE;
    const at::Tensor* t[3];
    dfa_strides_t s[3];
    for (int i = 0; i < 3; ++i) {
        if (!THPVariable_CheckExact(args[i])) Py_RETURN_NONE;
        t[i] = &THPVariable_Unpack(args[i]);
        if (!t[i]->is_cuda() || t[i]->dim() != 4 || t[i]->stride(3) != 1) Py_RETURN_NONE;
        s[i] = dfa_strides_t{t[i]->stride(0), t[i]->stride(1), t[i]->stride(2)};
    }
    const at::Tensor& q = *t[0];
    const at::ScalarType type = q.scalar_type();
    if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NONE;
    for (int i = 1; i < 3; ++i) {              // nor less than q, which the kernels would read past (binding.forward refuses it)
        if (t[i]->scalar_type() != type) Py_RETURN_NONE;
        for (int d = 0; d < 4; ++d)
            if (t[i]->size(d) < q.size(d)) Py_RETURN_NONE;
    }
    const int64_t B = q.size(0), N = q.size(1), H = q.size(2), D = q.size(3);
    if (B > INT32_MAX || N > INT32_MAX || H > INT32_MAX || D > INT32_MAX) Py_RETURN_NONE;

    const Sequence list(args[3]);
    if (list.n < 1 || list.n > DFA_MAX_BRANCHES) Py_RETURN_NONE;
    dfa_branch_t branches[DFA_MAX_BRANCHES];
    for (Py_ssize_t i = 0; i < list.n; ++i) {
        const Sequence pair(list.items[i]);
        if (pair.n != 2 || !as_int32(pair.items[0], &branches[i].w) || !as_int32(pair.items[1], &branches[i].r)) Py_RETURN_NONE;
    }
    if (!PyFloat_CheckExact(args[4])) Py_RETURN_NONE;
    const float scale = (float)PyFloat_AS_DOUBLE(args[4]);

    int32_t table[kMaxOffsets];
    if (args[5] != Py_None) {
        const Sequence rows(args[5]);
        if (rows.n != list.n || list.n * H > kMaxOffsets) Py_RETURN_NONE;
        for (Py_ssize_t i = 0; i < rows.n; ++i) {
            const Sequence row(rows.items[i]);
            if (row.n != H) Py_RETURN_NONE;
            for (Py_ssize_t h = 0; h < row.n; ++h)
                if (!as_int32(row.items[h], &table[i * H + h])) Py_RETURN_NONE;
        }
    }

    at::Tensor out = at::empty({B, N, H, D}, q.options());
    at::Tensor lse = at::empty({B, H, N}, q.options().dtype(at::kFloat));
    Workspace ws{q.options().dtype(at::kByte), at::Tensor(), nullptr};
    const void *const qp = q.data_ptr(), *const kp = t[1]->data_ptr(), *const vp = t[2]->data_ptr();
    int rc;
    {
        // Other threads run meanwhile: a shape's first call builds and uploads its plan, a dropped plan waits for the device, a
        // launch may wait for the queue.  (No Python object is touched; the workspace callback needs none either.)
        pybind11::gil_scoped_release release;
        rc = g_forward(qp, kp, vp, s[0], s[1], s[2], (int32_t)B, (int32_t)H, (int32_t)N, (int32_t)D, type == at::kFloat ? DFA_F32 : DFA_BF16,
                       scale, branches, (int32_t)list.n, args[5] != Py_None ? table : nullptr, out.data_ptr(), lse.data_ptr<float>(), allocate,
                       &ws, c10::hip::getCurrentHIPStream().stream());
    }
    if (ws.error) std::rethrow_exception(ws.error);
    if (rc != DFA_OK) return PyLong_FromLong(rc);
    PyObject* const po = THPVariable_Wrap(std::move(out));
    if (!po) return nullptr;
    PyObject* const pl = THPVariable_Wrap(std::move(lse));
    if (!pl) {
        Py_DECREF(po);
        return nullptr;
    }
    PyObject* const pair = PyTuple_New(2);
    if (!pair) {
        Py_DECREF(po);
        Py_DECREF(pl);
        return nullptr;
    }
    PyTuple_SET_ITEM(pair, 0, po);
    PyTuple_SET_ITEM(pair, 1, pl);
    return pair;
    END_HANDLE_TH_ERRORS
}

// bind(address of dfa_forward_alloc in the loaded libdfa.so)
PyObject* bind(PyObject*, PyObject* address) {
    g_forward = reinterpret_cast<ForwardAlloc>(PyLong_AsVoidPtr(address));
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr},
    {"bind", bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_dfa_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dfa_torch() { return PyModule_Create(&g_module); }
