// The calls of binding.py that programs make over and over, without the interpreter between the checks (CPython extension).
//
// A call from Python costs a launch (3.45 us on this runtime, whatever the launch function) and what Python does around it: six
// tensor queries, a device query, the stream, a ctypes call, 1.9 us for a product, 11 us for a build with its three arrays.
// Here the same checks read the tensors directly (32 x 32, k 3, batch 1: conv_spmv 5.6 -> 3.3 us, on a slower host 5.8 -> 4.1;
// conv_update_kernel 5.1 -> 3.2, conv_csr_build 14.4 -> 7.5, ConvMulti.apply 3.8 -> 3.1).
//
// Each function does a call only where every check of binding.py holds as it is, on the current device and stream; for anything
// else it answers None and binding.py's own code, which knows every case and every error, does the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "../../../include/convspmv.h"

namespace {

// What a call needs of a ConvPlan.  `plan` is null once the plan is closed; `elsewhere` says that the plan was used on
// another stream than the one its arrays were allocated on (`home`).
struct PlanRef {
    PyObject_HEAD
    conv_plan *plan;
    long long x_size, y_size, kernel_size;      // floats per batch column, floats of a kernel
    void *home;
    char elsewhere;
};

int plan_ref_init(PyObject *self, PyObject *args, PyObject *) {
    PlanRef *const r = reinterpret_cast<PlanRef *>(self);
    unsigned long long handle, home;
    int elsewhere;
    if (!PyArg_ParseTuple(args, "KLLLKp", &handle, &r->x_size, &r->y_size, &r->kernel_size, &home, &elsewhere)) return -1;
    r->plan = reinterpret_cast<conv_plan *>(static_cast<uintptr_t>(handle));
    r->home = reinterpret_cast<void *>(static_cast<uintptr_t>(home));
    r->elsewhere = elsewhere != 0;
    return 0;
}

PyObject *plan_ref_close(PyObject *self, PyObject *) {
    reinterpret_cast<PlanRef *>(self)->plan = nullptr;
    Py_RETURN_NONE;
}

PyMemberDef plan_ref_members[] = {{"elsewhere", T_BOOL, offsetof(PlanRef, elsewhere), 0, nullptr}, {nullptr, 0, 0, 0, nullptr}};
PyMethodDef plan_ref_methods[] = {{"close", plan_ref_close, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyTypeObject plan_ref_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// A float tensor of torch's own type with `count` elements one after the other on device `device`.
const at::Tensor *operand(PyObject *o, long long count, int device) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.is_cuda() && t.scalar_type() == at::kFloat && t.is_contiguous() && t.numel() == count && t.get_device() == device ? &t : nullptr;
}

void *stream_of(int device) { return c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(device)).stream(); }

// One call of the library on the current stream: `call` gets the stream, the interpreter is free meanwhile.
template <typename F>
int on_stream(PlanRef *r, int device, F &&call) {
    void *const stream = stream_of(device);
    if (stream != r->home) r->elsewhere = 1;
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = call(stream);
    Py_END_ALLOW_THREADS;
    return status;
}

using Product = int (*)(const conv_plan *, const float *, float *, int, void *);

PyObject *product(PyObject *const *args, Py_ssize_t nargs, Product call, bool swapped) {
    if (nargs != 4 || Py_TYPE(args[0]) != &plan_ref_type || !PyLong_CheckExact(args[3])) Py_RETURN_NONE;
    PlanRef *const r = reinterpret_cast<PlanRef *>(args[0]);
    int overflow = 0;
    const long batch = PyLong_AsLongAndOverflow(args[3], &overflow);
    if (!r->plan || overflow || batch < 1 || batch > INT_MAX || (swapped && conv_plan_is_transposed(r->plan) != 1)) Py_RETURN_NONE;
    int status;
    try {
        const int device = c10::hip::current_device();
        const at::Tensor *const x = operand(args[1], (swapped ? r->y_size : r->x_size) * batch, device);
        const at::Tensor *const y = operand(args[2], (swapped ? r->x_size : r->y_size) * batch, device);
        if (!x || !y) Py_RETURN_NONE;
        const float *const xd = static_cast<const float *>(x->const_data_ptr());
        float *const yd = static_cast<float *>(y->data_ptr());
        conv_plan *const plan = r->plan;
        status = on_stream(r, device, [&](void *stream) { return call(plan, xd, yd, static_cast<int>(batch), stream); });
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

PyObject *spmv(PyObject *, PyObject *const *args, Py_ssize_t nargs) { return product(args, nargs, conv_spmv, false); }
PyObject *spmv_from_csc(PyObject *, PyObject *const *args, Py_ssize_t nargs) { return product(args, nargs, conv_spmv_from_csc, true); }

PyObject *update_kernel(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 2 || Py_TYPE(args[0]) != &plan_ref_type) Py_RETURN_NONE;
    PlanRef *const r = reinterpret_cast<PlanRef *>(args[0]);
    if (!r->plan) Py_RETURN_NONE;
    int status;
    try {
        const int device = c10::hip::current_device();
        const at::Tensor *const kernel = operand(args[1], r->kernel_size, device);
        if (!kernel) Py_RETURN_NONE;
        const float *const kd = static_cast<const float *>(kernel->const_data_ptr());
        conv_plan *const plan = r->plan;
        status = on_stream(r, device, [&](void *stream) { return conv_update_kernel(plan, kd, stream); });
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

PyObject *multi_apply(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 1 || !PyLong_CheckExact(args[0])) Py_RETURN_NONE;
    const conv_multi *const multi = static_cast<const conv_multi *>(PyLong_AsVoidPtr(args[0]));
    if (!multi) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    int status;
    try {
        void *const stream = stream_of(c10::hip::current_device());
        Py_BEGIN_ALLOW_THREADS;
        status = conv_multi_apply(multi, stream);
        Py_END_ALLOW_THREADS;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

// (m, n, k, s, p, kernel, transposed): the arrays of conv_csr_build or conv_csc_build and their plan,
// (handle, m_out, n_out, nnz, pointers, indices, values, stream), or the status of a build that failed.
PyObject *build(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 7) Py_RETURN_NONE;
    int shape[5];
    for (int i = 0; i < 5; ++i) {
        if (!PyLong_CheckExact(args[i])) Py_RETURN_NONE;
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(args[i], &overflow);
        if (overflow || v < 0 || v > 1 << 20) Py_RETURN_NONE;      // (their products in 64 bits)
        shape[i] = static_cast<int>(v);
    }
    const int m = shape[0], n = shape[1], k = shape[2], s = shape[3], p = shape[4];
    const int transposed = PyObject_IsTrue(args[6]);
    if (transposed < 0) return nullptr;
    int m_out = 0, n_out = 0;
    if (conv_out_shape(m, n, k, s, p, &m_out, &n_out) != CONV_OK) Py_RETURN_NONE;
    const int64_t nnz = conv_nnz(m, n, k, s, p), in = static_cast<int64_t>(m) * n, out = static_cast<int64_t>(m_out) * n_out;
    if (nnz < 1 || nnz > INT_MAX || in >= INT_MAX || out >= INT_MAX) Py_RETURN_NONE;
    at::Tensor ptr, idx, vals;
    conv_plan *plan = nullptr;
    void *stream = nullptr;
    int status;
    try {
        const int device = c10::hip::current_device();
        const at::Tensor *const kernel = operand(args[5], static_cast<long long>(k) * k, device);
        if (!kernel) Py_RETURN_NONE;
        const at::TensorOptions ints = at::TensorOptions().dtype(at::kInt).device(kernel->device());
        ptr = at::empty({(transposed ? in : out) + 1}, ints);
        idx = at::empty({nnz}, ints);
        vals = at::empty({nnz}, ints.dtype(at::kFloat));
        stream = stream_of(device);
        const float *const kd = static_cast<const float *>(kernel->const_data_ptr());
        int32_t *const pd = static_cast<int32_t *>(ptr.data_ptr()), *const id = static_cast<int32_t *>(idx.data_ptr());
        float *const vd = static_cast<float *>(vals.data_ptr());
        Py_BEGIN_ALLOW_THREADS;
        status = (transposed ? conv_csc_build : conv_csr_build)(m, n, k, s, p, kd, pd, id, vd, stream, &plan);
        Py_END_ALLOW_THREADS;
    } catch (...) {
        Py_RETURN_NONE;
    }
    if (status != CONV_OK) return PyLong_FromLong(status);
    return Py_BuildValue("(KiiLNNNK)", static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(plan)), m_out, n_out,
                         static_cast<long long>(nnz), THPVariable_Wrap(ptr), THPVariable_Wrap(idx), THPVariable_Wrap(vals),
                         static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(stream)));
}

// A plan that only the default stream has seen is destroyed; its kernel tensor is recorded on that stream (ConvPlan.close).
PyObject *drop(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 2 || !PyLong_CheckExact(args[0]) || !THPVariable_CheckExact(args[1])) Py_RETURN_FALSE;
    conv_plan *const plan = static_cast<conv_plan *>(PyLong_AsVoidPtr(args[0]));
    if (!plan) {
        PyErr_Clear();
        Py_RETURN_FALSE;
    }
    try {
        const at::Tensor &kernel = THPVariable_Unpack(args[1]);
        if (!kernel.is_cuda()) Py_RETURN_FALSE;
        kernel.record_stream(c10::Stream(c10::Stream::DEFAULT, kernel.device()));
    } catch (...) {
        Py_RETURN_FALSE;
    }
    conv_plan_destroy(plan);
    Py_RETURN_TRUE;
}

template <typename F>
PyCFunction fast(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"spmv", fast(spmv), METH_FASTCALL, nullptr}, {"spmv_from_csc", fast(spmv_from_csc), METH_FASTCALL, nullptr},
    {"update_kernel", fast(update_kernel), METH_FASTCALL, nullptr}, {"multi_apply", fast(multi_apply), METH_FASTCALL, nullptr},
    {"build", fast(build), METH_FASTCALL, nullptr}, {"drop", fast(drop), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    plan_ref_type.tp_name = "_native.PlanRef";
    plan_ref_type.tp_basicsize = sizeof(PlanRef);
    plan_ref_type.tp_flags = Py_TPFLAGS_DEFAULT;
    plan_ref_type.tp_new = PyType_GenericNew;
    plan_ref_type.tp_init = plan_ref_init;
    plan_ref_type.tp_members = plan_ref_members;
    plan_ref_type.tp_methods = plan_ref_methods;
    if (PyType_Ready(&plan_ref_type) < 0) return nullptr;
    PyObject *const m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&plan_ref_type);
    if (PyModule_AddObject(m, "PlanRef", reinterpret_cast<PyObject *>(&plan_ref_type)) < 0) {
        Py_DECREF(&plan_ref_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
