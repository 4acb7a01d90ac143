// CPython extension of the binding: reads the tensors of a call and calls the C
// ABI of liblsgd.so. Every function returns the call's lsgd_status, or None
// where an argument is anything but what the call plainly takes (another type
// or dtype, another device, not contiguous, another size, a tensor subclass
// with its own dispatch, ...): the caller then takes the general Python path,
// which checks each argument and raises its error. Reading 130 tensors' dtype,
// device, size, layout and address from Python cost 80 to 90 us of a 95 us
// call; here it is 3 to 4.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "lsgd.h"
#include "marshal_call.h"

namespace {

// A plain dense GPU tensor, or null: a torch.Tensor or Parameter itself, as a
// subclass may answer for its address, size or dtype with __torch_function__.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.unsafeGetTensorImpl()->is_python_dispatch() ||
        t.is_conj() || t.is_neg() || !t.is_contiguous())
        return nullptr;
    return &t;
}

// A plain tensor of `dtype` with n elements (n < 0: any) on device `dev`.
const at::Tensor* plain(PyObject* o, at::ScalarType dtype, int64_t n, int dev) {
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == dtype && (n < 0 || t->numel() == n) && t->get_device() == dev ? t : nullptr;
}

// Addresses of a list or tuple of n-element tensors of one dtype (float32 or
// bfloat16; 0 entries: float32). False where it is anything else.
bool addresses(PyObject* seq, int64_t n, int dev, void** out, int most, int* count, lsgd_dtype* dt) {
    if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return false;
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(seq);
    if (k > most) return false;
    at::ScalarType type = at::kFloat;
    for (Py_ssize_t i = 0; i < k; ++i) {
        PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
        if (i == 0) {
            const at::Tensor* t = plain(o);
            if (!t) return false;
            type = t->scalar_type();
            if (type != at::kFloat && type != at::kBFloat16) return false;
        }
        const at::Tensor* t = plain(o, type, n, dev);
        if (!t) return false;
        out[i] = t->data_ptr();
    }
    *count = static_cast<int>(k);
    *dt = type == at::kBFloat16 ? LSGD_BF16 : LSGD_F32;
    return true;
}

bool small_int(PyObject* o, int32_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) return false;
    *out = static_cast<int32_t>(v);
    return true;
}

// group_of_worker of exactly `count` entries.
bool membership(PyObject* seq, int count, int32_t* out) {
    if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return false;
    if (PySequence_Fast_GET_SIZE(seq) != count) return false;
    for (int i = 0; i < count; ++i)
        if (!small_int(PySequence_Fast_GET_ITEM(seq, i), &out[i])) return false;
    return true;
}

bool number(PyObject* o, float* out) {
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
    const double v = PyFloat_AsDouble(o);
    if (PyErr_Occurred()) {   // an int beyond the double range
        PyErr_Clear();
        return false;
    }
    *out = static_cast<float>(v);
    return true;
}

void* stream_of(PyObject* o) { return PyLong_AsVoidPtr(o); }

// A C++ exception of a tensor accessor (a tensor without storage): the general
// path meets the same tensor and reports it. (without_gil lets none of the
// library's through.)
template <typename Body>
PyObject* guarded(const Body& body) {
    try {
        return body();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// step(params, momentum, grads, gow, n_groups, lr, mu, wd, replicas, reduction,
//      broadcast, lr_device or None, device, stream)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t na) {
    return guarded([&]() -> PyObject* {
        if (na != 14) Py_RETURN_NONE;
        int32_t dev, groups, reduction, bcast;
        const at::Tensor* p = plain(a[0]);
        if (!p || !small_int(a[12], &dev) || !(p = plain(a[0], at::kFloat, -1, dev))) Py_RETURN_NONE;
        const int64_t n = p->numel();
        const at::Tensor* m = plain(a[1], at::kFloat, n, dev);
        void *grads[LSGD_MAX_WORKERS], *reps[LSGD_MAX_REPLICAS];
        int32_t gow[LSGD_MAX_WORKERS];
        int N, R;
        lsgd_dtype gdt, rdt;
        float lr, mu, wd;
        if (!m || !addresses(a[2], n, dev, grads, LSGD_MAX_WORKERS, &N, &gdt) || !membership(a[3], N, gow) ||
            !small_int(a[4], &groups) || !number(a[5], &lr) || !number(a[6], &mu) || !number(a[7], &wd) ||
            !addresses(a[8], n, dev, reps, LSGD_MAX_REPLICAS, &R, &rdt) || !small_int(a[9], &reduction) ||
            !small_int(a[10], &bcast))
            Py_RETURN_NONE;
        lsgd_step_options o = {reduction, bcast, nullptr};
        if (a[11] != Py_None) {
            const at::Tensor* l = plain(a[11], at::kFloat, -1, dev);
            if (!l || l->numel() < 1) Py_RETURN_NONE;
            o.lr_device = static_cast<const float*>(l->data_ptr());
        }
        float* pp = static_cast<float*>(p->data_ptr());
        float* mp = static_cast<float*>(m->data_ptr());
        void* stream = stream_of(a[13]);
        return without_gil([&] {
            return lsgd_step_ex(pp, mp, grads, gdt, N, gow, groups, n, lr, mu, wd, reps, R, rdt, &o, stream);
        });
    });
}

// group_mean(grads, gow, n_groups, out, device, stream)
PyObject* group_mean(PyObject*, PyObject* const* a, Py_ssize_t na) {
    return guarded([&]() -> PyObject* {
        int32_t dev, groups;
        if (na != 6 || !small_int(a[2], &groups) || !small_int(a[4], &dev)) Py_RETURN_NONE;
        if ((!PyList_CheckExact(a[0]) && !PyTuple_CheckExact(a[0])) || PySequence_Fast_GET_SIZE(a[0]) < 1) Py_RETURN_NONE;
        const at::Tensor* first = plain(PySequence_Fast_GET_ITEM(a[0], 0));
        if (!first) Py_RETURN_NONE;
        const int64_t n = first->numel();
        void *grads[LSGD_MAX_WORKERS], *out[LSGD_MAX_WORKERS];
        int32_t gow[LSGD_MAX_WORKERS];
        int N, G;
        lsgd_dtype gdt, odt;
        if (!addresses(a[0], n, dev, grads, LSGD_MAX_WORKERS, &N, &gdt) || !membership(a[1], N, gow) ||
            !addresses(a[3], n, dev, out, LSGD_MAX_WORKERS, &G, &odt) || G != groups || odt != LSGD_F32)
            Py_RETURN_NONE;
        void* stream = stream_of(a[5]);
        return without_gil([&] {
            return lsgd_group_mean(grads, gdt, N, gow, groups, n, reinterpret_cast<float* const*>(out), stream);
        });
    });
}

// global_mean(means, out, device, stream)
PyObject* global_mean(PyObject*, PyObject* const* a, Py_ssize_t na) {
    return guarded([&]() -> PyObject* {
        int32_t dev;
        if (na != 4 || !small_int(a[2], &dev)) Py_RETURN_NONE;
        const at::Tensor* out = plain(a[1], at::kFloat, -1, dev);
        if (!out) Py_RETURN_NONE;
        const int64_t n = out->numel();
        void* in[LSGD_MAX_WORKERS];
        int G;
        lsgd_dtype dt;
        if (!addresses(a[0], n, dev, in, LSGD_MAX_WORKERS, &G, &dt) || dt != LSGD_F32) Py_RETURN_NONE;
        float* op = static_cast<float*>(out->data_ptr());
        void* stream = stream_of(a[3]);
        return without_gil([&] { return lsgd_global_mean(reinterpret_cast<const float* const*>(in), G, n, op, stream); });
    });
}

// sgd_step(params, momentum, grad_mean, lr, mu, wd, replicas, device, stream)
PyObject* sgd_step(PyObject*, PyObject* const* a, Py_ssize_t na) {
    return guarded([&]() -> PyObject* {
        int32_t dev;
        if (na != 9 || !small_int(a[7], &dev)) Py_RETURN_NONE;
        const at::Tensor* p = plain(a[0], at::kFloat, -1, dev);
        if (!p) Py_RETURN_NONE;
        const int64_t n = p->numel();
        const at::Tensor *m = plain(a[1], at::kFloat, n, dev), *g = plain(a[2], at::kFloat, n, dev);
        void* reps[LSGD_MAX_REPLICAS];
        int R;
        lsgd_dtype rdt;
        float lr, mu, wd;
        if (!m || !g || !number(a[3], &lr) || !number(a[4], &mu) || !number(a[5], &wd) ||
            !addresses(a[6], n, dev, reps, LSGD_MAX_REPLICAS, &R, &rdt))
            Py_RETURN_NONE;
        float *pp = static_cast<float*>(p->data_ptr()), *mp = static_cast<float*>(m->data_ptr());
        const float* gp = static_cast<const float*>(g->data_ptr());
        void* stream = stream_of(a[8]);
        return without_gil([&] { return lsgd_sgd_step(pp, mp, gp, n, lr, mu, wd, reps, R, rdt, stream); });
    });
}

// copy_out(params, replicas, device, stream)
PyObject* copy_out(PyObject*, PyObject* const* a, Py_ssize_t na) {
    return guarded([&]() -> PyObject* {
        int32_t dev;
        if (na != 4 || !small_int(a[2], &dev)) Py_RETURN_NONE;
        const at::Tensor* p = plain(a[0], at::kFloat, -1, dev);
        if (!p) Py_RETURN_NONE;
        const int64_t n = p->numel();
        void* reps[LSGD_MAX_REPLICAS];
        int R;
        lsgd_dtype rdt;
        if (!addresses(a[1], n, dev, reps, LSGD_MAX_REPLICAS, &R, &rdt)) Py_RETURN_NONE;
        const float* pp = static_cast<const float*>(p->data_ptr());
        void* stream = stream_of(a[3]);
        return without_gil([&] { return lsgd_copy_out(pp, n, reps, R, rdt, stream); });
    });
}

PyMethodDef methods[] = {
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(step)), METH_FASTCALL, nullptr},
    {"group_mean", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(group_mean)), METH_FASTCALL, nullptr},
    {"global_mean", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(global_mean)), METH_FASTCALL, nullptr},
    {"sgd_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(sgd_step)), METH_FASTCALL, nullptr},
    {"copy_out", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(copy_out)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_build", LSGD_TORCH_BUILD) < 0) Py_CLEAR(m);
    return m;
}
