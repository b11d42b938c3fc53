// The calls that a training step makes, as functions of a Python extension: tensors in, the C ABI's status out.
//
// A small layer's call takes less time on the GPU than its arguments took on their way through Python and ctypes
// (checks, addresses and conversions of up to 18 arguments: 4 to 5 us of a call); here they take 0.5 us.
// Argument checks are those of the binding: every tensor contiguous and on the GPU, None stands for NULL.  The
// interpreter lock is given back while the library launches, as ctypes does.
#include <exception>

#include <torch/csrc/autograd/python_variable.h>

#include "falqon.h"

namespace {

// Arguments of one call, read in order.  After a failed read (Python error set) the others return nothing.
class Args {
public:
    Args(PyObject* const* args, Py_ssize_t count, Py_ssize_t want) : args_(args)
    {
        if (count != want) {
            PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", count, want);
            failed_ = true;
        }
    }
    bool failed() const { return failed_; }

    const at::Tensor* tensor()                                       // null for None
    {
        if (failed_) return nullptr;
        PyObject* const o = args_[next_++];
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) return fail(PyExc_TypeError, "a tensor or None expected");
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) return fail(PyExc_ValueError, "tensors must be contiguous GPU tensors");
        return &t;
    }
    const at::Tensor* matrix(bool longer = false)                    // its shape is asked for; longer: the first two dimensions of it
    {
        const at::Tensor* const t = tensor();
        if (failed_) return nullptr;
        if (!t) return fail(PyExc_AttributeError, "'NoneType' object has no attribute 'shape'");
        if (longer ? t->dim() < 2 : t->dim() != 2) return fail(PyExc_ValueError, "a tensor of two dimensions expected");
        return t;
    }
    int64_t integer()
    {
        if (failed_) return 0;
        const long long v = PyLong_AsLongLong(args_[next_++]);
        if (v == -1 && PyErr_Occurred()) failed_ = true;
        return v;
    }
    double real()
    {
        if (failed_) return 0.0;
        const double v = PyFloat_AsDouble(args_[next_++]);
        if (v == -1.0 && PyErr_Occurred()) failed_ = true;
        return v;
    }
    void* address() { return reinterpret_cast<void*>(static_cast<uintptr_t>(unsigned_integer())); }
    // of an output whose type the caller chooses; `absent` for None
    falqon_dtype dtype(const at::Tensor* t, falqon_dtype absent)
    {
        if (failed_ || !t) return absent;
        if (t->scalar_type() == at::kBFloat16) return FALQON_BF16;
        if (t->scalar_type() == at::kFloat) return FALQON_F32;
        PyErr_Format(PyExc_TypeError, "unsupported dtype %s", c10::toString(t->scalar_type()));
        failed_ = true;
        return absent;
    }
    const at::Tensor* fail(PyObject* type, const char* what)
    {
        PyErr_SetString(type, what);
        failed_ = true;
        return nullptr;
    }

private:
    uint64_t unsigned_integer()
    {
        if (failed_) return 0;
        const unsigned long long v = PyLong_AsUnsignedLongLong(args_[next_++]);
        if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) failed_ = true;
        return v;
    }
    PyObject* const* args_;
    Py_ssize_t next_ = 0;
    bool failed_ = false;
};

template <typename T = void>
T* data(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }
size_t bytes(const at::Tensor* t) { return t ? t->nbytes() : 0; }

// f() without the interpreter lock; its status as a Python integer
template <typename F>
PyObject* status_of(F f)
{
    falqon_status status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// No C++ exception leaves a call.
template <typename F>
PyObject* guarded(F f)
{
    try {
        return f();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}

PyObject* melded_fwd(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject* {
        Args a(args, count, 12);
        const at::Tensor *x = a.tensor(), *wq = a.tensor(), *s_w = a.tensor();
        const int64_t m = a.integer(), r = a.integer();
        const at::Tensor *xq = a.matrix(), *s_x = a.tensor(), *y = a.tensor(), *o_a = a.tensor(), *amax = a.tensor(), *ws = a.tensor();
        if (!a.failed() && !y) a.fail(PyExc_AttributeError, "'NoneType' object has no attribute 'dtype'");
        const falqon_dtype yt = a.dtype(y, FALQON_BF16);
        void* const stream = a.address();
        if (a.failed()) return nullptr;
        const int64_t T = xq->size(0), n = xq->size(1);
        void *const px = data(x), *const py = data(y), *const po = data(o_a), *const pw = data(ws);
        uint8_t *const pwq = data<uint8_t>(wq), *const pxq = data<uint8_t>(xq);
        float *const psw = data<float>(s_w), *const psx = data<float>(s_x), *const pam = data<float>(amax);
        const size_t size = bytes(ws);
        return status_of([=] { return falqon_melded_fwd(px, pwq, psw, T, n, m, r, pxq, psx, py, yt, po, pam, pw, size, stream); });
    });
}

template <bool ADDS>
PyObject* melded_bwd(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject* {
        Args a(args, count, 16);
        const at::Tensor *dy = a.matrix(), *wq = a.tensor(), *s_w = a.tensor(), *o_a = a.tensor(), *amax = a.tensor();
        const int64_t n = a.integer(), r = a.integer();
        const at::Tensor *dyq = a.tensor(), *s_dy = a.tensor(), *dx = a.tensor(), *d_b = a.tensor(), *buf = a.tensor();
        const float lr = static_cast<float>(a.real());
        const at::Tensor *ws = a.tensor(), *scores = a.tensor();
        const falqon_dtype dxt = a.dtype(dx, FALQON_BF16);
        void* const stream = a.address();
        if (a.failed()) return nullptr;
        const int64_t T = dy->size(0), m = dy->size(1);
        void *const pdy = data(dy), *const po = data(o_a), *const pdx = data(dx), *const pw = data(ws);
        uint8_t *const pwq = data<uint8_t>(wq), *const pq = data<uint8_t>(dyq);
        float *const psw = data<float>(s_w), *const pam = data<float>(amax), *const ps = data<float>(s_dy), *const pdb = data<float>(d_b), *const pb = data<float>(buf);
        double* const psc = data<double>(scores);
        const size_t size = bytes(ws);
        return status_of([=] {
            return ADDS ? falqon_melded_bwd_add(pdy, pwq, psw, po, pam, T, n, m, r, pq, ps, pdx, pdb, pb, lr, psc, pw, size, stream)
                        : falqon_melded_bwd(pdy, pwq, psw, po, pam, T, n, m, r, pq, ps, pdx, dxt, pdb, pb, lr, psc, pw, size, stream);
        });
    });
}

PyObject* proxy_update(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject* {
        Args a(args, count, 10);
        const at::Tensor *buf = a.tensor(), *wq = a.matrix(true);
        const int64_t m = a.integer(), r = a.integer(), k = a.integer();
        const at::Tensor *idx = a.tensor(), *ws = a.tensor();
        const int clear = a.integer() != 0;
        const at::Tensor* scores = a.tensor();
        void* const stream = a.address();
        if (a.failed()) return nullptr;
        const int64_t n = wq->size(1);
        float* const pb = data<float>(buf);
        uint8_t* const pwq = data<uint8_t>(wq);
        int32_t* const pi = data<int32_t>(idx);
        double* const psc = data<double>(scores);
        void* const pw = data(ws);
        const size_t size = bytes(ws);
        return status_of([=] { return falqon_proxy_update(pb, pwq, n, m, r, k, pi, clear, psc, pw, size, stream); });
    });
}

PyObject* grad_sqnorm(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject* {
        Args a(args, count, 4);
        const at::Tensor *g = a.tensor(), *sum = a.tensor(), *ws = a.tensor();
        if (!a.failed() && !g) a.fail(PyExc_AttributeError, "'NoneType' object has no attribute 'numel'");
        void* const stream = a.address();
        if (a.failed()) return nullptr;
        float* const pg = data<float>(g);
        double* const ps = data<double>(sum);
        void* const pw = data(ws);
        const int64_t elements = g->numel();
        const size_t size = bytes(ws);
        return status_of([=] { return falqon_grad_sqnorm(pg, elements, ps, pw, size, stream); });
    });
}

PyObject* adamw_delta(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    return guarded([&]() -> PyObject* {
        Args a(args, count, 12);
        const at::Tensor *d_b = a.matrix(), *avg = a.tensor(), *avg_sq = a.tensor(), *buf = a.tensor();
        const int64_t step = a.integer();
        const double lr = a.real(), beta1 = a.real(), beta2 = a.real(), eps = a.real();
        const at::Tensor* sum = a.tensor();
        const double max_norm = a.real();
        void* const stream = a.address();
        if (a.failed()) return nullptr;
        const int64_t m = d_b->size(0), r = d_b->size(1);
        float *const pd = data<float>(d_b), *const pa = data<float>(avg), *const pq = data<float>(avg_sq), *const pb = data<float>(buf);
        double* const ps = data<double>(sum);
        return status_of([=] { return falqon_adamw_delta(pd, pa, pq, pb, m, r, step, lr, beta1, beta2, eps, ps, max_norm, stream); });
    });
}

PyObject* workspace_bytes(PyObject*, PyObject* const* args, Py_ssize_t count)
{
    Args a(args, count, 4);
    const int64_t T = a.integer(), n = a.integer(), m = a.integer(), r = a.integer();
    if (a.failed()) return nullptr;
    return PyLong_FromSize_t(falqon_workspace_bytes(T, n, m, r));
}

PyCFunction fast(PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t))
{
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef methods[] = {
    {"melded_fwd", fast(melded_fwd), METH_FASTCALL, nullptr},
    {"melded_bwd", fast(melded_bwd<false>), METH_FASTCALL, nullptr},
    {"melded_bwd_add", fast(melded_bwd<true>), METH_FASTCALL, nullptr},
    {"proxy_update", fast(proxy_update), METH_FASTCALL, nullptr},
    {"grad_sqnorm", fast(grad_sqnorm), METH_FASTCALL, nullptr},
    {"adamw_delta", fast(adamw_delta), METH_FASTCALL, nullptr},
    {"workspace_bytes", fast(workspace_bytes), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
