// gs_call.cpp -- marshalling of the binding's calls that a step is made of, for arguments of the usual form.
//
// A call on a small range takes 2-4 us on the GPU and as much in the runtime's launch, and reading the arguments
// in Python (four attributes of each tensor, a struct from the hyper-parameters, ctypes' own conversions) took as
// long again: 13 k elements, k = 4 / 16, 7.7/10.4 us of host time per gs_accum_adamw against 3.9/4.1 here, of which 3.3
// are the launch (on a core that another program shares; 3.0 and 2.3 on one that none does).  The current stream is asked of torch natively
// too: all of a call but its launch takes 0.38 us, k = 4, against 0.50 through torch's Python functions.
//
// Every function here either makes the call and returns its status, or touches nothing and returns None: gs.py
// then reads the same arguments in its general way, which decides what is accepted and raises what it raises.
// So this file only has to recognise the usual form, never to refuse: plain CUDA tensors (torch.Tensor or
// Parameter, no subclass and no torch function mode), gradients in a list or tuple, whole numbers as int,
// HParams as gs.py defines it, the stream as None, an int or an object with an int `cuda_stream`.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include <pthread.h>

#include <cstdint>

#include "gs.h"

namespace {

// what gs.py hands over once: the library's entry points and the Python objects that are asked each time
decltype(&::gs_grad_sqnorm) f_grad_sqnorm;
decltype(&::gs_grad_sqnorm_noalloc) f_grad_sqnorm_noalloc;
decltype(&::gs_grad_accum_sqnorm) f_grad_accum_sqnorm;
decltype(&::gs_accum_add) f_accum_add;
decltype(&::gs_acc_sqnorm) f_acc_sqnorm;
decltype(&::gs_accum_adamw) f_accum_adamw;
decltype(&::gs_adamw_from_acc) f_adamw_from_acc;
decltype(&::gs_accum_adamw_oop) f_accum_adamw_oop;
decltype(&::gs_accum_adamw_spec) f_accum_adamw_spec;
PyTypeObject *hparams_type;
PyObject *in_bad_fork;
bool forked;                       // this process is a child of the one that made the set-up, or torch called it a bad fork then
PyObject *hp_names[7];

// torch's word on whether this process was forked from one that used the GPU before; any answer but False counts
bool is_bad_fork()
{
    PyObject *bad = PyObject_CallNoArgs(in_bad_fork);
    const bool yes = bad != Py_False;
    Py_XDECREF(bad);
    return yes;
}

// The reading of one call's arguments; `usual` turns false at the first that is not of the usual form.
struct Reader {
    bool usual = true;

    int64_t whole(PyObject *o)
    {
        if (!PyLong_CheckExact(o)) return no();
        int over = 0;
        const long long x = PyLong_AsLongLongAndOverflow(o, &over);
        return over ? no() : x;
    }

    int flag(PyObject *o)          // int(bool(o))
    {
        if (o == Py_True) return 1;
        if (o == Py_False) return 0;
        return (int)no();
    }

    const at::Tensor *tensor(PyObject *o)
    {
        if (!THPVariable_CheckExact(o)) return no(), nullptr;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided) return no(), nullptr;
        return &t;
    }

    // address of a tensor that holds `end` contiguous elements of `bytes` each
    template <typename T>
    T *array(PyObject *o, int64_t end, int64_t bytes)
    {
        const at::Tensor *t = tensor(o);
        if (!t) return nullptr;
        if ((int64_t)t->element_size() != bytes || t->numel() < end || !t->is_contiguous()) return no(), nullptr;
        return static_cast<T *>(t->data_ptr());
    }

    // a scalar or a workspace: any tensor, or None
    void *address(PyObject *o)
    {
        if (o == Py_None) return nullptr;
        const at::Tensor *t = tensor(o);
        return t ? t->data_ptr() : nullptr;
    }

    size_t workspace_bytes(PyObject *given, PyObject *workspace)
    {
        if (given != Py_None) {
            const int64_t n = whole(given);
            return n < 0 ? (size_t)no() : (size_t)n;
        }
        if (workspace == Py_None) return 0;
        const at::Tensor *t = tensor(workspace);
        return t ? (size_t)t->numel() * t->element_size() : 0;
    }

    // the address table, and in `k` the number of buffers unless a number is given
    void grads(PyObject *o, int64_t end, PyObject *given, const uint16_t **table, int &k)
    {
        k = 0;
        if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return (void)no();
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
        if (n < 1 || n > GS_MAX_K) return (void)no();
        for (Py_ssize_t j = 0; j < n && usual; ++j) table[j] = array<const uint16_t>(PySequence_Fast_GET_ITEM(o, j), end, 2);
        k = (int)n;
        if (given != Py_None) {
            const int64_t want = whole(given);
            if (want != n) no();           // a number of its own for the table is rare
        }
    }

    void hparams(PyObject *o, gs_adamw_hparams &hp)
    {
        if (Py_TYPE(o) != hparams_type) return (void)no();
        float *const to[6] = {&hp.lr, &hp.beta1, &hp.beta2, &hp.eps, &hp.weight_decay, &hp.max_grad_norm};
        for (int i = 0; i < 7 && usual; ++i) {
            PyObject *x = PyObject_GetAttr(o, hp_names[i]);
            if (!x) return (void)no();
            if (i == 6) {
                const int64_t step = whole(x);
                if (step < INT32_MIN || step > INT32_MAX) no();
                hp.step = (int32_t)step;
            } else if (PyFloat_CheckExact(x)) {
                *to[i] = (float)PyFloat_AS_DOUBLE(x);
            } else {
                no();
            }
            Py_DECREF(x);
        }
    }

    void *stream(PyObject *o)
    {
        if (!usual) return nullptr;
        PyObject *h = nullptr;
        if (o == Py_None) {
            // forked before the GPU was first used: as ever; after: torch refuses
            if (forked && is_bad_fork()) return no(), nullptr;
            return c10::hip::getCurrentHIPStream().stream();
        } else if (PyLong_CheckExact(o)) {
            h = Py_NewRef(o);
        } else {
            h = PyObject_GetAttrString(o, "cuda_stream");
        }
        void *s = nullptr;
        if (!h || !PyLong_CheckExact(h)) no();
        else s = PyLong_AsVoidPtr(h);
        Py_XDECREF(h);
        if (PyErr_Occurred()) no();
        return s;
    }

    int64_t no()
    {
        usual = false;
        return 0;
    }
};

// Reads with `read` and, if all is of the usual form, calls with `call`, without the interpreter's lock.
template <int NARGS, typename Read, typename Call>
PyObject *run(Py_ssize_t nargs, Read read, Call call)
{
    Reader r;
    try {
        if (nargs != NARGS || at::impl::torch_function_mode_enabled()) r.no();
        else read(r);
    } catch (...) {                        // a tensor without an address: the general way raises for it
        r.no();
    }
    if (!r.usual) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    gs_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// grads, begin, end, d_sqnorm, d_workspace, workspace_bytes, accumulate, stream, k
PyObject *grad_sqnorm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    int k = 0, acc = 0;
    int64_t b = 0, e = 0;
    double *sq = nullptr;
    void *ws = nullptr, *s = nullptr;
    size_t bytes = 0;
    return run<9>(n, [&](Reader &r) {
        b = r.whole(a[1]), e = r.whole(a[2]);
        r.grads(a[0], e, a[8], g, k);
        sq = static_cast<double *>(r.address(a[3])), ws = r.address(a[4]);
        bytes = r.workspace_bytes(a[5], a[4]), acc = r.flag(a[6]), s = r.stream(a[7]);
    }, [&] { return f_grad_sqnorm(g, k, b, e, sq, acc, ws, bytes, s); });
}

// grads, begin, end, d_sqnorm, accumulate, stream, k
PyObject *grad_sqnorm_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    int k = 0, acc = 0;
    int64_t b = 0, e = 0;
    double *sq = nullptr;
    void *s = nullptr;
    return run<7>(n, [&](Reader &r) {
        b = r.whole(a[1]), e = r.whole(a[2]);
        r.grads(a[0], e, a[6], g, k);
        sq = static_cast<double *>(r.address(a[3])), acc = r.flag(a[4]), s = r.stream(a[5]);
    }, [&] { return f_grad_sqnorm_noalloc(g, k, b, e, sq, acc, s); });
}

// grads, begin, end, acc_f32, d_sqnorm, d_workspace, workspace_bytes, accumulate, stream, k
PyObject *grad_accum_sqnorm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    int k = 0, acc = 0;
    int64_t b = 0, e = 0;
    float *sum = nullptr;
    double *sq = nullptr;
    void *ws = nullptr, *s = nullptr;
    size_t bytes = 0;
    return run<10>(n, [&](Reader &r) {
        b = r.whole(a[1]), e = r.whole(a[2]);
        r.grads(a[0], e, a[9], g, k);
        sum = r.array<float>(a[3], e, 4);
        sq = static_cast<double *>(r.address(a[4])), ws = r.address(a[5]);
        bytes = r.workspace_bytes(a[6], a[5]), acc = r.flag(a[7]), s = r.stream(a[8]);
    }, [&] { return f_grad_accum_sqnorm(g, k, b, e, sum, sq, acc, ws, bytes, s); });
}

// acc_f32, grad_bf16, first, begin, end, d_sqnorm, d_workspace, workspace_bytes, accumulate, stream
PyObject *accum_add(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int first = 0, acc = 0;
    int64_t b = 0, e = 0;
    float *sum = nullptr;
    const uint16_t *g = nullptr;
    double *sq = nullptr;
    void *ws = nullptr, *s = nullptr;
    size_t bytes = 0;
    return run<10>(n, [&](Reader &r) {
        b = r.whole(a[3]), e = r.whole(a[4]);
        sum = r.array<float>(a[0], e, 4), g = r.array<const uint16_t>(a[1], e, 2), first = r.flag(a[2]);
        sq = static_cast<double *>(r.address(a[5])), ws = r.address(a[6]);
        bytes = r.workspace_bytes(a[7], a[6]), acc = r.flag(a[8]), s = r.stream(a[9]);
    }, [&] { return f_accum_add(sum, g, first, b, e, sq, acc, ws, bytes, s); });
}

// acc_f32, begin, end, d_sqnorm, d_workspace, workspace_bytes, accumulate, stream
PyObject *acc_sqnorm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    int acc = 0;
    int64_t b = 0, e = 0;
    const float *sum = nullptr;
    double *sq = nullptr;
    void *ws = nullptr, *s = nullptr;
    size_t bytes = 0;
    return run<8>(n, [&](Reader &r) {
        b = r.whole(a[1]), e = r.whole(a[2]);
        sum = r.array<const float>(a[0], e, 4);
        sq = static_cast<double *>(r.address(a[3])), ws = r.address(a[4]);
        bytes = r.workspace_bytes(a[5], a[4]), acc = r.flag(a[6]), s = r.stream(a[7]);
    }, [&] { return f_acc_sqnorm(sum, b, e, sq, acc, ws, bytes, s); });
}

// p, m, v, w_bf16, grads, begin, end, hp, d_sqnorm, stream, k
PyObject *accum_adamw(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    gs_adamw_hparams hp = {};
    int k = 0;
    int64_t b = 0, e = 0;
    float *p = nullptr, *m = nullptr, *v = nullptr;
    uint16_t *w = nullptr;
    const double *sq = nullptr;
    void *s = nullptr;
    return run<11>(n, [&](Reader &r) {
        b = r.whole(a[5]), e = r.whole(a[6]);
        r.grads(a[4], e, a[10], g, k);
        p = r.array<float>(a[0], e, 4), m = r.array<float>(a[1], e, 4), v = r.array<float>(a[2], e, 4);
        w = r.array<uint16_t>(a[3], e, 2);
        r.hparams(a[7], hp);
        sq = static_cast<const double *>(r.address(a[8])), s = r.stream(a[9]);
    }, [&] { return f_accum_adamw(p, m, v, w, g, k, b, e, &hp, sq, s); });
}

// p, m, v, w_bf16, acc_f32, begin, end, hp, d_sqnorm, stream
PyObject *adamw_from_acc(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    gs_adamw_hparams hp = {};
    int64_t b = 0, e = 0;
    float *p = nullptr, *m = nullptr, *v = nullptr;
    const float *sum = nullptr;
    uint16_t *w = nullptr;
    const double *sq = nullptr;
    void *s = nullptr;
    return run<10>(n, [&](Reader &r) {
        b = r.whole(a[5]), e = r.whole(a[6]);
        p = r.array<float>(a[0], e, 4), m = r.array<float>(a[1], e, 4), v = r.array<float>(a[2], e, 4);
        w = r.array<uint16_t>(a[3], e, 2), sum = r.array<const float>(a[4], e, 4);
        r.hparams(a[7], hp);
        sq = static_cast<const double *>(r.address(a[8])), s = r.stream(a[9]);
    }, [&] { return f_adamw_from_acc(p, m, v, w, sum, b, e, &hp, sq, s); });
}

// p, m, v, p_out, m_out, v_out, w_bf16, grads, begin, end, hp, d_sqnorm, stream, k
PyObject *accum_adamw_oop(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    gs_adamw_hparams hp = {};
    int k = 0;
    int64_t b = 0, e = 0;
    float *st[6] = {};
    uint16_t *w = nullptr;
    const double *sq = nullptr;
    void *s = nullptr;
    return run<14>(n, [&](Reader &r) {
        b = r.whole(a[8]), e = r.whole(a[9]);
        r.grads(a[7], e, a[13], g, k);
        for (int i = 0; i < 6; ++i) st[i] = r.array<float>(a[i], e, 4);
        w = r.array<uint16_t>(a[6], e, 2);
        r.hparams(a[10], hp);
        sq = static_cast<const double *>(r.address(a[11])), s = r.stream(a[12]);
    }, [&] { return f_accum_adamw_oop(st[0], st[1], st[2], st[3], st[4], st[5], w, g, k, b, e, &hp, sq, s); });
}

// p, m, v, p_out, m_out, v_out, w_bf16, grads, begin, end, hp, d_sqnorm, d_workspace, workspace_bytes, accumulate, stream, k
PyObject *accum_adamw_spec(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    const uint16_t *g[GS_MAX_K];
    gs_adamw_hparams hp = {};
    int k = 0, acc = 0;
    int64_t b = 0, e = 0;
    float *st[6] = {};
    uint16_t *w = nullptr;
    double *sq = nullptr;
    void *ws = nullptr, *s = nullptr;
    size_t bytes = 0;
    return run<17>(n, [&](Reader &r) {
        b = r.whole(a[8]), e = r.whole(a[9]);
        r.grads(a[7], e, a[16], g, k);
        for (int i = 0; i < 6; ++i) st[i] = r.array<float>(a[i], e, 4);
        w = r.array<uint16_t>(a[6], e, 2);
        r.hparams(a[10], hp);
        sq = static_cast<double *>(r.address(a[11])), ws = r.address(a[12]);
        bytes = r.workspace_bytes(a[13], a[12]), acc = r.flag(a[14]), s = r.stream(a[15]);
    }, [&] {
        return f_accum_adamw_spec(st[0], st[1], st[2], st[3], st[4], st[5], w, g, k, b, e, &hp, sq, acc, ws, bytes, s);
    });
}

// entry points by name (addresses in the order below), HParams, in a bad fork
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *f[9];
    if (n != 11) return PyErr_Format(PyExc_TypeError, "setup takes 11 arguments"), nullptr;
    for (int i = 0; i < 9; ++i)
        if (!(f[i] = PyLong_AsVoidPtr(a[i]))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "null entry point");
    if (!PyType_Check(a[9])) return PyErr_Format(PyExc_TypeError, "HParams is not a class");
    f_grad_sqnorm = reinterpret_cast<decltype(f_grad_sqnorm)>(f[0]);
    f_grad_sqnorm_noalloc = reinterpret_cast<decltype(f_grad_sqnorm_noalloc)>(f[1]);
    f_grad_accum_sqnorm = reinterpret_cast<decltype(f_grad_accum_sqnorm)>(f[2]);
    f_accum_add = reinterpret_cast<decltype(f_accum_add)>(f[3]);
    f_acc_sqnorm = reinterpret_cast<decltype(f_acc_sqnorm)>(f[4]);
    f_accum_adamw = reinterpret_cast<decltype(f_accum_adamw)>(f[5]);
    f_adamw_from_acc = reinterpret_cast<decltype(f_adamw_from_acc)>(f[6]);
    f_accum_adamw_oop = reinterpret_cast<decltype(f_accum_adamw_oop)>(f[7]);
    f_accum_adamw_spec = reinterpret_cast<decltype(f_accum_adamw_spec)>(f[8]);
    const char *const names[7] = {"lr", "beta1", "beta2", "eps", "weight_decay", "max_grad_norm", "step"};
    for (int i = 0; i < 7; ++i)
        if (!(hp_names[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
    hparams_type = reinterpret_cast<PyTypeObject *>(Py_NewRef(a[9]));       // kept until the process ends
    in_bad_fork = Py_NewRef(a[10]);
    forked = is_bad_fork();                    // a child that makes the set-up itself: the handler below did not run in it
    PyErr_Clear();
    if (pthread_atfork(nullptr, nullptr, [] { forked = true; }) != 0) return PyErr_NoMemory();
    Py_RETURN_NONE;
}

#define GS_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    GS_METHOD(setup), GS_METHOD(grad_sqnorm), GS_METHOD(grad_sqnorm_noalloc), GS_METHOD(grad_accum_sqnorm),
    GS_METHOD(accum_add), GS_METHOD(acc_sqnorm), GS_METHOD(accum_adamw), GS_METHOD(adamw_from_acc),
    GS_METHOD(accum_adamw_oop), GS_METHOD(accum_adamw_spec), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gs_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__gs_call(void) { return PyModule_Create(&module); }
