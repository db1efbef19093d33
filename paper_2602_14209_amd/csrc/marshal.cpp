// Argument marshalling of the Python binding: torch tensors in, C-ABI calls out (include/mage.h).
//
// A denoising step takes 6 us on the GPU and is one Python call, so what the host spends per call decides
// how fast a decoder that does not capture graphs runs.  Marshalled with ctypes and torch's Python API a call
// took 8.2 us of host time (2.8 us of it torch.cuda.current_stream(), ~0.2 us per tensor for the device and layout
// checks and the address, the rest ctypes' own conversions).  The same work on the C++ side of torch is a few
// loads per argument.  The checks and their messages are those of the ctypes path (binding._ptr).
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/mage.h"

namespace {

// The positional arguments of one call; the first failed conversion sets the Python error and `bad`.
struct Args {
    PyObject *const *v;
    bool bad;

    Args(PyObject *const *values, Py_ssize_t n, Py_ssize_t want) : v(values), bad(false)
    {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
            bad = true;
        }
    }

    // a ctypes mage_shape (its buffer is the struct)
    mage_shape shape(int i)
    {
        mage_shape s{};
        if (bad) return s;
        Py_buffer view;
        if (PyObject_GetBuffer(v[i], &view, PyBUF_SIMPLE) != 0) {
            bad = true;
            return s;
        }
        if (view.len == (Py_ssize_t)sizeof(s)) {
            memcpy(&s, view.buf, sizeof(s));
        } else {
            PyErr_SetString(PyExc_TypeError, "mage_shape expected");
            bad = true;
        }
        PyBuffer_Release(&view);
        return s;
    }

    const at::Tensor *tensor(int i)      // nullptr for None
    {
        if (bad || v[i] == Py_None) return nullptr;
        if (!THPVariable_Check(v[i])) {
            PyErr_SetString(PyExc_TypeError, "torch tensor or None expected");
            bad = true;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(v[i]);
        const char *what = !t.is_cuda() ? "device tensor expected" : !t.is_contiguous() ? "contiguous tensor expected" : nullptr;
        if (what) {
            PyErr_SetString(PyExc_ValueError, what);
            bad = true;
            return nullptr;
        }
        return &t;
    }

    template <class T = void>
    T *ptr(int i)
    {
        const at::Tensor *t = tensor(i);
        return t ? static_cast<T *>(t->data_ptr()) : nullptr;
    }

    size_t bytes(int i)                  // of an argument that ptr() has accepted
    {
        return bad || v[i] == Py_None ? 0 : THPVariable_Unpack(v[i]).nbytes();
    }

    int integer(int i)
    {
        if (bad) return 0;
        PyObject *o = PyNumber_Long(v[i]);           // as int(v): numpy and torch scalars too
        if (!o) {
            bad = true;
            return 0;
        }
        const long x = PyLong_AsLong(o);
        Py_DECREF(o);
        if (x == -1 && PyErr_Occurred()) {
            bad = true;
        } else if (x != (int)x) {
            PyErr_SetString(PyExc_OverflowError, "argument does not fit a C int");
            bad = true;
        }
        return (int)x;
    }

    // None: the current stream of the current device; otherwise any object with a cuda_stream handle
    void *stream(int i)
    {
        if (bad) return nullptr;
        if (v[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject *h = PyObject_GetAttrString(v[i], "cuda_stream");
        if (!h) {
            bad = true;
            return nullptr;
        }
        void *p = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
        if (!p && PyErr_Occurred()) bad = true;
        return p;
    }
};

// Converts, calls without the interpreter lock (a launch can block while its queue is full), returns the status code.
template <class Convert>
PyObject *call(PyObject *const *v, Py_ssize_t n, Py_ssize_t want, Convert convert)
{
    try {
        Args a(v, n, want);
        auto launch = convert(a);
        if (a.bad) return nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = launch();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define MAGE_ENTRY(name, want, ...)                                        \
    PyObject *py_##name(PyObject *, PyObject *const *v, Py_ssize_t n)      \
    {                                                                      \
        return call(v, n, want, [](Args &a) { __VA_ARGS__ });              \
    }

MAGE_ENTRY(select, 7,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2); auto *idx = a.ptr<int32_t>(3); auto *alpha = a.ptr<float>(4);
    void *ws = a.ptr(5); const size_t wb = a.bytes(5); void *st = a.stream(6);
    return [=] { return mage_select(&s, q, kc, idx, alpha, ws, wb, st); };)

MAGE_ENTRY(select_static, 6,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2); auto *idx = a.ptr<int32_t>(3); auto *alpha = a.ptr<float>(4);
    void *st = a.stream(5);
    return [=] { return mage_select_static(&s, q, kc, idx, alpha, st); };)

MAGE_ENTRY(block_probs, 6,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2); auto *pbar = a.ptr<float>(3);
    void *ws = a.ptr(4); const size_t wb = a.bytes(4); void *st = a.stream(5);
    return [=] { return mage_block_probs(&s, q, kc, pbar, ws, wb, st); };)

MAGE_ENTRY(exact_attn, 10,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2), *vc = a.ptr(3), *kb = a.ptr(4), *vb = a.ptr(5);
    auto *out = a.ptr<float>(6); auto *lse = a.ptr<float>(7); void *ws = a.ptr(8); const size_t wb = a.bytes(8); void *st = a.stream(9);
    return [=] { return mage_exact_attn(&s, q, kc, vc, kb, vb, out, lse, ws, wb, st); };)

MAGE_ENTRY(sparse_attn, 11,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2), *vc = a.ptr(3); auto *idx = a.ptr<int32_t>(4);
    const void *kb = a.ptr(5), *vb = a.ptr(6); auto *out = a.ptr<float>(7); auto *lse = a.ptr<float>(8);
    void *ws = a.ptr(9); const size_t wb = a.bytes(9); void *st = a.stream(10);
    return [=] { return mage_sparse_attn(&s, q, kc, vc, idx, kb, vb, out, lse, ws, wb, st); };)

MAGE_ENTRY(step1, 12,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *kc = a.ptr(2), *vc = a.ptr(3), *kb = a.ptr(4), *vb = a.ptr(5);
    auto *out = a.ptr<float>(6); auto *lse = a.ptr<float>(7); auto *idx = a.ptr<int32_t>(8); auto *alpha = a.ptr<float>(9);
    void *ws = a.ptr(10); const size_t wb = a.bytes(10); void *st = a.stream(11);
    return [=] { return mage_step1(&s, q, kc, vc, kb, vb, out, lse, idx, alpha, ws, wb, st); };)

MAGE_ENTRY(compact, 7,
    const mage_shape s = a.shape(0); const void *kc = a.ptr(1), *vc = a.ptr(2); auto *idx = a.ptr<int32_t>(3);
    void *ks = a.ptr(4), *vs = a.ptr(5); void *st = a.stream(6);
    return [=] { return mage_compact(&s, kc, vc, idx, ks, vs, st); };)

MAGE_ENTRY(sparse_attn_compact, 10,
    const mage_shape s = a.shape(0); const void *q = a.ptr(1), *ks = a.ptr(2), *vs = a.ptr(3), *kb = a.ptr(4), *vb = a.ptr(5);
    auto *out = a.ptr<float>(6); auto *lse = a.ptr<float>(7); void *ws = a.ptr(8); const size_t wb = a.bytes(8); void *st = a.stream(9);
    return [=] { return mage_sparse_attn_compact(&s, q, ks, vs, kb, vb, out, lse, ws, wb, st); };)

MAGE_ENTRY(sparse_attn_batched, 11,
    const mage_shape s = a.shape(0); const int n_seq = a.integer(1); const void *q = a.ptr(2), *kc = a.ptr(3), *vc = a.ptr(4);
    auto *idx = a.ptr<int32_t>(5); const void *kb = a.ptr(6), *vb = a.ptr(7); auto *out = a.ptr<float>(8); auto *lse = a.ptr<float>(9);
    void *st = a.stream(10);
    return [=] { return mage_sparse_attn_batched(&s, n_seq, q, kc, vc, idx, kb, vb, out, lse, st); };)

MAGE_ENTRY(page_summary, 5,
    const mage_shape s = a.shape(0); const int p = a.integer(1); const void *kc = a.ptr(2); void *summary = a.ptr(3); void *st = a.stream(4);
    return [=] { return mage_page_summary(&s, p, kc, summary, st); };)

MAGE_ENTRY(quest_select, 8,
    const mage_shape s = a.shape(0); const int p = a.integer(1); const void *q = a.ptr(2), *summary = a.ptr(3);
    auto *idx = a.ptr<int32_t>(4); auto *est = a.ptr<float>(5); void *ws = a.ptr(6); const size_t wb = a.bytes(6); void *st = a.stream(7);
    return [=] { return mage_quest_select(&s, p, q, summary, idx, est, ws, wb, st); };)

MAGE_ENTRY(set_overlap, 7,
    auto *x = a.ptr<int32_t>(0), *y = a.ptr<int32_t>(1); const int n_rows = a.integer(2), k = a.integer(3), a_rows = a.integer(4);
    auto *out = a.ptr<float>(5); void *st = a.stream(6);
    return [=] { return mage_set_overlap(x, y, n_rows, k, a_rows, out, st); };)

#define MAGE_METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    MAGE_METHOD(select), MAGE_METHOD(select_static), MAGE_METHOD(block_probs), MAGE_METHOD(exact_attn), MAGE_METHOD(sparse_attn),
    MAGE_METHOD(step1), MAGE_METHOD(compact), MAGE_METHOD(sparse_attn_compact), MAGE_METHOD(sparse_attn_batched),
    MAGE_METHOD(page_summary), MAGE_METHOD(quest_select), MAGE_METHOD(set_overlap), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
