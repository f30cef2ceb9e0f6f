// The calls of small layers with their arguments checked and passed natively: binding.py's functions of the same names try these first.
//
// Such a call is bound by the host.  Of the 5.9 us of snn_subbit_conv2d_sign_prepared from Python 3.5 are the launch; checks, fields of the
// descriptor, pointers, the stream's handle and the conversion of nine arguments were the rest.  Here they take 0.3 us.
//
// A function here takes the ordinary case alone: plain torch.Tensor objects of the right type and size, on the GPU and contiguous, outputs and
// workspace given.  It returns true if it has enqueued the call.  For anything else, and where the library has refused the arguments (nothing
// is enqueued then), it returns false, and the caller goes on with its own checks, which say what is wrong.  Any other status raises here and
// now: after SNN_ERR_LAUNCH some of the call's work may be on the stream (the error can be that of a second launch, or of some earlier
// call on the thread), and a second call would do it twice.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "snn.h"

namespace {

// The library's functions, by address: this module is not linked to it.
struct Library {
    decltype(&snn_subbit_conv2d) subbit_conv2d;
    decltype(&snn_subbit_conv2d_prepared) subbit_conv2d_prepared;
    decltype(&snn_subbit_conv2d_sign_prepared) subbit_conv2d_sign_prepared;
    decltype(&snn_subbit_conv1x1_prepared) subbit_conv1x1_prepared;
    decltype(&snn_bnn_conv2d_prepared) bnn_conv2d_prepared;
    decltype(&snn_pack_activations) pack_activations;
    decltype(&snn_packed_bytes) packed_bytes;
    decltype(&snn_project_backward) project_backward;
    decltype(&snn_subset_update) subset_update;
};
Library lib;
PyTypeObject *desc_type = nullptr;
PyObject *error_type = nullptr;              // called with the status and the function's name

// Plain tensors only: subclasses have their own say in Python.
const at::Tensor *tensor(PyObject *o) { return Py_TYPE(o) == (PyTypeObject *)THPVariableClass ? &THPVariable_Unpack(o) : nullptr; }

const at::Tensor *checked(PyObject *o, at::ScalarType type)
{
    const at::Tensor *const t = tensor(o);
    return t && t->is_cuda() && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}

bool descriptor(PyObject *o, snn_conv_desc &d)
{
    if (Py_TYPE(o) != desc_type) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = view.len == (Py_ssize_t)sizeof d;
    if (ok) std::memcpy(&d, view.buf, sizeof d);
    PyBuffer_Release(&view);
    return ok && d.stride > 0;
}

int64_t out_rows(const snn_conv_desc &d) { return (d.H - 1) / d.stride + 1; }
int64_t out_cols(const snn_conv_desc &d) { return (d.W - 1) / d.stride + 1; }

// A convolution's fp32 output of the right size
const at::Tensor *output(PyObject *o, const snn_conv_desc &d)
{
    const at::Tensor *const t = checked(o, at::kFloat);
    return t && t->numel() == d.N * (int64_t)d.C_out * out_rows(d) * out_cols(d) ? t : nullptr;
}

void *stream() { return (void *)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

// Makes the call, without the interpreter's lock: whether it has been enqueued.
template <class Call>
PyObject *enqueued(const char *name, Call &&call)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    if (status == SNN_OK) Py_RETURN_TRUE;
    if (status == SNN_ERR_INVALID_ARG || status == SNN_ERR_UNSUPPORTED || status == SNN_ERR_WORKSPACE) Py_RETURN_FALSE;
    if (PyObject *const args = Py_BuildValue("(is)", status, name)) {
        PyErr_SetObject(error_type, args);
        Py_DECREF(args);
    }
    return nullptr;
}

// What raises (a tensor without memory, say) is left to the caller, too.
template <PyObject *(*F)(PyObject *const *), int N>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N) Py_RETURN_FALSE;
    try {
        return F(args);
    } catch (...) {
        Py_RETURN_FALSE;
    }
}

PyObject *subbit_conv2d(PyObject *const *a)
{
    snn_conv_desc d;
    const at::Tensor *x, *codebook, *idx, *alpha, *y, *ws;
    if (!descriptor(a[0], d) || !(x = tensor(a[1])) || !(codebook = checked(a[2], at::kShort)) || !(idx = checked(a[3], at::kShort)) ||
        !(alpha = checked(a[4], at::kFloat)) || !(y = output(a[5], d)) || !(ws = tensor(a[6])))
        Py_RETURN_FALSE;
    const void *const px = x->data_ptr(), *const pc = codebook->data_ptr(), *const pi = idx->data_ptr(), *const pa = alpha->data_ptr();
    void *const py = y->data_ptr(), *const pw = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_subbit_conv2d", [&] {
        return lib.subbit_conv2d(&d, px, (const uint16_t *)pc, (const uint16_t *)pi, (const float *)pa, (float *)py, pw, bytes, s);
    });
}

PyObject *subbit_conv2d_prepared(PyObject *const *a)
{
    snn_conv_desc d;
    const at::Tensor *x, *alpha, *ws, *y;
    if (!descriptor(a[0], d) || !(x = tensor(a[1])) || !(alpha = checked(a[2], at::kFloat)) || !(ws = tensor(a[3])) || !(y = output(a[4], d)))
        Py_RETURN_FALSE;
    const void *const px = x->data_ptr(), *const pa = alpha->data_ptr();
    void *const py = y->data_ptr(), *const pw = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_subbit_conv2d_prepared", [&] { return lib.subbit_conv2d_prepared(&d, px, (const float *)pa, (float *)py, pw, bytes, s); });
}

PyObject *bnn_conv2d_prepared(PyObject *const *a)
{
    snn_conv_desc d;
    const at::Tensor *x, *alpha, *ws, *y;
    if (!descriptor(a[0], d) || !(x = tensor(a[1])) || !(alpha = checked(a[2], at::kFloat)) || !(ws = tensor(a[3])) || !(y = output(a[4], d)))
        Py_RETURN_FALSE;
    const void *const px = x->data_ptr(), *const pa = alpha->data_ptr();
    void *const py = y->data_ptr(), *const pw = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_bnn_conv2d_prepared", [&] { return lib.bnn_conv2d_prepared(&d, px, (const float *)pa, (float *)py, pw, bytes, s); });
}

PyObject *subbit_conv2d_sign_prepared(PyObject *const *a)
{
    snn_conv_desc d;
    const at::Tensor *x, *ws, *out;
    if (!descriptor(a[0], d) || !(x = checked(a[1], at::kInt)) || !(ws = tensor(a[2])) || !(out = checked(a[3], at::kInt)) ||
        out->numel() < d.N * (int64_t)d.C_out * out_rows(d) * ((out_cols(d) + 31) / 32))
        Py_RETURN_FALSE;
    const void *const px = x->data_ptr();
    void *const po = out->data_ptr(), *const pw = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_subbit_conv2d_sign_prepared", [&] { return lib.subbit_conv2d_sign_prepared(&d, px, po, pw, bytes, s); });
}

PyObject *subbit_conv1x1_prepared(PyObject *const *a)
{
    snn_conv_desc d;
    const at::Tensor *x, *ws, *y;
    if (!descriptor(a[0], d) || !(x = checked(a[1], at::kInt)) || !(ws = tensor(a[2])) || !(y = output(a[3], d))) Py_RETURN_FALSE;
    const void *const px = x->data_ptr();
    void *const py = y->data_ptr(), *const pw = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_subbit_conv1x1_prepared", [&] { return lib.subbit_conv1x1_prepared(&d, px, (float *)py, pw, bytes, s); });
}

PyObject *pack_activations(PyObject *const *a)
{
    const at::Tensor *x, *out;
    if (!(x = checked(a[0], at::kFloat)) || x->dim() != 4 || !PyLong_CheckExact(a[1]) || !(out = checked(a[2], at::kInt))) Py_RETURN_FALSE;
    const long layout = PyLong_AsLong(a[1]);
    if (layout != SNN_ACT_BIN_ROWS && layout != SNN_ACT_BIN_CHANNELS) {
        PyErr_Clear();
        Py_RETURN_FALSE;
    }
    const auto shape = x->sizes();
    for (const int64_t v : shape)
        if (v > 0x7fffffff) Py_RETURN_FALSE;
    const int N = (int)shape[0], C = (int)shape[1], H = (int)shape[2], W = (int)shape[3];
    if ((size_t)out->numel() * 4 < lib.packed_bytes(N, C, H, W, (int)layout)) Py_RETURN_FALSE;
    const void *const px = x->data_ptr();
    void *const po = out->data_ptr(), *const s = stream();
    return enqueued("snn_pack_activations", [&] { return lib.pack_activations((const float *)px, po, N, C, H, W, (int)layout, s); });
}

PyObject *project_backward(PyObject *const *a)
{
    const at::Tensor *w, *g, *idx, *g_w, *g_p, *ws;
    if (!(w = checked(a[0], at::kFloat)) || !(g = checked(a[1], at::kFloat)) || !(idx = checked(a[2], at::kShort)) || !PyLong_CheckExact(a[3]) ||
        !(g_w = checked(a[4], at::kFloat)) || !(g_p = checked(a[5], at::kFloat)) || !(ws = tensor(a[6])))
        Py_RETURN_FALSE;
    const long K = PyLong_AsLong(a[3]);
    const int64_t n = w->numel() / 9;
    if (K < 1 || K > 512 || g->numel() != n * 9 || idx->numel() != n) {
        PyErr_Clear();
        Py_RETURN_FALSE;
    }
    const void *const pw = w->data_ptr(), *const pg = g->data_ptr(), *const pi = idx->data_ptr();
    void *const ow = g_w->data_ptr(), *const op = g_p->data_ptr(), *const pws = ws->data_ptr(), *const s = stream();
    const size_t bytes = (size_t)ws->numel();
    return enqueued("snn_project_backward", [&] {
        return lib.project_backward((const float *)pw, (const float *)pg, (const uint16_t *)pi, n, (int)K, (float *)ow, (float *)op, pws, bytes, s);
    });
}

// (codebook, dup), or false
PyObject *subset_update(PyObject *const *a)
{
    const at::Tensor *p, *m;
    if (!(p = checked(a[0], at::kFloat)) || !(m = checked(a[1], at::kChar)) || !PyFloat_CheckExact(a[2])) Py_RETURN_FALSE;
    const float theta = (float)PyFloat_AS_DOUBLE(a[2]);
    const int64_t K = p->numel() / 9;
    if (K < 1 || K > 512 || m->numel() != K * 9) Py_RETURN_FALSE;
    at::Tensor cb = at::empty({K}, p->options().dtype(at::kShort).requires_grad(false));
    at::Tensor dup = at::empty({K}, p->options().dtype(at::kByte).requires_grad(false));
    const void *const pp = p->data_ptr();
    void *const pm = m->data_ptr(), *const pc = cb.data_ptr(), *const pd = dup.data_ptr(), *const s = stream();
    PyObject *const ok = enqueued("snn_subset_update", [&] {
        return lib.subset_update((const float *)pp, (int8_t *)pm, theta, (int)K, (uint16_t *)pc, (uint8_t *)pd, s);
    });
    if (ok != Py_True) return ok;
    Py_DECREF(ok);
    PyObject *const c = THPVariable_Wrap(std::move(cb)), *const u = THPVariable_Wrap(std::move(dup));
    PyObject *const both = c && u ? PyTuple_Pack(2, c, u) : nullptr;
    Py_XDECREF(c);
    Py_XDECREF(u);
    return both;
}

// use(descriptor type, type of the errors, addresses of the library's functions in the order of Library)
PyObject *use(PyObject *, PyObject *args)
{
    PyObject *type, *error;
    unsigned long long f[9];
    if (!PyArg_ParseTuple(args, "O!O(KKKKKKKKK)", &PyType_Type, &type, &error, f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, f + 7, f + 8))
        return nullptr;
    static_assert(sizeof(Library) == sizeof f, "one address each");
    std::memcpy(&lib, f, sizeof f);
    Py_INCREF(type);
    Py_XDECREF(desc_type);
    desc_type = (PyTypeObject *)type;
    Py_INCREF(error);
    Py_XDECREF(error_type);
    error_type = error;
    Py_RETURN_NONE;
}

#define SNN_FAST(name, n) {#name, (PyCFunction)(void (*)(void))guarded<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"use", use, METH_VARARGS, nullptr},
    SNN_FAST(subbit_conv2d, 7),
    SNN_FAST(subbit_conv2d_prepared, 5),
    SNN_FAST(subbit_conv2d_sign_prepared, 4),
    SNN_FAST(subbit_conv1x1_prepared, 4),
    SNN_FAST(bnn_conv2d_prepared, 5),
    SNN_FAST(pack_activations, 3),
    SNN_FAST(project_backward, 7),
    SNN_FAST(subset_update, 3),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
