// Native half of the Python binding: what a call does between Python and the
// C ABI when its arguments are the plain case (exact strided tensors in device
// memory, unit point stride, a supported type).  run() reads pointers and
// strides, fills an fdbb_task and calls fdbb_task_run; the empty_* helpers
// allocate padded outputs.  Everything else returns None, and the Python
// functions in fdbb.py, which hold the checks and their errors, take over.
//
// A call is bounded by host time below about 2^20 points: fdbb_cons2prim spent
// 7.7 us on the host of which 3.6 us are the launch itself (stream object 2.6,
// argument checks 1.0, ctypes 0.5).
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/fdbb.h"

namespace {

int (*g_task_run)(const fdbb_task *, void *) = nullptr;
decltype(&fdbb_char_apply) g_char_apply = nullptr;
decltype(&fdbb_viscous_flux) g_viscous_flux = nullptr;
PyObject *g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

// How a slot's tensor lies: > 0 that many field rows, or one of these.
enum : long { kAbsent = 0, kBlocks = -1, kFlat = -2 };

struct Slot {
    void *ptr = nullptr;
    int64_t ld = 0;
};

// The tensor behind `o` if the plain case covers it: an exact torch.Tensor (or
// Parameter) in device memory that no transform wraps.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided) return nullptr;
    static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                              c10::DispatchKey::FuncTorchGradWrapper,
                                              c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate,
                                              c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    return t.key_set().has_any(wrapped) ? nullptr : &t;
}

// Pointer and leading dimension of a slot, with the checks of fdbb.py's
// _fields and _blocks; false where they would refuse it or the case is not
// plain.
bool slot_of(PyObject *o, long kind, long dim, Slot *s)
{
    if (kind == kAbsent) return true;
    const at::Tensor *t = plain(o);
    if (!t) return false;
    if (kind > 0) {
        if (t->dim() != 2 || t->size(0) != kind) return false;
        if (t->size(1) > 1 && t->stride(1) != 1) return false;
        s->ld = kind > 1 ? t->stride(0) : std::max<int64_t>(t->size(1), 1);
    } else if (kind == kBlocks) {
        const int64_t K = dim + 2;
        if (t->dim() != 4 || t->size(0) != dim || t->size(2) != K || t->size(3) != K) return false;
        if (t->stride(3) != 1 || t->stride(2) != K || t->stride(1) != K * K || t->stride(0) % (K * K)) return false;
        s->ld = t->stride(0) / (K * K);
    }
    s->ptr = t->data_ptr();
    return true;
}

bool dtype_of(PyObject *o, int32_t *code)
{
    const at::ScalarType st = THPVariable_Unpack(o).scalar_type();
    if (st == at::kDouble) *code = FDBB_F64;
    else if (st == at::kFloat) *code = FDBB_F32;
    else return false;
    return true;
}

bool points_of(PyObject *n, PyObject *in0, int64_t *out)
{
    if (n == Py_None) {
        *out = THPVariable_Unpack(in0).size(1);
        return true;
    }
    if (!PyLong_CheckExact(n)) return false;
    *out = PyLong_AsLongLong(n);
    return !PyErr_Occurred();
}

// The caller's stream handle, or the current stream of the current device.
bool stream_of(PyObject *stream, void **out)
{
    PyObject *h = nullptr;
    if (stream == Py_None) {
        const c10::impl::VirtualGuardImpl guard(c10::DeviceType::CUDA);
        PyObject *dev = PyLong_FromLong(guard.getDevice().index());
        if (!dev) return false;
        h = PyObject_CallOneArg(g_raw_stream, dev);
        Py_DECREF(dev);
    } else if (PyLong_CheckExact(stream)) {
        Py_INCREF(stream);
        h = stream;
    }
    if (!h) return false;
    *out = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

// Numbers as ctypes takes them for the C types of the ABI: an int for an int,
// an int or a float for a double; nothing that merely converts.
bool int_of(PyObject *o, long *out)
{
    if (!PyLong_Check(o)) return false;
    *out = PyLong_AsLong(o);
    return !PyErr_Occurred();
}

bool double_of(PyObject *o, double *out)
{
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
    *out = PyFloat_AsDouble(o);
    return !PyErr_Occurred();
}

PyObject *not_plain()
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

// run(op, dim, dir, gamma, n, stream, in0, k, in1, k, out0, k, out1, k, out2, k)
PyObject *run(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    HANDLE_TH_ERRORS
    if (na != 16 || !g_task_run) return not_plain();
    fdbb_task t{};
    long op, dim, dir;
    if (!int_of(a[0], &op) || !int_of(a[1], &dim) || !int_of(a[2], &dir) || !double_of(a[3], &t.gamma)) return not_plain();
    t.op = (int32_t)op, t.dim = (int32_t)dim, t.dir = (int32_t)dir;
    Slot s[5];
    for (int k = 0; k < 5; ++k) {
        long kind;
        if (!int_of(a[7 + 2 * k], &kind) || (k == 0 && kind <= 0)) return not_plain();
        if (!slot_of(a[6 + 2 * k], kind, dim, &s[k])) return not_plain();
    }
    void *stream = nullptr;
    if (!dtype_of(a[6], &t.dtype) || !points_of(a[4], a[6], &t.n) || !stream_of(a[5], &stream)) return not_plain();
    t.in0 = s[0].ptr, t.ld_in0 = s[0].ld;
    t.in1 = s[1].ptr, t.ld_in1 = s[1].ld;
    t.out0 = s[2].ptr, t.ld_out0 = s[2].ld;
    t.out1 = s[3].ptr, t.ld_out1 = s[3].ld;
    t.out2 = s[4].ptr, t.ld_out2 = s[4].ld;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_task_run(&t, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// char_apply(dim, dir, mode, gamma, n, stream, U, X, Y)
PyObject *char_apply(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    HANDLE_TH_ERRORS
    if (na != 9 || !g_char_apply) return not_plain();
    long dim, dir, mode;
    double gamma;
    if (!int_of(a[0], &dim) || !int_of(a[1], &dir) || !int_of(a[2], &mode) || !double_of(a[3], &gamma)) return not_plain();
    Slot s[3];
    for (int k = 0; k < 3; ++k)
        if (dim + 2 <= 0 || !slot_of(a[6 + k], dim + 2, dim, &s[k])) return not_plain();
    int32_t dtype;
    int64_t n;
    void *stream = nullptr;
    if (!dtype_of(a[6], &dtype) || !points_of(a[4], a[6], &n) || !stream_of(a[5], &stream)) return not_plain();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_char_apply((int)dim, (int)dir, (int)mode, gamma, dtype, s[0].ptr, s[0].ld, s[1].ptr, s[1].ld, s[2].ptr,
                      s[2].ld, n, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// viscous_flux(dim, mu, kappa, n, stream, U, G, gradT, Fv)
PyObject *viscous_flux(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    HANDLE_TH_ERRORS
    if (na != 9 || !g_viscous_flux) return not_plain();
    long dim;
    double mu, kappa;
    if (!int_of(a[0], &dim) || !double_of(a[1], &mu) || !double_of(a[2], &kappa)) return not_plain();
    const long kind[4] = {dim + 2, dim * dim, dim, (dim + 2) * dim};
    Slot s[4];
    for (int k = 0; k < 4; ++k)
        if (kind[k] <= 0 || !slot_of(a[5 + k], kind[k], dim, &s[k])) return not_plain();
    int32_t dtype;
    int64_t n;
    void *stream = nullptr;
    if (!dtype_of(a[5], &dtype) || !points_of(a[3], a[5], &n) || !stream_of(a[4], &stream)) return not_plain();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_viscous_flux((int)dim, mu, kappa, dtype, s[0].ptr, s[0].ld, s[1].ptr, s[1].ld, s[2].ptr, s[2].ld,
                        s[3].ptr, s[3].ld, n, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// Uninitialised values of `shape`, whose second dimension is padded, for u's
// points, on its device and of its type.  Other Python threads run meanwhile: an allocation that has to
// give cached blocks back waits for the device.
at::Tensor empty_like_points(at::DimVector shape, const at::Tensor &u)
{
    struct NoGil {
        PyThreadState *state = PyEval_SaveThread();
        ~NoGil() { PyEval_RestoreThread(state); }
    } no_gil;
    return at::empty(shape, u.options()).narrow(1, 0, u.size(1));
}

int64_t padded(int64_t n) { return std::max<int64_t>(64, (n + 63) / 64 * 64); }

// empty_fields(fields, U): uninitialised rows for U's points, of its type and
// on its device, padded as fdbb.empty_fields pads them
PyObject *empty_fields(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    HANDLE_TH_ERRORS
    if (na != 2) return not_plain();
    long fields;
    if (!int_of(a[0], &fields) || fields < 0) return not_plain();
    const at::Tensor *u = plain(a[1]);
    if (!u || u->dim() != 2) return not_plain();
    return THPVariable_Wrap(empty_like_points({fields, padded(u->size(1))}, *u));
    END_HANDLE_TH_ERRORS
}

// empty_blocks(dim, U): K x K blocks for U's points
PyObject *empty_blocks(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    HANDLE_TH_ERRORS
    if (na != 2) return not_plain();
    long dim;
    if (!int_of(a[0], &dim) || dim < 0) return not_plain();
    const at::Tensor *u = plain(a[1]);
    if (!u || u->dim() != 2) return not_plain();
    const int64_t K = dim + 2;
    return THPVariable_Wrap(empty_like_points({dim, padded(u->size(1)), K, K}, *u));
    END_HANDLE_TH_ERRORS
}

// bind(task_run, char_apply, viscous_flux, raw_stream): the loaded library's
// entry points, as addresses
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    if (na != 4) {
        PyErr_SetString(PyExc_TypeError, "bind takes four arguments");
        return nullptr;
    }
    void *f[3];
    for (int k = 0; k < 3; ++k) {
        f[k] = PyLong_AsVoidPtr(a[k]);
        if (PyErr_Occurred()) return nullptr;
    }
    g_task_run = reinterpret_cast<decltype(g_task_run)>(f[0]);
    g_char_apply = reinterpret_cast<decltype(g_char_apply)>(f[1]);
    g_viscous_flux = reinterpret_cast<decltype(g_viscous_flux)>(f[2]);
    Py_INCREF(a[3]);
    Py_XSETREF(g_raw_stream, a[3]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(run),          METHOD(char_apply),   METHOD(viscous_flux), METHOD(empty_fields),
                         METHOD(empty_blocks), METHOD(bind),         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
