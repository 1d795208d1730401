// The Python binding's call path: one built-in function per entry point of include/mxc.h that takes the same arguments
// as the Python definitions it stands for, reads pointers and sizes straight from the tensors, takes the current stream
// and calls the C ABI.  What bounds a small layer's step is the host: marshalled by ctypes, with the stream looked up
// through torch.cuda, a call cost 5 us before the library saw it (a launch is 2 us); this way it is about 0.5 us.
#include <Python.h>

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mxc.h"

namespace {

PyObject *g_error = nullptr;            // MxcError
PyObject *g_raw_stream = nullptr;       // torch._C._cuda_getCurrentRawStream
PyObject *g_device = nullptr;           // torch._C._cuda_getDevice
PyObject *g_slow_stream = nullptr;      // () -> int, for a stream when the two above are not to be had

constexpr int MAX_ARGS = 20;

// Positional and keyword arguments in the order of `names`; the ones from `required` on default to nullptr (None).
struct Args {
    PyObject *v[MAX_ARGS] = {};
    bool ok = false;
    Args(const char *fn, const char *const *names, int n, int required, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
    {
        if (nargs > n) {
            PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", fn, n, nargs);
            return;
        }
        for (Py_ssize_t i = 0; i < nargs; ++i) v[i] = args[i];
        const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
        for (Py_ssize_t k = 0; k < nkw; ++k) {
            PyObject *name = PyTuple_GET_ITEM(kwnames, k);
            int at = 0;
            while (at < n && PyUnicode_CompareWithASCIIString(name, names[at]) != 0) ++at;
            if (at == n || v[at] != nullptr) {
                PyErr_Format(PyExc_TypeError, at == n ? "%s() got an unexpected keyword argument '%U'" : "%s() got multiple values for argument '%U'", fn, name);
                return;
            }
            v[at] = args[nargs + k];
        }
        for (int i = 0; i < required; ++i)
            if (v[i] == nullptr) {
                PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", fn, names[i]);
                return;
            }
        ok = true;
    }
};

bool to_int(PyObject *o, int *out)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) return false;
    *out = (int)v;
    return true;
}

bool to_ints(PyObject *const *o, int *out, int n)
{
    for (int i = 0; i < n; ++i)
        if (!to_int(o[i], out + i)) return false;
    return true;
}

// device pointer (and size) of a contiguous GPU tensor; None: null
bool to_ptr(PyObject *o, void **ptr, size_t *bytes = nullptr)
{
    *ptr = nullptr;
    if (bytes) *bytes = 0;
    if (o == nullptr || o == Py_None) return true;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %s", Py_TYPE(o)->tp_name);
        return false;
    }
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "tensors must be contiguous GPU tensors");
        return false;
    }
    *ptr = t.data_ptr();
    if (bytes) *bytes = t.nbytes();
    return true;
}

bool to_stream(PyObject *o, void **stream)
{
    PyObject *n;
    if (o == nullptr || o == Py_None) {
        PyObject *dev = g_device ? PyObject_CallNoArgs(g_device) : nullptr;
        n = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
        Py_XDECREF(dev);
        if (n == nullptr) {
            PyErr_Clear();
            n = PyObject_CallNoArgs(g_slow_stream);
        }
    } else if (PyLong_Check(o)) {
        n = Py_NewRef(o);
    } else {
        n = PyObject_GetAttrString(o, "cuda_stream");
        if (n == nullptr) {
            PyErr_Clear();
            n = PyNumber_Long(o);
        }
    }
    if (n == nullptr) return false;
    *stream = (void *)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}

// the interpreter runs on while a call enqueues its work; an exception, too, takes the lock back before Python sees it
struct WithoutGil {
    PyThreadState *ts = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(ts); }
};

PyObject *done(int rc)
{
    if (rc == MXC_OK) Py_RETURN_NONE;
    PyObject *e = g_error ? PyObject_CallFunction(g_error, "i", rc) : nullptr;
    if (e != nullptr) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred())
        PyErr_Format(PyExc_RuntimeError, "mxc status %d", rc);
    return nullptr;
}

#define DIMS "N", "C", "H", "W", "K", "R", "S", "stride", "pad", "dtype", "layout"
#define D11 d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], d[8], d[9], d[10]
// Declares the wrapper FN with its argument names (the first REQ required), runs BODY with `a` (Args) and returns its rc.
// torch's accessors throw C++ exceptions (data_ptr() of a tensor without storage, as torch.func.vmap and torch.func.grad hand
// out): they become Python exceptions here, for nothing may unwind through the interpreter's C frames.
#define WRAP(FN, REQ, NAMES, ...)                                                                                      \
    PyObject *py_##FN(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kw)                                \
    {                                                                                                                   \
        HANDLE_TH_ERRORS                                                                                                \
        static const char *const names[] = NAMES;                                                                      \
        constexpr int n = (int)(sizeof(names) / sizeof(names[0]));                                                      \
        static_assert(n <= MAX_ARGS, "arguments");                                                                      \
        Args a(#FN, names, n, REQ, args, nargs, kw);                                                                    \
        if (!a.ok) return nullptr;                                                                                      \
        int rc = MXC_OK;                                                                                                \
        __VA_ARGS__                                                                                                     \
        return done(rc);                                                                                                \
        END_HANDLE_TH_ERRORS                                                                                            \
    }
#define N_(...) {__VA_ARGS__}
#define RUN(EXPR) do { WithoutGil off; rc = EXPR; } while (0)
#define INTS(COUNT) int d[COUNT]; if (!to_ints(a.v, d, COUNT)) return nullptr
#define PTR(NAME, AT) void *NAME; if (!to_ptr(a.v[AT], &NAME)) return nullptr
#define BUF(NAME, AT) void *NAME; size_t NAME##_n; if (!to_ptr(a.v[AT], &NAME, &NAME##_n)) return nullptr
#define STREAM(AT) void *st; if (!to_stream(a.v[AT], &st)) return nullptr
#define INT(NAME, AT) int NAME; if (!to_int(a.v[AT], &NAME)) return nullptr
#define BOOL(NAME, AT) const int NAME##_t = PyObject_IsTrue(a.v[AT]); int NAME = 0; if (NAME##_t < 0) return nullptr; \
    if (PyLong_Check(a.v[AT])) { if (!to_int(a.v[AT], &NAME)) return nullptr; } else NAME = NAME##_t
#define FLOAT(NAME, AT) const double NAME = PyFloat_AsDouble(a.v[AT]); if (NAME == -1.0 && PyErr_Occurred()) return nullptr

#define CONV3(FN, A, B, O)                                                                                              \
    WRAP(FN, 14, N_(DIMS, A, B, O, "workspace", "stream"),                                                              \
         INTS(11); PTR(x, 11); PTR(w, 12); PTR(y, 13); BUF(ws, 14); STREAM(15); RUN(FN(D11, x, w, y, ws, ws_n, st));)
CONV3(mxc_conv2d_fwd, "x", "w", "y")
CONV3(mxc_conv2d_bwd_data, "dy", "w", "dx")
CONV3(mxc_conv2d_bwd_weight, "x", "dy", "dw")
CONV3(mxc_conv2d_bwd_weight_bf16, "x", "dy", "dw")

WRAP(mxc_conv2d_bwd_weight_static, 14, N_(DIMS, "x", "dy", "dw", "stream"),
     INTS(11); PTR(x, 11); PTR(dy, 12); PTR(dw, 13); STREAM(14); RUN(mxc_conv2d_bwd_weight_static(D11, x, dy, dw, st));)
WRAP(mxc_conv2d_fwd_bias_act, 16, N_(DIMS, "x", "w", "bias", "relu", "y", "workspace", "stream"),
     INTS(11); PTR(x, 11); PTR(w, 12); PTR(bias, 13); BOOL(relu, 14); PTR(y, 15); BUF(ws, 16); STREAM(17);
     RUN(mxc_conv2d_fwd_bias_act(D11, x, w, (const float *)bias, relu, y, ws, ws_n, st));)
WRAP(mxc_conv2d_bwd_data_relu, 15, N_(DIMS, "dy", "w", "x", "dx", "workspace", "stream"),
     INTS(11); PTR(dy, 11); PTR(w, 12); PTR(x, 13); PTR(dx, 14); BUF(ws, 15); STREAM(16);
     RUN(mxc_conv2d_bwd_data_relu(D11, dy, w, x, dx, ws, ws_n, st));)
WRAP(mxc_conv2d_bwd_data_prepare_filter, 13, N_(DIMS, "w", "w_prepared", "stream"),
     INTS(11); PTR(w, 11); BUF(wp, 12); STREAM(13); RUN(mxc_conv2d_bwd_data_prepare_filter(D11, w, wp, wp_n, st));)
WRAP(mxc_conv2d_bwd_data_prepared, 15, N_(DIMS, "dy", "w_prepared", "x_mask", "dx", "workspace", "stream"),
     INTS(11); PTR(dy, 11); BUF(wp, 12); PTR(mask, 13); PTR(dx, 14); BUF(ws, 15); STREAM(16);
     RUN(mxc_conv2d_bwd_data_prepared(D11, dy, wp, wp_n, mask, dx, ws, ws_n, st));)
WRAP(mxc_conv2d_fwd_transform, 16, N_(DIMS, "x", "w", "bias", "relu", "y", "workspace", "stream"),
     INTS(11); PTR(x, 11); PTR(w, 12); PTR(bias, 13); BOOL(relu, 14); PTR(y, 15); BUF(ws, 16); STREAM(17);
     RUN(mxc_conv2d_fwd_transform(D11, x, w, (const float *)bias, relu, y, ws, ws_n, st));)
WRAP(mxc_conv2d_prepare_input, 13, N_(DIMS, "x", "x_prepared", "stream"),
     INTS(11); PTR(x, 11); BUF(xp, 12); STREAM(13); RUN(mxc_conv2d_prepare_input(D11, x, xp, xp_n, st));)
WRAP(mxc_conv2d_fwd_prepared_input, 16, N_(DIMS, "x_prepared", "w", "bias", "relu", "y", "workspace", "stream"),
     INTS(11); BUF(xp, 11); PTR(w, 12); PTR(bias, 13); BOOL(relu, 14); PTR(y, 15); BUF(ws, 16); STREAM(17);
     RUN(mxc_conv2d_fwd_prepared_input(D11, xp, xp_n, w, (const float *)bias, relu, y, ws, ws_n, st));)
WRAP(mxc_conv2d_bwd_weight_prepared_input, 15, N_(DIMS, "x_prepared", "dy", "dw", "dw_dtype", "workspace", "stream"),
     INTS(11); BUF(xp, 11); PTR(dy, 12); PTR(dw, 13); INT(dw_dtype, 14); BUF(ws, 15); STREAM(16);
     RUN(mxc_conv2d_bwd_weight_prepared_input(D11, xp, xp_n, dy, dw, dw_dtype, ws, ws_n, st));)
WRAP(mxc_bias_grad, 8, N_("N", "K", "P", "Q", "dtype", "layout", "dy", "db", "workspace", "stream"),
     INTS(6); PTR(dy, 6); PTR(db, 7); BUF(ws, 8); STREAM(9);
     RUN(mxc_bias_grad(d[0], d[1], d[2], d[3], d[4], d[5], dy, (float *)db, ws, ws_n, st));)
WRAP(mxc_fc_fwd, 9, N_("N", "C", "K", "dtype", "x", "w", "bias", "relu", "y", "workspace", "stream"),
     INTS(4); PTR(x, 4); PTR(w, 5); PTR(bias, 6); BOOL(relu, 7); PTR(y, 8); BUF(ws, 9); STREAM(10);
     RUN(mxc_fc_fwd(d[0], d[1], d[2], d[3], x, w, (const float *)bias, relu, y, ws, ws_n, st));)
WRAP(mxc_fc_bwd_data, 8, N_("N", "C", "K", "dtype", "dy", "w", "x_mask", "dx", "workspace", "stream"),
     INTS(4); PTR(dy, 4); PTR(w, 5); PTR(mask, 6); PTR(dx, 7); BUF(ws, 8); STREAM(9);
     RUN(mxc_fc_bwd_data(d[0], d[1], d[2], d[3], dy, w, mask, dx, ws, ws_n, st));)
WRAP(mxc_fc_bwd_weight, 7, N_("N", "C", "K", "dtype", "x", "dy", "dw", "workspace", "stream"),
     INTS(4); PTR(x, 4); PTR(dy, 5); PTR(dw, 6); BUF(ws, 7); STREAM(8);
     RUN(mxc_fc_bwd_weight(d[0], d[1], d[2], d[3], x, dy, dw, ws, ws_n, st));)
WRAP(mxc_softmax_fwd, 5, N_("N", "K", "dtype", "z", "p", "stream"),
     INTS(3); PTR(z, 3); PTR(p, 4); STREAM(5); RUN(mxc_softmax_fwd(d[0], d[1], d[2], z, p, st));)
WRAP(mxc_softmax_xent_bwd, 7, N_("N", "K", "dtype", "p", "labels", "scale", "dz", "stream"),
     INTS(3); PTR(p, 3); PTR(labels, 4); FLOAT(scale, 5); PTR(dz, 6); STREAM(7);
     RUN(mxc_softmax_xent_bwd(d[0], d[1], d[2], p, (const int *)labels, (float)scale, dz, st));)
WRAP(mxc_sgd_update, 7, N_("w", "g", "v", "w_bf16", "lr", "momentum", "wd", "stream"),
     BUF(w, 0); PTR(g, 1); PTR(v, 2); PTR(wb, 3); FLOAT(lr, 4); FLOAT(mom, 5); FLOAT(wd, 6); STREAM(7);
     // the element count is w's, whatever its type
     const size_t count = a.v[0] == Py_None ? 0 : (size_t)THPVariable_Unpack(a.v[0]).numel();
     RUN(mxc_sgd_update(count, (float *)w, (const float *)g, (float *)v, wb, (float)lr, (float)mom, (float)wd, st));)
WRAP(mxc_layout_convert, 9, N_("n", "c", "h", "w", "dtype", "src_layout", "dst_layout", "src", "dst", "stream"),
     INTS(7); PTR(src, 7); PTR(dst, 8); STREAM(9);
     RUN(mxc_layout_convert(d[0], d[1], d[2], d[3], d[4], d[5], d[6], src, dst, st));)

PyObject *py_mxc_conv2d_workspace_bytes(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kw)
{
    HANDLE_TH_ERRORS
    static const char *const names[] = {"op", DIMS};
    Args a("mxc_conv2d_workspace_bytes", names, 12, 12, args, nargs, kw);
    if (!a.ok) return nullptr;
    int d[12];
    if (!to_ints(a.v, d, 12)) return nullptr;
    size_t bytes = 0;
    const int rc = mxc_conv2d_workspace_bytes(d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], d[8], d[9], d[10], d[11], &bytes);
    return rc == MXC_OK ? PyLong_FromSize_t(bytes) : done(rc);
    END_HANDLE_TH_ERRORS
}

// set_hooks(MxcError, raw_stream, device, slow_stream)
PyObject *py_set_hooks(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 4) {
        PyErr_SetString(PyExc_TypeError, "set_hooks takes 4 arguments");
        return nullptr;
    }
    PyObject **to[4] = {&g_error, &g_raw_stream, &g_device, &g_slow_stream};
    for (int i = 0; i < 4; ++i) {
        PyObject *old = *to[i];
        *to[i] = args[i] == Py_None ? nullptr : Py_NewRef(args[i]);
        Py_XDECREF(old);
    }
    if (g_raw_stream == nullptr) Py_CLEAR(g_device);
    Py_RETURN_NONE;
}

#define ENTRY(FN) {#FN, (PyCFunction)(void *)py_##FN, METH_FASTCALL | METH_KEYWORDS, nullptr}
PyMethodDef methods[] = {
    ENTRY(mxc_conv2d_fwd), ENTRY(mxc_conv2d_bwd_data), ENTRY(mxc_conv2d_bwd_weight), ENTRY(mxc_conv2d_bwd_weight_bf16),
    ENTRY(mxc_conv2d_bwd_weight_static), ENTRY(mxc_conv2d_fwd_bias_act), ENTRY(mxc_conv2d_bwd_data_relu),
    ENTRY(mxc_conv2d_bwd_data_prepare_filter), ENTRY(mxc_conv2d_bwd_data_prepared), ENTRY(mxc_conv2d_fwd_transform),
    ENTRY(mxc_conv2d_prepare_input), ENTRY(mxc_conv2d_fwd_prepared_input), ENTRY(mxc_conv2d_bwd_weight_prepared_input),
    ENTRY(mxc_bias_grad), ENTRY(mxc_fc_fwd), ENTRY(mxc_fc_bwd_data), ENTRY(mxc_fc_bwd_weight), ENTRY(mxc_softmax_fwd),
    ENTRY(mxc_softmax_xent_bwd), ENTRY(mxc_sgd_update), ENTRY(mxc_layout_convert), ENTRY(mxc_conv2d_workspace_bytes),
    {"set_hooks", (PyCFunction)(void *)py_set_hooks, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Call path of the mxc binding", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
