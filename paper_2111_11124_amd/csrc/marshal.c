/*
 * marshal.c -- the binding's argument marshalling as a CPython extension: the ordinary form of every compute call, straight
 * from the Python objects to the C entry point.
 *
 * A small kernel is launched in 2 to 3 us, and marshalling a call in Python (four to eight tensors at half a microsecond
 * each, a ctypes structure, the current stream, the foreign call itself) took another 6 to 8 us of the host: a Transformer
 * block's thirty-two calls took 340 us whatever its size.
 *
 * A function here returns the call's status, or None when an argument is not of the form it knows (another type, a tensor
 * on the host or not contiguous, a type mismatch): nothing has been called then, and the Python function goes through
 * ctypes as ever, raising what it raises.  Nothing is kept from one call for the next but the interned names and the
 * type objects looked up when the module is loaded.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include "mesa.h"

static PyObject *n_is_cuda, *n_is_contiguous, *n_data_ptr, *n_dtype, *n_numel, *n_element_size;
static PyObject *t_f16, *t_f32, *t_bf16;          /* torch.float16, torch.float32, torch.bfloat16 */
static PyObject *conv_type;                       /* the binding's Conv2d structure */
static PyObject *get_device, *get_raw_stream;     /* torch._C._cuda_getDevice, _cuda_getCurrentRawStream */

struct call {
    PyObject *const *args;
    int ok;
};

static struct call begin(PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want)
{
    struct call c = {args, nargs == want};
    return c;
}

static PyObject *leave(void)
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

/* an attribute or method result that is a truth value: 1, 0, or -1 on an error */
static int truth(PyObject *v)
{
    if (!v) return -1;
    const int r = v == Py_True ? 1 : v == Py_False ? 0 : -1;
    Py_DECREF(v);
    return r;
}

static void *take_ptr(struct call *c, int i)
{
    if (!c->ok || c->args[i] == Py_None) return NULL;
    PyObject *t = c->args[i];
    if (truth(PyObject_GetAttr(t, n_is_cuda)) != 1 || truth(PyObject_CallMethodNoArgs(t, n_is_contiguous)) != 1) { c->ok = 0; return NULL; }
    PyObject *p = PyObject_CallMethodNoArgs(t, n_data_ptr);
    if (!p || !PyLong_Check(p)) { Py_XDECREF(p); c->ok = 0; return NULL; }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return (void *)(uintptr_t)v;
}

static size_t take_size(struct call *c, PyObject *t, PyObject *method)
{
    PyObject *p = c->ok ? PyObject_CallMethodNoArgs(t, method) : NULL;
    if (!p || !PyLong_Check(p)) { Py_XDECREF(p); c->ok = 0; return 0; }
    const size_t v = PyLong_AsSize_t(p);
    Py_DECREF(p);
    return v;
}

static void *take_ws(struct call *c, int i, size_t *bytes)
{
    *bytes = 0;
    void *p = take_ptr(c, i);
    if (c->ok && c->args[i] != Py_None) *bytes = take_size(c, c->args[i], n_numel) * take_size(c, c->args[i], n_element_size);
    return p;
}

static mesa_dtype take_dtype(struct call *c, int i)
{
    if (!c->ok || c->args[i] == Py_None) { c->ok = 0; return MESA_F32; }
    PyObject *d = PyObject_GetAttr(c->args[i], n_dtype);
    Py_XDECREF(d);                                /* torch's types live as long as torch */
    if (d == t_f16) return MESA_F16;
    if (d == t_bf16) return MESA_BF16;
    if (d != t_f32) c->ok = 0;
    return MESA_F32;
}

static void same_dtype(struct call *c, int i, int j)
{
    if (!c->ok || c->args[i] == Py_None || c->args[j] == Py_None) { c->ok = 0; return; }
    PyObject *a = PyObject_GetAttr(c->args[i], n_dtype), *b = PyObject_GetAttr(c->args[j], n_dtype);
    if (!a || a != b) c->ok = 0;
    Py_XDECREF(a);
    Py_XDECREF(b);
}

static uint64_t int_of(struct call *c, PyObject *v)
{
    if (!c->ok || !PyLong_Check(v)) { c->ok = 0; return 0; }
    return PyLong_AsUnsignedLongLongMask(v);      /* as ctypes does: the low 64 bits */
}
static uint64_t take_int(struct call *c, int i) { return c->ok ? int_of(c, c->args[i]) : 0; }

static float take_float(struct call *c, int i)
{
    if (!c->ok) return 0.0f;
    PyObject *v = c->args[i];
    if (PyFloat_Check(v)) return (float)PyFloat_AS_DOUBLE(v);
    if (PyLong_Check(v)) {
        const double d = PyLong_AsDouble(v);
        if (!(d == -1.0 && PyErr_Occurred())) return (float)d;
    }
    c->ok = 0;
    return 0.0f;
}

static int take_bool(struct call *c, int i)
{
    if (!c->ok) return 0;
    const int r = PyObject_IsTrue(c->args[i]);
    if (r < 0) c->ok = 0;
    return r > 0;
}

static mesa_layout take_layout(struct call *c, int i)
{
    mesa_layout L = {0, 0, 0};
    if (!c->ok) return L;
    PyObject *v = c->args[i];
    if (!(PyTuple_CheckExact(v) || PyList_CheckExact(v)) || PySequence_Fast_GET_SIZE(v) != 3) { c->ok = 0; return L; }
    PyObject **e = PySequence_Fast_ITEMS(v);
    L.outer = (int64_t)int_of(c, e[0]);
    L.groups = (int64_t)int_of(c, e[1]);
    L.inner = (int64_t)int_of(c, e[2]);
    return L;
}

static mesa_conv2d take_conv(struct call *c, int i)
{
    mesa_conv2d cv;
    memset(&cv, 0, sizeof cv);
    Py_buffer b;
    if (!c->ok) return cv;
    if ((PyObject *)Py_TYPE(c->args[i]) != conv_type || PyObject_GetBuffer(c->args[i], &b, PyBUF_SIMPLE) != 0) { c->ok = 0; return cv; }
    if (b.len == (Py_ssize_t)sizeof cv) memcpy(&cv, b.buf, sizeof cv);
    else c->ok = 0;
    PyBuffer_Release(&b);
    return cv;
}

/* torch.cuda.current_stream().cuda_stream: the current stream of the current device */
static void *take_stream(struct call *c)
{
    if (!c->ok) return NULL;
    PyObject *dev = PyObject_CallNoArgs(get_device);
    PyObject *s = dev ? PyObject_CallOneArg(get_raw_stream, dev) : NULL;
    Py_XDECREF(dev);
    if (!s || !PyLong_Check(s)) { Py_XDECREF(s); c->ok = 0; return NULL; }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(s);
    Py_DECREF(s);
    return (void *)(uintptr_t)v;
}

#define ENTRY(name, n) static PyObject *py_##name(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
#define RUN(c, expr) \
    do { \
        void *stream = take_stream(&c); \
        if (!c.ok || PyErr_Occurred()) return leave(); \
        int status; \
        Py_BEGIN_ALLOW_THREADS status = (int)(expr); \
        Py_END_ALLOW_THREADS return PyLong_FromLong(status); \
    } while (0)

ENTRY(update_running_params, 7)
{
    struct call c = begin(args, nargs, 7);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    const int first_call = take_bool(&c, 5);
    size_t ws_bytes;
    void *ws = take_ws(&c, 6, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_update_running_params(x, dt, layout, alpha, beta, lam, first_call, ws, ws_bytes, stream));
}

ENTRY(update_running_params_sym, 7)
{
    struct call c = begin(args, nargs, 7);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    const int first_call = take_bool(&c, 5);
    size_t ws_bytes;
    void *ws = take_ws(&c, 6, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_update_running_params_sym(x, dt, layout, alpha, beta, lam, first_call, ws, ws_bytes, stream));
}

ENTRY(update_running_params_fixed_beta, 8)
{
    struct call c = begin(args, nargs, 8);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    const int first_call = take_bool(&c, 5);
    const float beta_fixed = take_float(&c, 6);
    size_t ws_bytes;
    void *ws = take_ws(&c, 7, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_update_running_params_fixed_beta(x, dt, layout, alpha, beta, lam, first_call, beta_fixed, ws, ws_bytes, stream));
}

ENTRY(update_running_params_static, 6)
{
    struct call c = begin(args, nargs, 6);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    const int first_call = take_bool(&c, 5);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_update_running_params_static(x, dt, layout, alpha, beta, lam, first_call, stream));
}

ENTRY(update_running_scale_sym, 6)
{
    struct call c = begin(args, nargs, 6);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *m = take_ptr(&c, 2);
    const float lam = take_float(&c, 3);
    const int first_call = take_bool(&c, 4);
    size_t ws_bytes;
    void *ws = take_ws(&c, 5, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_update_running_scale_sym(x, dt, layout, m, lam, first_call, ws, ws_bytes, stream));
}

ENTRY(quantize_headwise, 8)
{
    struct call c = begin(args, nargs, 8);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *q = take_ptr(&c, 4);
    const int mode = (int)take_int(&c, 5);
    const uint64_t seed = take_int(&c, 6);
    const uint64_t offset = take_int(&c, 7);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_quantize_headwise(x, dt, layout, alpha, beta, q, mode, seed, offset, stream));
}

ENTRY(quantize_headwise_b4, 8)
{
    struct call c = begin(args, nargs, 8);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *q4 = take_ptr(&c, 4);
    const int mode = (int)take_int(&c, 5);
    const uint64_t seed = take_int(&c, 6);
    const uint64_t offset = take_int(&c, 7);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_quantize_headwise_b4(x, dt, layout, alpha, beta, q4, mode, seed, offset, stream));
}

ENTRY(quantize_sym, 7)
{
    struct call c = begin(args, nargs, 7);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *m = take_ptr(&c, 2);
    void *q = take_ptr(&c, 3);
    const int mode = (int)take_int(&c, 4);
    const uint64_t seed = take_int(&c, 5);
    const uint64_t offset = take_int(&c, 6);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_quantize_sym(x, dt, layout, m, q, mode, seed, offset, stream));
}

ENTRY(quantize_update_fused, 10)
{
    struct call c = begin(args, nargs, 10);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    void *q = take_ptr(&c, 5);
    size_t ws_bytes;
    void *ws = take_ws(&c, 6, &ws_bytes);
    const int mode = (int)take_int(&c, 7);
    const uint64_t seed = take_int(&c, 8);
    const uint64_t offset = take_int(&c, 9);
    const mesa_dtype dt = take_dtype(&c, 0);
    RUN(c, mesa_quantize_update_fused(x, dt, layout, alpha, beta, lam, q, mode, seed, offset, ws, ws_bytes, stream));
}

ENTRY(gelu_fwd_q, 11)
{
    struct call c = begin(args, nargs, 11);
    void *x = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    const float lam = take_float(&c, 4);
    void *y = take_ptr(&c, 5);
    void *q = take_ptr(&c, 6);
    size_t ws_bytes;
    void *ws = take_ws(&c, 7, &ws_bytes);
    const int mode = (int)take_int(&c, 8);
    const uint64_t seed = take_int(&c, 9);
    const uint64_t offset = take_int(&c, 10);
    const mesa_dtype dt = take_dtype(&c, 0);
    same_dtype(&c, 5, 0);
    RUN(c, mesa_gelu_fwd_q(x, dt, layout, alpha, beta, lam, y, q, mode, seed, offset, ws, ws_bytes, stream));
}

ENTRY(softmax_fwd_q, 14)
{
    struct call c = begin(args, nargs, 14);
    void *s = take_ptr(&c, 0);
    const int64_t B = (int64_t)take_int(&c, 1);
    const int64_t H = (int64_t)take_int(&c, 2);
    const int64_t rows = (int64_t)take_int(&c, 3);
    const int64_t cols = (int64_t)take_int(&c, 4);
    void *alpha = take_ptr(&c, 5);
    void *beta = take_ptr(&c, 6);
    const float lam = take_float(&c, 7);
    void *y = take_ptr(&c, 8);
    void *q = take_ptr(&c, 9);
    size_t ws_bytes;
    void *ws = take_ws(&c, 10, &ws_bytes);
    const int mode = (int)take_int(&c, 11);
    const uint64_t seed = take_int(&c, 12);
    const uint64_t offset = take_int(&c, 13);
    const mesa_dtype dt = take_dtype(&c, 0);
    same_dtype(&c, 8, 0);
    RUN(c, mesa_softmax_fwd_q(s, B, H, rows, cols, alpha, beta, lam, y, q, mode, seed, offset, ws, ws_bytes, dt, stream));
}

ENTRY(layernorm_fwd_q, 18)
{
    struct call c = begin(args, nargs, 18);
    void *x = take_ptr(&c, 0);
    const int64_t M = (int64_t)take_int(&c, 1);
    const int64_t D = (int64_t)take_int(&c, 2);
    const int64_t G = (int64_t)take_int(&c, 3);
    void *gamma = take_ptr(&c, 4);
    void *bias = take_ptr(&c, 5);
    const float eps = take_float(&c, 6);
    void *alpha = take_ptr(&c, 7);
    void *beta = take_ptr(&c, 8);
    const float lam = take_float(&c, 9);
    void *y = take_ptr(&c, 10);
    void *mean = take_ptr(&c, 11);
    void *rstd = take_ptr(&c, 12);
    void *q = take_ptr(&c, 13);
    size_t ws_bytes;
    void *ws = take_ws(&c, 14, &ws_bytes);
    const int mode = (int)take_int(&c, 15);
    const uint64_t seed = take_int(&c, 16);
    const uint64_t offset = take_int(&c, 17);
    const mesa_dtype dt = take_dtype(&c, 0);
    same_dtype(&c, 4, 0);
    same_dtype(&c, 5, 0);
    same_dtype(&c, 10, 0);
    RUN(c, mesa_layernorm_fwd_q(x, M, D, G, gamma, bias, eps, alpha, beta, lam, y, mean, rstd, q, mode, seed, offset, ws, ws_bytes, dt, stream));
}

ENTRY(dequantize, 5)
{
    struct call c = begin(args, nargs, 5);
    void *q = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *x_hat = take_ptr(&c, 4);
    const mesa_dtype dt = take_dtype(&c, 4);
    RUN(c, mesa_dequantize(q, layout, alpha, beta, x_hat, dt, stream));
}

ENTRY(dequantize_b4, 5)
{
    struct call c = begin(args, nargs, 5);
    void *q4 = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *x_hat = take_ptr(&c, 4);
    const mesa_dtype dt = take_dtype(&c, 4);
    RUN(c, mesa_dequantize_b4(q4, layout, alpha, beta, x_hat, dt, stream));
}

ENTRY(dequantize_sym, 4)
{
    struct call c = begin(args, nargs, 4);
    void *q = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *m = take_ptr(&c, 2);
    void *x_hat = take_ptr(&c, 3);
    const mesa_dtype dt = take_dtype(&c, 3);
    RUN(c, mesa_dequantize_sym(q, layout, m, x_hat, dt, stream));
}

ENTRY(gelu_bwd_q, 6)
{
    struct call c = begin(args, nargs, 6);
    void *xq = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *dy = take_ptr(&c, 4);
    void *dx = take_ptr(&c, 5);
    const mesa_dtype dt = take_dtype(&c, 4);
    same_dtype(&c, 5, 4);
    RUN(c, mesa_gelu_bwd_q(xq, layout, alpha, beta, dy, dx, dt, stream));
}

ENTRY(gelu_bwd_q_b4, 6)
{
    struct call c = begin(args, nargs, 6);
    void *q4 = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *dy = take_ptr(&c, 4);
    void *dx = take_ptr(&c, 5);
    const mesa_dtype dt = take_dtype(&c, 4);
    same_dtype(&c, 5, 4);
    RUN(c, mesa_gelu_bwd_q_b4(q4, layout, alpha, beta, dy, dx, dt, stream));
}

ENTRY(relu_bwd_q, 6)
{
    struct call c = begin(args, nargs, 6);
    void *xq = take_ptr(&c, 0);
    const mesa_layout layout = take_layout(&c, 1);
    void *alpha = take_ptr(&c, 2);
    void *beta = take_ptr(&c, 3);
    void *dy = take_ptr(&c, 4);
    void *dx = take_ptr(&c, 5);
    const mesa_dtype dt = take_dtype(&c, 4);
    same_dtype(&c, 5, 4);
    RUN(c, mesa_relu_bwd_q(xq, layout, alpha, beta, dy, dx, dt, stream));
}

ENTRY(softmax_bwd_q, 9)
{
    struct call c = begin(args, nargs, 9);
    void *yq = take_ptr(&c, 0);
    const int64_t B = (int64_t)take_int(&c, 1);
    const int64_t H = (int64_t)take_int(&c, 2);
    const int64_t rows = (int64_t)take_int(&c, 3);
    const int64_t cols = (int64_t)take_int(&c, 4);
    void *alpha = take_ptr(&c, 5);
    void *beta = take_ptr(&c, 6);
    void *dy = take_ptr(&c, 7);
    void *dx = take_ptr(&c, 8);
    const mesa_dtype dt = take_dtype(&c, 7);
    same_dtype(&c, 8, 7);
    RUN(c, mesa_softmax_bwd_q(yq, B, H, rows, cols, alpha, beta, dy, dx, dt, stream));
}

ENTRY(layernorm_bwd_q, 14)
{
    struct call c = begin(args, nargs, 14);
    void *xq = take_ptr(&c, 0);
    const int64_t M = (int64_t)take_int(&c, 1);
    const int64_t D = (int64_t)take_int(&c, 2);
    const int64_t G = (int64_t)take_int(&c, 3);
    void *alpha = take_ptr(&c, 4);
    void *beta = take_ptr(&c, 5);
    void *mean = take_ptr(&c, 6);
    void *rstd = take_ptr(&c, 7);
    void *gamma = take_ptr(&c, 8);
    void *dy = take_ptr(&c, 9);
    void *dx = take_ptr(&c, 10);
    void *dgamma = take_ptr(&c, 11);
    void *dbeta = take_ptr(&c, 12);
    size_t ws_bytes;
    void *ws = take_ws(&c, 13, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 9);
    same_dtype(&c, 8, 9);
    same_dtype(&c, 10, 9);
    RUN(c, mesa_layernorm_bwd_q(xq, M, D, G, alpha, beta, mean, rstd, gamma, dy, dx, dgamma, dbeta, dt, ws, ws_bytes, stream));
}

ENTRY(linear_dw_q, 11)
{
    struct call c = begin(args, nargs, 11);
    void *xq = take_ptr(&c, 0);
    const int64_t M = (int64_t)take_int(&c, 1);
    const int64_t K = (int64_t)take_int(&c, 2);
    const int64_t G = (int64_t)take_int(&c, 3);
    void *alpha = take_ptr(&c, 4);
    void *beta = take_ptr(&c, 5);
    void *dy = take_ptr(&c, 6);
    const int64_t N_out = (int64_t)take_int(&c, 7);
    void *dW = take_ptr(&c, 8);
    void *db = take_ptr(&c, 9);
    size_t ws_bytes;
    void *ws = take_ws(&c, 10, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 6);
    RUN(c, mesa_linear_dw_q(xq, M, K, G, alpha, beta, dy, N_out, dt, dW, db, ws, ws_bytes, stream));
}

ENTRY(conv2d_dw_q, 9)
{
    struct call c = begin(args, nargs, 9);
    void *xq = take_ptr(&c, 0);
    const mesa_conv2d cv = take_conv(&c, 1);
    const int64_t G = (int64_t)take_int(&c, 2);
    void *alpha = take_ptr(&c, 3);
    void *beta = take_ptr(&c, 4);
    void *dy = take_ptr(&c, 5);
    void *dW = take_ptr(&c, 6);
    void *db = take_ptr(&c, 7);
    size_t ws_bytes;
    void *ws = take_ws(&c, 8, &ws_bytes);
    const mesa_dtype dt = take_dtype(&c, 5);
    RUN(c, mesa_conv2d_dw_q(xq, cv, G, alpha, beta, dy, dt, dW, db, ws, ws_bytes, stream));
}

ENTRY(attn_av_bwd_q, 13)
{
    struct call c = begin(args, nargs, 13);
    void *aq = take_ptr(&c, 0);
    void *vq = take_ptr(&c, 1);
    const int64_t B = (int64_t)take_int(&c, 2);
    const int64_t H = (int64_t)take_int(&c, 3);
    const int64_t N = (int64_t)take_int(&c, 4);
    const int64_t Dh = (int64_t)take_int(&c, 5);
    void *alpha_a = take_ptr(&c, 6);
    void *beta_a = take_ptr(&c, 7);
    void *alpha_v = take_ptr(&c, 8);
    void *beta_v = take_ptr(&c, 9);
    void *dO = take_ptr(&c, 10);
    void *dA = take_ptr(&c, 11);
    void *dV = take_ptr(&c, 12);
    const mesa_dtype dt = take_dtype(&c, 10);
    same_dtype(&c, 11, 10);
    same_dtype(&c, 12, 10);
    RUN(c, mesa_attn_av_bwd_q(aq, vq, B, H, N, Dh, alpha_a, beta_a, alpha_v, beta_v, dO, dA, dV, dt, stream));
}

ENTRY(attn_qk_bwd_q, 14)
{
    struct call c = begin(args, nargs, 14);
    void *qq = take_ptr(&c, 0);
    void *kq = take_ptr(&c, 1);
    const int64_t B = (int64_t)take_int(&c, 2);
    const int64_t H = (int64_t)take_int(&c, 3);
    const int64_t N = (int64_t)take_int(&c, 4);
    const int64_t Dh = (int64_t)take_int(&c, 5);
    void *alpha_q = take_ptr(&c, 6);
    void *beta_q = take_ptr(&c, 7);
    void *alpha_k = take_ptr(&c, 8);
    void *beta_k = take_ptr(&c, 9);
    void *dS = take_ptr(&c, 10);
    const float scale = take_float(&c, 11);
    void *dQ = take_ptr(&c, 12);
    void *dK = take_ptr(&c, 13);
    const mesa_dtype dt = take_dtype(&c, 10);
    same_dtype(&c, 12, 10);
    same_dtype(&c, 13, 10);
    RUN(c, mesa_attn_qk_bwd_q(qq, kq, B, H, N, Dh, alpha_q, beta_q, alpha_k, beta_k, dS, scale, dQ, dK, dt, stream));
}

/* setup(float16, float32, bfloat16, Conv2d, get_device, get_raw_stream) */
static PyObject *py_setup(PyObject *self, PyObject *args)
{
    PyObject *o[6];
    if (!PyArg_ParseTuple(args, "OOOOOO", &o[0], &o[1], &o[2], &o[3], &o[4], &o[5])) return NULL;
    PyObject **slot[6] = {&t_f16, &t_f32, &t_bf16, &conv_type, &get_device, &get_raw_stream};
    for (int i = 0; i < 6; ++i) {
        Py_INCREF(o[i]);
        Py_XSETREF(*slot[i], o[i]);
    }
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    {"setup", py_setup, METH_VARARGS, NULL},
    METHOD(update_running_params),
    METHOD(update_running_params_sym),
    METHOD(update_running_params_fixed_beta),
    METHOD(update_running_params_static),
    METHOD(update_running_scale_sym),
    METHOD(quantize_headwise),
    METHOD(quantize_headwise_b4),
    METHOD(quantize_sym),
    METHOD(quantize_update_fused),
    METHOD(gelu_fwd_q),
    METHOD(softmax_fwd_q),
    METHOD(layernorm_fwd_q),
    METHOD(dequantize),
    METHOD(dequantize_b4),
    METHOD(dequantize_sym),
    METHOD(gelu_bwd_q),
    METHOD(gelu_bwd_q_b4),
    METHOD(relu_bwd_q),
    METHOD(softmax_bwd_q),
    METHOD(layernorm_bwd_q),
    METHOD(linear_dw_q),
    METHOD(conv2d_dw_q),
    METHOD(attn_av_bwd_q),
    METHOD(attn_qk_bwd_q),
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void)
{
    struct { PyObject **slot; const char *name; } names[] = {
        {&n_is_cuda, "is_cuda"}, {&n_is_contiguous, "is_contiguous"}, {&n_data_ptr, "data_ptr"},
        {&n_dtype, "dtype"}, {&n_numel, "numel"}, {&n_element_size, "element_size"},
    };
    for (size_t i = 0; i < sizeof names / sizeof names[0]; ++i)
        if (!(*names[i].slot = PyUnicode_InternFromString(names[i].name))) return NULL;
    return PyModule_Create(&module);
}
