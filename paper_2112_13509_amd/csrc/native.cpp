// Argument marshalling of binding.py in native code: checks torch tensors, reads their addresses and sizes, fills the
// plain structs of include/autobyte.h and calls the C ABI.  Small calls are bound by the host: with the same work done
// in Python (ctypes structs, one attribute call per tensor property) a call cost about 8 us before the library saw it.
// The library itself is the one binding.py loaded: its entry points arrive as addresses (bind()).
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include <Python.h>
#include "../../include/autobyte.h"

namespace {

decltype(&ab_score_candidates) p_score;
decltype(&ab_score_candidates_v) p_score_v;
decltype(&ab_score_candidates_static) p_score_static;
decltype(&ab_select_best) p_select;
decltype(&ab_trigger) p_trigger;
decltype(&ab_online_update_tail) p_update;
decltype(&ab_replay_mix) p_mix;

struct Failed {};                       // a Python exception is set

[[noreturn]] void fail(PyObject *type, const char *fmt, const char *what)
{
    PyErr_Format(type, fmt, what);
    throw Failed{};
}

const at::Tensor *tensor_or_null(PyObject *o, const char *what)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o) || !THPVariable_Unpack(o).is_cuda()) fail(PyExc_TypeError, "%s must be a tensor on the GPU", what);
    return &THPVariable_Unpack(o);
}
// Address of a contiguous GPU tensor of the given type (NULL for None), as binding.py promises its callers.
void *ptr(PyObject *o, at::ScalarType dt, const char *what)
{
    const at::Tensor *t = tensor_or_null(o, what);
    if (!t) return nullptr;
    if (t->scalar_type() != dt) {
        PyErr_Format(PyExc_TypeError, "%s must have dtype torch.%s, got torch.%s", what,
                     dt == at::kFloat ? "float32" : dt == at::kInt ? "int32" : "uint8",
                     t->scalar_type() == at::kFloat ? "float32" : t->scalar_type() == at::kDouble ? "float64" :
                     t->scalar_type() == at::kBFloat16 ? "bfloat16" : t->scalar_type() == at::kHalf ? "float16" :
                     t->scalar_type() == at::kLong ? "int64" : t->scalar_type() == at::kInt ? "int32" :
                     t->scalar_type() == at::kByte ? "uint8" : c10::toString(t->scalar_type()));
        throw Failed{};
    }
    if (!t->is_contiguous()) fail(PyExc_TypeError, "%s must be contiguous", what);
    return t->data_ptr();
}
float *fptr(PyObject *o, const char *what) { return (float *)ptr(o, at::kFloat, what); }
int32_t *iptr(PyObject *o, const char *what) { return (int32_t *)ptr(o, at::kInt, what); }
uint8_t *bptr(PyObject *o, const char *what) { return (uint8_t *)ptr(o, at::kByte, what); }

// Shape queries take any tensor: its place, type and layout are looked at where its address is taken.
const at::Tensor &any_tensor(PyObject *o, const char *what)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a tensor on the GPU", what);
    return THPVariable_Unpack(o);
}
int64_t size_at(const at::Tensor &t, int64_t d, const char *what)
{
    if (t.dim() <= (d < 0 ? -d - 1 : d)) fail(PyExc_IndexError, "%s has too few dimensions", what);
    return t.size(d);
}
void want_numel(PyObject *o, int64_t n, const char *what)
{
    if (o == Py_None) return;
    const int64_t have = any_tensor(o, what).numel();
    if (have != n) {
        PyErr_Format(PyExc_ValueError, "%s has %lld elements, expected %lld", what, (long long)have, (long long)n);
        throw Failed{};
    }
}

// The memory behind a ctypes structure (desc, params), through the buffer protocol.
struct Struct {
    Py_buffer b;
    Struct(PyObject *o, Py_ssize_t bytes)
    {
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw Failed{};
        if (b.len != bytes) {
            PyBuffer_Release(&b);
            fail(PyExc_TypeError, "%s", "not a structure of the expected size");
        }
    }
    ~Struct() { PyBuffer_Release(&b); }
    Struct(const Struct &) = delete;
};

// None: torch's current stream; an object with .cuda_stream, or a plain handle.
void *stream_of(PyObject *o)
{
    if (o == Py_None) return (void *)c10::hip::getCurrentHIPStream().stream();
    PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
        PyErr_Clear();
        Py_INCREF(o);
        h = o;
    }
    PyObject *i = PyNumber_Long(h);
    Py_DECREF(h);
    if (!i) throw Failed{};
    void *v = PyLong_AsVoidPtr(i);
    Py_DECREF(i);
    if (!v && PyErr_Occurred()) throw Failed{};
    return v;
}
// Whatever int() takes: 256.0 and 0-dimensional arrays count as whole numbers.
int64_t int_of(PyObject *o)
{
    PyObject *i = PyNumber_Long(o);
    if (!i) throw Failed{};
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
}
float float_of(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Failed{};
    return (float)v;
}
int64_t n_outputs(const ab_model_desc *d) { return d->n_outputs > 1 ? d->n_outputs : 1; }

// The library is called without the interpreter's lock (an enqueue can wait for room in the queue; a trace callback
// takes the lock itself).  The tensors and structures behind the addresses are the caller's arguments and stay alive.
template <typename F>
long unlocked(F f)
{
    PyThreadState *save = PyEval_SaveThread();
    const long rc = f();
    PyEval_RestoreThread(save);
    return rc;
}
template <typename F>
PyObject *guarded(PyObject *const *a, Py_ssize_t n, Py_ssize_t want, F f)
{
    if (n != want || !p_score) {
        PyErr_SetString(PyExc_TypeError, "internal call with the wrong number of arguments");
        return nullptr;
    }
    try {
        return PyLong_FromLong(f());
    } catch (const Failed &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// desc, params, dyn, scalars, partition, credit, scores, best_idx, best_score, workspace, stream, layers_of, static, v_best
PyObject *score(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(a, n, 14, [&]() -> long {
        Struct ds(a[0], sizeof(ab_model_desc)), ps(a[1], sizeof(ab_params));
        const ab_model_desc *d = (const ab_model_desc *)ds.b.buf;
        const at::Tensor &dyn = any_tensor(a[2], "dyn"), &scal = any_tensor(a[3], "scalars");
        const at::Tensor &part = any_tensor(a[4], "partition_bytes"), &cred = any_tensor(a[5], "credit_mult");
        const int64_t S = size_at(dyn, 0, "dyn");
        if (a[11] != Py_None && any_tensor(a[11], "layers_of").numel() != S)
            fail(PyExc_ValueError, "%s", "layers_of must have one entry per scenario");
        ab_stats st{fptr(a[2], "dyn"), fptr(a[3], "scalars"), S, iptr(a[11], "layers_of")};
        const bool per_scenario = part.dim() == 2;
        if (per_scenario && (cred.dim() != 2 || part.size(0) != S || cred.size(0) != S))
            fail(PyExc_ValueError, "%s", "per-scenario grids must be [S, P] and [S, Q]");
        const int64_t P = size_at(part, -1, "partition_bytes"), Q = size_at(cred, -1, "credit_mult");
        ab_grid gr{fptr(a[4], "partition_bytes"), (int32_t)P, fptr(a[5], "credit_mult"), (int32_t)Q, per_scenario ? 1 : 0};
        if (dyn.numel() != S * d->n_layers * d->n_stats || scal.numel() != S * d->n_scalars)
            fail(PyExc_ValueError, "%s", "dyn / scalars do not match the description");
        want_numel(a[6], S * P * Q, "scores");
        want_numel(a[7], S, "best_idx");
        want_numel(a[8], S, "best_score");
        want_numel(a[13], S * n_outputs(d), "v_best");
        const int is_static = PyObject_IsTrue(a[12]);
        if (is_static < 0) throw Failed{};
        if (is_static && (a[9] != Py_None || a[13] != Py_None))
            fail(PyExc_ValueError, "%s", "the static-scratch form takes neither a workspace nor v_best");
        const ab_params *prm = (const ab_params *)ps.b.buf;
        float *scores = fptr(a[6], "scores"), *best = fptr(a[8], "best_score");
        int32_t *idx = iptr(a[7], "best_idx");
        float *v = fptr(a[13], "v_best");
        void *ws = bptr(a[9], "workspace");
        const size_t wb = a[9] != Py_None ? (size_t)THPVariable_Unpack(a[9]).numel() : 0;
        void *sm = stream_of(a[10]);
        return unlocked([&]() -> long {
            if (is_static) return p_score_static(d, prm, &st, &gr, scores, idx, best, sm);
            if (a[13] != Py_None) return p_score_v(d, prm, &st, &gr, scores, idx, best, v, ws, wb, sm);
            return p_score(d, prm, &st, &gr, scores, idx, best, ws, wb, sm);
        });
    });
}

struct Rows { int64_t S, C, stride; };
Rows rows_of(PyObject *scores, PyObject *C_, PyObject *row_stride)
{
    const at::Tensor &t = any_tensor(scores, "scores");
    if (t.dim() != 2) fail(PyExc_ValueError, "%s", "scores must be 2-D");
    Rows r{t.size(0), 0, row_stride == Py_None ? t.size(1) : int_of(row_stride)};
    r.C = C_ == Py_None ? r.stride : int_of(C_);
    return r;
}
bool numel_is(PyObject *o, int64_t n, const char *what) { return o == Py_None || any_tensor(o, what).numel() == n; }

// scores, best_idx, best_score, C_, row_stride, stream
PyObject *select(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(a, n, 6, [&]() -> long {
        const Rows r = rows_of(a[0], a[3], a[4]);
        if (any_tensor(a[1], "best_idx").numel() != r.S || !numel_is(a[2], r.S, "best_score"))
            fail(PyExc_ValueError, "%s", "best_idx / best_score must have one element per row");
        const float *sc = fptr(a[0], "scores");
        int32_t *idx = iptr(a[1], "best_idx");
        float *best = fptr(a[2], "best_score");
        void *sm = stream_of(a[5]);
        return unlocked([&]() -> long { return p_select(sc, r.S, (int32_t)r.C, r.stride, idx, best, sm); });
    });
}

// scores, current_idx, best_idx, reconfigure, observed, gain, adapt, gain_threshold, error_threshold, C_, row_stride, stream
PyObject *trigger(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(a, n, 12, [&]() -> long {
        const Rows r = rows_of(a[0], a[9], a[10]);
        static const char *names[7] = {"scores", "current_idx", "best_idx", "reconfigure", "observed", "gain", "adapt"};
        for (int i = 1; i < 7; ++i)
            if (!numel_is(a[i], r.S, names[i])) fail(PyExc_ValueError, "%s must have one element per row", names[i]);
        const float *sc = fptr(a[0], "scores"), *obs = fptr(a[4], "observed");
        const int32_t *cur = iptr(a[1], "current_idx");
        const float gt = float_of(a[7]), et = float_of(a[8]);
        int32_t *idx = iptr(a[2], "best_idx");
        float *gain = fptr(a[5], "gain");
        uint8_t *rec = bptr(a[3], "reconfigure"), *ad = bptr(a[6], "adapt");
        void *sm = stream_of(a[11]);
        return unlocked([&]() -> long {
            return p_trigger(sc, r.S, (int32_t)r.C, r.stride, cur, obs, gt, et, idx, gain, rec, ad, sm);
        });
    });
}

// desc, params, has_step, x_raw, target, first_trainable, lr, beta1, beta2, eps, loss_out, workspace, stream
PyObject *update(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(a, n, 13, [&]() -> long {
        Struct ds(a[0], sizeof(ab_model_desc)), ps(a[1], sizeof(ab_params));
        const ab_model_desc *d = (const ab_model_desc *)ds.b.buf;
        const at::Tensor &x = any_tensor(a[3], "x_raw");
        const int64_t B = size_at(x, 0, "x_raw"), F = (int64_t)d->n_layers * d->n_stats + d->n_scalars + 2;
        if (x.numel() != B * F || any_tensor(a[4], "target").numel() != B * n_outputs(d)) {
            PyErr_Format(PyExc_ValueError, "x_raw must be [B, %lld] and target [B, n_outputs]", (long long)F);
            throw Failed{};
        }
        if (a[2] != Py_True) fail(PyExc_ValueError, "%s", "params were not created with trainable=True");
        void *ws = bptr(a[11], "workspace");
        const size_t wb = a[11] != Py_None ? (size_t)THPVariable_Unpack(a[11]).numel() : 0;
        const float *xp = fptr(a[3], "x_raw"), *yp = fptr(a[4], "target");
        const int32_t first = (int32_t)int_of(a[5]);
        const float lr = float_of(a[6]), b1 = float_of(a[7]), b2 = float_of(a[8]), eps = float_of(a[9]);
        float *loss = fptr(a[10], "loss_out");
        void *sm = stream_of(a[12]);
        return unlocked([&]() -> long {
            return p_update(d, (ab_params *)ps.b.buf, xp, yp, B, first, lr, b1, b2, eps, loss, ws, wb, sm);
        });
    });
}

// x_new, target_new, x_old, target_old, pick, x_out, target_out, stream
PyObject *replay_mix(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(a, n, 8, [&]() -> long {
        const at::Tensor &x = any_tensor(a[5], "x_out");
        const int64_t B = size_at(x, 0, "x_out"), F = size_at(x, 1, "x_out");
        int64_t rows[2] = {0, 0};
        for (int i = 0; i < 2; ++i) {
            if (a[2 * i] == Py_None) continue;
            const at::Tensor &p = any_tensor(a[2 * i], i ? "x_old" : "x_new");
            rows[i] = size_at(p, 0, i ? "x_old" : "x_new");
            if (size_at(p, 1, i ? "x_old" : "x_new") != F)
                fail(PyExc_ValueError, "%s", "pools and output must have the same row width");
        }
        const int64_t nt = any_tensor(a[6], "target_out").numel();
        if (B == 0) fail(PyExc_ZeroDivisionError, "%s", "integer modulo by zero");
        if (any_tensor(a[4], "pick").numel() != B || nt % B != 0)
            fail(PyExc_ValueError, "%s", "pick must have one entry and target_out n_outputs entries per output row");
        const int64_t n_out = nt / B;
        for (int i = 0; i < 2; ++i)
            if (!numel_is(a[2 * i + 1], rows[i] * n_out, i ? "target_old" : "target_new")) {
                PyErr_Format(PyExc_ValueError, "pool targets must have %lld entries per row", (long long)n_out);
                throw Failed{};
            }
        const float *xn = fptr(a[0], "x_new"), *tn = fptr(a[1], "target_new"), *xo = fptr(a[2], "x_old"), *to = fptr(a[3], "target_old");
        const int32_t *pick = iptr(a[4], "pick");
        float *xout = fptr(a[5], "x_out"), *tout = fptr(a[6], "target_out");
        void *sm = stream_of(a[7]);
        return unlocked([&]() -> long {
            return p_mix(xn, tn, rows[0], xo, to, rows[1], pick, B, (int32_t)F, (int32_t)n_out, xout, tout, sm);
        });
    });
}

// The addresses of the library's entry points, in the order of the pointers above.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "bind takes seven addresses");
        return nullptr;
    }
    void *p[7];
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: a null address");
            return nullptr;
        }
    }
    p_score = (decltype(p_score))p[0];
    p_score_v = (decltype(p_score_v))p[1];
    p_score_static = (decltype(p_score_static))p[2];
    p_select = (decltype(p_select))p[3];
    p_trigger = (decltype(p_trigger))p[4];
    p_update = (decltype(p_update))p[5];
    p_mix = (decltype(p_mix))p[6];
    Py_RETURN_NONE;
}

#define AB_FAST(f) {#f, (PyCFunction)(void *)f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {AB_FAST(bind), AB_FAST(score), AB_FAST(select), AB_FAST(trigger), AB_FAST(update), AB_FAST(replay_mix),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
