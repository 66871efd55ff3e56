// tbn_torch.cpp -- the Python calls of the package in native code: tensors checked, outputs and
// workspace taken from torch's allocator, the C ABI (include/tbn.h) called on the current stream.
//
// What it is for: a small layer runs 3-10 us on the GPU, while the same marshalling through
// ctypes took 12-14 us of host time per call (a dozen argument conversions, three foreign calls
// for sizes, a workspace and a stream query), so that every chain of small layers ran at the
// speed of the interpreter.  Here a call takes 3.5 us, of which 1.5 us are the output's allocation
// and most of the rest the launch: ResNet-18 at batch 1, called layer by layer, 356 -> 208 us (the
// time of its kernels), one 5x5 layer on 16 digits 12.4 -> 4.4 us.
//
// Each function takes the positional arguments of its Python namesake in __init__.py and handles
// the ordinary call: plain dense GPU tensors, contiguous, of the expected types and sizes.
// Anything else returns NotImplemented before anything is allocated or queued, and the Python
// code then handles it (and raises its errors); so this file refuses nothing by itself.  Like a
// ctypes call, the library call runs without the interpreter lock.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include "tbn.h"

namespace {

PyObject* g_desc_type = nullptr;   // ConvDesc
PyObject* g_error_type = nullptr;  // TbnError

// ---- arguments ---------------------------------------------------------------------------
// A plain dense contiguous GPU tensor (no subclass, no dispatch mode behind it); null otherwise.
const at::Tensor* dense(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided) return nullptr;
    if (t.unsafeGetTensorImpl()->key_set().has(c10::DispatchKey::Python)) return nullptr;
    return t.is_contiguous() ? &t : nullptr;
}

// ... of this type, with at least `need` elements (the kernels use the first `need`).
const at::Tensor* dense(PyObject* o, at::ScalarType type, int64_t need = 0) {
    const at::Tensor* t = dense(o);
    return t && t->scalar_type() == type && t->numel() >= need ? t : nullptr;
}

bool float_type(const at::Tensor& t, tbn_dtype* out) {
    *out = t.scalar_type() == at::kFloat ? TBN_F32 : TBN_BF16;
    return t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16;
}

bool float_type(PyObject* o, at::ScalarType* out) {
    if (!THPDtype_Check(o)) return false;
    *out = reinterpret_cast<THPDtype*>(o)->scalar_type;
    return *out == at::kFloat || *out == at::kBFloat16;
}

bool number(PyObject* o, float* out) {
    if (!PyFloat_Check(o) && !PyLong_CheckExact(o)) return false;
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    *out = (float)v;
    return true;
}

bool integer(PyObject* o, int32_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v != (int32_t)v) return false;
    *out = (int32_t)v;
    return true;
}

bool truth(PyObject* o, bool* out) {
    if (!PyBool_Check(o)) return false;
    *out = o == Py_True;
    return true;
}

// A layer description and its output size (false also for one the library refuses).
struct Desc {
    tbn_conv_desc d;
    int32_t p, q;
    bool get(PyObject* o) {
        if ((PyObject*)Py_TYPE(o) != g_desc_type) return false;
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return false;
        }
        const bool ok = view.len == (Py_ssize_t)sizeof d;
        if (ok) memcpy(&d, view.buf, sizeof d);
        PyBuffer_Release(&view);
        return ok && tbn_conv_out_dims(&d, &p, &q) == TBN_OK;
    }
    int64_t x_numel() const { return (int64_t)d.n * d.h * d.w * d.c; }
    int64_t y_numel() const { return (int64_t)d.n * p * q * d.k; }
    int64_t w_numel() const { return (int64_t)d.k * d.r * d.s * d.c; }
    int64_t words() const { return tbn_packed_words(d.k, (int64_t)d.r * d.s * d.c); }
};

// An output: the caller's tensor (checked) or one allocated when everything else has been checked.
struct Out {
    PyObject* given = nullptr;
    at::Tensor t;
    bool take(PyObject* o, at::ScalarType type, int64_t numel) {
        if (o == Py_None) return true;
        const at::Tensor* g = dense(o);
        if (!g || g->scalar_type() != type || g->numel() != numel) return false;
        given = o;
        t = *g;
        return true;
    }
    void make(at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& like) {
        if (!given) t = at::empty(sizes, like.options().dtype(type));
    }
    PyObject* object() const {
        if (!given) return THPVariable_Wrap(t);
        Py_INCREF(given);
        return given;
    }
};

at::Tensor bytes_like(const at::Tensor& like, size_t n) {
    return at::empty({(int64_t)n}, like.options().dtype(at::kByte));
}

struct Ws {
    at::Tensor t;
    bool given = false;
    bool take(PyObject* o) {
        if (o == Py_None) return true;
        const at::Tensor* g = dense(o);
        if (!g) return false;
        given = true;
        t = *g;
        return true;
    }
    void make(size_t need, const at::Tensor& like) {
        if (!given && need) t = bytes_like(like, need);
    }
    void* ptr() const { return t.defined() ? t.data_ptr() : nullptr; }
    size_t bytes() const { return t.defined() ? (size_t)t.nbytes() : 0; }
};

hipStream_t stream() { return c10::hip::getCurrentHIPStream().stream(); }

float* f32(const at::Tensor& t) { return reinterpret_cast<float*>(t.data_ptr()); }
uint32_t* u32(const at::Tensor& t) { return reinterpret_cast<uint32_t*>(t.data_ptr()); }
int32_t* i32(const at::Tensor& t) { return reinterpret_cast<int32_t*>(t.data_ptr()); }

// The library call without the interpreter lock; a failed status raises TbnError.
template <typename F>
bool call(const char* name, F f) {
    tbn_status st;
    {
        pybind11::gil_scoped_release unlocked;
        st = f();
    }
    if (st == TBN_OK) return true;
    PyObject* e = PyObject_CallFunction(g_error_type, "iss", (int)st, name, tbn_last_error());
    if (e) {
        PyErr_SetObject(g_error_type, e);
        Py_DECREF(e);
    }
    return false;
}

PyObject* declined() { Py_RETURN_NOTIMPLEMENTED; }

PyObject* pack(std::initializer_list<PyObject*> items) {  // steals the references
    PyObject* t = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject* o : items) PyTuple_SET_ITEM(t, i++, o);
    return t;
}

PyObject* none() {
    Py_INCREF(Py_None);
    return Py_None;
}

#define TBN_ARGS(count)                                                 \
    if (n != (count)) return PyErr_Format(PyExc_TypeError, "%d arguments expected", (int)(count))

// ---- convolutions ------------------------------------------------------------------------
// Optional epilogue operands: false = not an ordinary call.
struct Ep {
    tbn_epilogue e = {};
    bool any = false;
    bool get(PyObject* scale, PyObject* bias, PyObject* residual, PyObject* relu, int32_t k, int64_t y_numel,
             at::ScalarType yt) {
        bool r;
        if (!truth(relu, &r)) return false;
        e.relu = r ? 1 : 0;
        any = r;
        if (scale != Py_None) {
            const at::Tensor* t = dense(scale, at::kFloat, k);
            if (!t) return false;
            e.scale = f32(*t);
            any = true;
        }
        if (bias != Py_None) {
            const at::Tensor* t = dense(bias, at::kFloat, k);
            if (!t) return false;
            e.bias = f32(*t);
            any = true;
        }
        if (residual != Py_None) {
            const at::Tensor* t = dense(residual, yt);
            if (!t || t->numel() != y_numel) return false;
            e.residual = t->data_ptr();
            any = true;
        }
        return true;
    }
    const tbn_epilogue* ptr() const { return any ? &e : nullptr; }
};

// The type of an output: the given tensor's, or the requested one.
bool out_type(PyObject* given, PyObject* requested, at::ScalarType* out) {
    if (given == Py_None) return float_type(requested, out);
    const at::Tensor* t = dense(given);
    tbn_dtype unused;
    if (!t || !float_type(*t, &unused)) return false;
    *out = t->scalar_type();
    return true;
}

tbn_dtype code(at::ScalarType t) { return t == at::kFloat ? TBN_F32 : TBN_BF16; }

// (desc, x, codes, alpha, y, out_dtype, scale, bias, residual, relu, ws)
PyObject* conv2d_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(11);
    Desc d;
    tbn_dtype xt;
    at::ScalarType yt;
    const at::Tensor *x = dense(v[1]), *codes = dense(v[2], at::kInt), *alpha = dense(v[3], at::kFloat);
    if (!d.get(v[0]) || !x || !codes || !alpha || !float_type(*x, &xt) || !out_type(v[4], v[5], &yt)) return declined();
    Out y;
    Ep ep;
    Ws ws;
    if (x->numel() != d.x_numel() || codes->numel() != d.words() || alpha->numel() != d.d.k ||
        !y.take(v[4], yt, d.y_numel()) || !ep.get(v[6], v[7], v[8], v[9], d.d.k, d.y_numel(), yt) || !ws.take(v[10]))
        return declined();
    size_t need = 0;
    if (!ws.given && tbn_workspace_size(TBN_OP_FWD, &d.d, &need) != TBN_OK) return declined();
    y.make({d.d.n, d.p, d.q, d.d.k}, yt, *x);
    ws.make(need, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call("tbn_conv2d_fwd", [&] {
            return tbn_conv2d_fwd(&d.d, xp, xt, u32(*codes), f32(*alpha), ep.ptr(), yp, code(yt), ws.ptr(), ws.bytes(),
                                  stream());
        }))
        return nullptr;
    return y.object();
    END_HANDLE_TH_ERRORS
}

// (desc, x, w, y, out_dtype, scale, bias, residual, relu)
PyObject* conv2d_fwd_dense(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(9);
    Desc d;
    tbn_dtype xt;
    at::ScalarType yt;
    const at::Tensor *x = dense(v[1]), *w = dense(v[2], at::kFloat);
    if (!d.get(v[0]) || !x || !w || !float_type(*x, &xt) || !out_type(v[3], v[4], &yt)) return declined();
    Out y;
    Ep ep;
    if (x->numel() != d.x_numel() || w->numel() != d.w_numel() || !y.take(v[3], yt, d.y_numel()) ||
        !ep.get(v[5], v[6], v[7], v[8], d.d.k, d.y_numel(), yt))
        return declined();
    y.make({d.d.n, d.p, d.q, d.d.k}, yt, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call("tbn_conv2d_fwd_dense",
              [&] { return tbn_conv2d_fwd_dense(&d.d, xp, xt, f32(*w), ep.ptr(), yp, code(yt), stream()); }))
        return nullptr;
    return y.object();
    END_HANDLE_TH_ERRORS
}

// (desc, xq, codes, alpha, x_scale, y, out_dtype, relu), int8 or E4M3 activation codes
template <at::ScalarType XT, typename F>
PyObject* conv2d_fwd_codes(PyObject* const* v, Py_ssize_t n, const char* name, F launch) {
    HANDLE_TH_ERRORS
    TBN_ARGS(8);
    Desc d;
    float scale;
    bool relu;
    at::ScalarType yt;
    const at::Tensor *x = dense(v[1], XT), *codes = dense(v[2], at::kInt), *alpha = dense(v[3], at::kFloat);
    if (!d.get(v[0]) || !x || !codes || !alpha || !number(v[4], &scale) || !out_type(v[5], v[6], &yt) ||
        !truth(v[7], &relu))
        return declined();
    Out y;
    if (x->numel() != d.x_numel() || codes->numel() != d.words() || alpha->numel() != d.d.k ||
        !y.take(v[5], yt, d.y_numel()))
        return declined();
    y.make({d.d.n, d.p, d.q, d.d.k}, yt, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call(name, [&] {
            return launch(&d.d, xp, u32(*codes), f32(*alpha), scale, relu ? 1 : 0, yp, code(yt), stream());
        }))
        return nullptr;
    return y.object();
    END_HANDLE_TH_ERRORS
}

PyObject* conv2d_fwd_i8(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return conv2d_fwd_codes<at::kChar>(v, n, "tbn_conv2d_fwd_i8", [](auto d, void* x, auto... rest) {
        return tbn_conv2d_fwd_i8(d, reinterpret_cast<const int8_t*>(x), rest...);
    });
}

PyObject* conv2d_fwd_fp8(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return conv2d_fwd_codes<at::kByte>(v, n, "tbn_conv2d_fwd_fp8", [](auto d, void* x, auto... rest) {
        return tbn_conv2d_fwd_fp8(d, reinterpret_cast<const uint8_t*>(x), rest...);
    });
}

// (desc, dy, codes, alpha, dx, out_dtype, ws)
PyObject* conv2d_bwd_data(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(7);
    Desc d;
    at::ScalarType xt;
    const at::Tensor *dy = dense(v[1], at::kBFloat16), *codes = dense(v[2], at::kInt), *alpha = dense(v[3], at::kFloat);
    if (!d.get(v[0]) || !dy || !codes || !alpha || !out_type(v[4], v[5], &xt)) return declined();
    Out dx;
    Ws ws;
    if (dy->numel() != d.y_numel() || codes->numel() != d.words() || alpha->numel() != d.d.k ||
        !dx.take(v[4], xt, d.x_numel()) || !ws.take(v[6]))
        return declined();
    size_t need = 0;
    if (!ws.given && tbn_workspace_size(TBN_OP_BWD_DATA, &d.d, &need) != TBN_OK) return declined();
    dx.make({d.d.n, d.d.h, d.d.w, d.d.c}, xt, *dy);
    ws.make(need < 16 ? 16 : need, *dy);
    void *dyp = dy->data_ptr(), *dxp = dx.t.data_ptr();
    if (!call("tbn_conv2d_bwd_data", [&] {
            return tbn_conv2d_bwd_data(&d.d, dyp, u32(*codes), f32(*alpha), dxp, code(xt), ws.ptr(), ws.bytes(), stream());
        }))
        return nullptr;
    return dx.object();
    END_HANDLE_TH_ERRORS
}

// (desc, x, dy, dw, accumulate, ws)
PyObject* conv2d_bwd_weight(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(6);
    Desc d;
    bool acc;
    const at::Tensor *x = dense(v[1], at::kBFloat16), *dy = dense(v[2], at::kBFloat16);
    if (!d.get(v[0]) || !x || !dy || !truth(v[4], &acc)) return declined();
    Out dw;
    Ws ws;
    if (x->numel() != d.x_numel() || dy->numel() != d.y_numel() || !dw.take(v[3], at::kFloat, d.w_numel()) ||
        !ws.take(v[5]))
        return declined();
    size_t need = 0;
    if (!ws.given && tbn_workspace_size(TBN_OP_BWD_WEIGHT, &d.d, &need) != TBN_OK) return declined();
    dw.make({d.d.k, d.d.r, d.d.s, d.d.c}, at::kFloat, *x);
    ws.make(need < 16 ? 16 : need, *x);
    void *xp = x->data_ptr(), *dyp = dy->data_ptr();
    if (!call("tbn_conv2d_bwd_weight", [&] {
            return tbn_conv2d_bwd_weight(&d.d, xp, dyp, f32(dw.t), acc ? 1 : 0, ws.ptr(), ws.bytes(), stream());
        }))
        return nullptr;
    return dw.object();
    END_HANDLE_TH_ERRORS
}

// ---- quantisation and update -------------------------------------------------------------
// The filters [K][...] and the outputs of a quantisation.
struct Filters {
    int64_t k = 0, n = 0;
    Out codes, alpha, counts;
    bool want = false;
    bool get(const at::Tensor& w, PyObject* pc, PyObject* pa, PyObject* pn, PyObject* want_counts) {
        bool wanted;
        if (w.dim() < 1 || w.size(0) < 1 || w.numel() < 1 || !truth(want_counts, &wanted)) return false;
        k = w.size(0);
        n = w.numel() / k;
        want = wanted || pn != Py_None;
        if (pn != Py_None) {  // any size that holds the counts
            const at::Tensor* t = dense(pn, at::kInt, 2 * k);
            if (!t || !counts.take(pn, at::kInt, t->numel())) return false;
        }
        return codes.take(pc, at::kInt, tbn_packed_words(k, n)) && alpha.take(pa, at::kFloat, k);
    }
    void make(const at::Tensor& like) {
        codes.make({tbn_packed_words(k, n)}, at::kInt, like);
        alpha.make({k}, at::kFloat, like);
        if (want) counts.make({k, 2}, at::kInt, like);
    }
    int32_t* counts_ptr() const { return want ? i32(counts.t) : nullptr; }
    PyObject* result() const { return pack({codes.object(), alpha.object(), want ? counts.object() : none()}); }
};

// (w, codes, alpha, counts, want_counts)
PyObject* quantize(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(5);
    const at::Tensor* w = dense(v[0], at::kFloat);
    Filters f;
    if (!w || !f.get(*w, v[1], v[2], v[3], v[4])) return declined();
    f.make(*w);
    if (!call("tbn_quantize", [&] {
            return tbn_quantize(f32(*w), f.k, f.n, u32(f.codes.t), f32(f.alpha.t), f.counts_ptr(), stream());
        }))
        return nullptr;
    return f.result();
    END_HANDLE_TH_ERRORS
}

// (w, v, g, lr, momentum, weight_decay)
PyObject* sgd_step(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(6);
    float lr, mu, wd;
    const at::Tensor *w = dense(v[0], at::kFloat), *m = dense(v[1], at::kFloat), *g = dense(v[2], at::kFloat);
    if (!w || !m || !g || m->numel() != w->numel() || g->numel() != w->numel() || !number(v[3], &lr) ||
        !number(v[4], &mu) || !number(v[5], &wd))
        return declined();
    if (!call("tbn_sgd_step", [&] { return tbn_sgd_step(f32(*w), f32(*m), f32(*g), w->numel(), lr, mu, wd, stream()); }))
        return nullptr;
    Py_INCREF(v[0]);
    Py_INCREF(v[1]);
    return pack({v[0], v[1]});
    END_HANDLE_TH_ERRORS
}

// (w, v, g, lr, momentum, weight_decay, codes, alpha, counts, want_counts)
PyObject* sgd_step_quantize(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(10);
    float lr, mu, wd;
    const at::Tensor *w = dense(v[0], at::kFloat), *m = dense(v[1], at::kFloat), *g = dense(v[2], at::kFloat);
    Filters f;
    if (!w || !m || !g || !f.get(*w, v[6], v[7], v[8], v[9]) || m->numel() != f.k * f.n || g->numel() != f.k * f.n ||
        !number(v[3], &lr) || !number(v[4], &mu) || !number(v[5], &wd))
        return declined();
    f.make(*w);
    if (!call("tbn_sgd_step_quantize", [&] {
            return tbn_sgd_step_quantize(f32(*w), f32(*m), f32(*g), f.k, f.n, lr, mu, wd, u32(f.codes.t), f32(f.alpha.t),
                                         f.counts_ptr(), stream());
        }))
        return nullptr;
    return f.result();
    END_HANDLE_TH_ERRORS
}

// (x, inv_scale, q)
template <at::ScalarType QT, typename F>
PyObject* quantize_act(PyObject* const* v, Py_ssize_t n, const char* name, F launch) {
    HANDLE_TH_ERRORS
    TBN_ARGS(3);
    float inv;
    tbn_dtype xt;
    const at::Tensor* x = dense(v[0]);
    Out q;
    if (!x || !float_type(*x, &xt) || !number(v[1], &inv) || !q.take(v[2], QT, x->numel())) return declined();
    q.make(x->sizes(), QT, *x);
    void *xp = x->data_ptr(), *qp = q.t.data_ptr();
    if (!call(name, [&] { return launch(xp, xt, x->numel(), inv, qp, stream()); })) return nullptr;
    return q.object();
    END_HANDLE_TH_ERRORS
}

PyObject* quantize_act_i8(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return quantize_act<at::kChar>(v, n, "tbn_quantize_act_i8",
                                   [](void* x, tbn_dtype xt, int64_t c, float inv, void* q, hipStream_t s) {
                                       return tbn_quantize_act_i8(x, xt, c, inv, reinterpret_cast<int8_t*>(q), s);
                                   });
}

PyObject* quantize_act_fp8(PyObject*, PyObject* const* v, Py_ssize_t n) {
    return quantize_act<at::kByte>(v, n, "tbn_quantize_act_fp8",
                                   [](void* x, tbn_dtype xt, int64_t c, float inv, void* q, hipStream_t s) {
                                       return tbn_quantize_act_fp8(x, xt, c, inv, reinterpret_cast<uint8_t*>(q), s);
                                   });
}

// ---- layers around the convolutions ------------------------------------------------------
bool pool_desc(const at::Tensor& x, PyObject* k, PyObject* stride, PyObject* pad, tbn_pool_desc* d) {
    if (x.dim() != 4) return false;
    for (int i = 0; i < 4; ++i)
        if (x.size(i) != (int32_t)x.size(i)) return false;
    d->n = (int32_t)x.size(0);
    d->h = (int32_t)x.size(1);
    d->w = (int32_t)x.size(2);
    d->c = (int32_t)x.size(3);
    return integer(k, &d->k) && integer(stride, &d->stride) && integer(pad, &d->pad);
}

// (x, k, stride, pad, want_argmax)
PyObject* maxpool2d_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(5);
    const at::Tensor* x = dense(v[0], at::kBFloat16);
    tbn_pool_desc d;
    int32_t p, q;
    bool want;
    if (!x || !pool_desc(*x, v[1], v[2], v[3], &d) || !truth(v[4], &want) || tbn_pool_out_dims(&d, &p, &q) != TBN_OK)
        return declined();
    Out y, arg;
    y.make({d.n, p, q, d.c}, at::kBFloat16, *x);
    if (want) arg.make({d.n, p, q, d.c}, at::kInt, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call("tbn_maxpool2d_fwd", [&] { return tbn_maxpool2d_fwd(&d, xp, yp, want ? i32(arg.t) : nullptr, stream()); }))
        return nullptr;
    return pack({y.object(), want ? arg.object() : none()});
    END_HANDLE_TH_ERRORS
}

// (x, out_dtype)
PyObject* avgpool_global(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(2);
    const at::Tensor* x = dense(v[0], at::kBFloat16);
    at::ScalarType yt;
    if (!x || x->dim() != 4 || !float_type(v[1], &yt)) return declined();
    for (int i = 0; i < 4; ++i)
        if (x->size(i) != (int32_t)x->size(i)) return declined();
    Out y;
    y.make({x->size(0), x->size(3)}, yt, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call("tbn_avgpool_global", [&] {
            return tbn_avgpool_global((int32_t)x->size(0), (int32_t)x->size(1), (int32_t)x->size(2), (int32_t)x->size(3),
                                      xp, yp, code(yt), stream());
        }))
        return nullptr;
    return y.object();
    END_HANDLE_TH_ERRORS
}

bool rows_of(const at::Tensor& x, int64_t* rows, int32_t* c) {
    if (x.dim() < 1 || x.numel() < 1 || x.size(-1) != (int32_t)x.size(-1)) return false;
    *c = (int32_t)x.size(-1);
    *rows = x.numel() / *c;
    return true;
}

// (x, gamma, beta, eps, relu, ws)
PyObject* batchnorm_train_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(6);
    const at::Tensor *x = dense(v[0], at::kBFloat16), *gamma = dense(v[1], at::kFloat), *beta = dense(v[2], at::kFloat);
    int64_t rows;
    int32_t c;
    float eps;
    bool relu;
    Ws ws;
    size_t need = 0;
    if (!x || !gamma || !beta || !rows_of(*x, &rows, &c) || gamma->numel() < c || beta->numel() < c ||
        !number(v[3], &eps) || !truth(v[4], &relu) || !ws.take(v[5]) ||
        tbn_batchnorm_workspace_size(rows, c, &need) != TBN_OK)
        return declined();
    Out y, mean, inv;
    y.make(x->sizes(), at::kBFloat16, *x);
    mean.make({c}, at::kFloat, *x);
    inv.make({c}, at::kFloat, *x);
    ws.make(need, *x);
    void *xp = x->data_ptr(), *yp = y.t.data_ptr();
    if (!call("tbn_batchnorm_train_fwd", [&] {
            return tbn_batchnorm_train_fwd(xp, rows, c, f32(*gamma), f32(*beta), eps, relu ? 1 : 0, yp, f32(mean.t),
                                           f32(inv.t), ws.ptr(), ws.bytes(), stream());
        }))
        return nullptr;
    return pack({y.object(), mean.object(), inv.object()});
    END_HANDLE_TH_ERRORS
}

// (x, y, dy, mean, inv_std, gamma, relu, ws, dgamma, dbeta)
PyObject* batchnorm_train_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(10);
    const at::Tensor *x = dense(v[0], at::kBFloat16), *y = dense(v[1], at::kBFloat16), *dy = dense(v[2], at::kBFloat16);
    const at::Tensor *mean = dense(v[3], at::kFloat), *inv = dense(v[4], at::kFloat), *gamma = dense(v[5], at::kFloat);
    int64_t rows;
    int32_t c;
    bool relu;
    Ws ws;
    size_t need = 0;
    Out dx, dgamma, dbeta;
    if (!x || !y || !dy || !mean || !inv || !gamma || !rows_of(*x, &rows, &c) ||
        y->numel() < x->numel() || dy->numel() < x->numel() || mean->numel() < c || inv->numel() < c ||
        gamma->numel() < c || !truth(v[6], &relu) || !ws.take(v[7]) ||
        !dgamma.take(v[8], at::kFloat, c) || !dbeta.take(v[9], at::kFloat, c) ||
        tbn_batchnorm_workspace_size(rows, c, &need) != TBN_OK)
        return declined();
    dx.make(x->sizes(), at::kBFloat16, *x);
    dgamma.make({c}, at::kFloat, *x);
    dbeta.make({c}, at::kFloat, *x);
    ws.make(need, *x);
    void *xp = x->data_ptr(), *yp = y->data_ptr(), *dyp = dy->data_ptr(), *dxp = dx.t.data_ptr();
    if (!call("tbn_batchnorm_train_bwd", [&] {
            return tbn_batchnorm_train_bwd(xp, yp, dyp, rows, c, relu ? 1 : 0, f32(*mean), f32(*inv), f32(*gamma),
                                           f32(dgamma.t), f32(dbeta.t), dxp, ws.ptr(), ws.bytes(), stream());
        }))
        return nullptr;
    return pack({dx.object(), dgamma.object(), dbeta.object()});
    END_HANDLE_TH_ERRORS
}

// (y, dy)
PyObject* relu_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(2);
    const at::Tensor *y = dense(v[0], at::kBFloat16), *dy = dense(v[1], at::kBFloat16);
    if (!y || !dy || y->numel() < dy->numel()) return declined();
    Out dx;
    dx.make(dy->sizes(), at::kBFloat16, *dy);
    void *yp = y->data_ptr(), *dyp = dy->data_ptr(), *dxp = dx.t.data_ptr();
    if (!call("tbn_relu_bwd", [&] { return tbn_relu_bwd(yp, dyp, dy->numel(), dxp, stream()); })) return nullptr;
    return dx.object();
    END_HANDLE_TH_ERRORS
}

// (logits, labels)
PyObject* softmax_xent(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(2);
    const at::Tensor *z = dense(v[0], at::kFloat), *labels = dense(v[1], at::kInt);
    if (!z || !labels || z->dim() != 2 || z->size(0) != (int32_t)z->size(0) || z->size(1) != (int32_t)z->size(1) ||
        labels->numel() < z->size(0))
        return declined();
    Out loss, per, dz;
    loss.make({1}, at::kFloat, *z);
    per.make({z->size(0)}, at::kFloat, *z);
    dz.make(z->sizes(), at::kBFloat16, *z);
    void* dzp = dz.t.data_ptr();
    if (!call("tbn_softmax_xent", [&] {
            return tbn_softmax_xent(f32(*z), i32(*labels), (int32_t)z->size(0), (int32_t)z->size(1), f32(loss.t),
                                    f32(per.t), dzp, stream());
        }))
        return nullptr;
    return pack({loss.object(), dz.object()});
    END_HANDLE_TH_ERRORS
}

// (dy, argmax, n, h, w, c, k, stride, pad, out_dtype)
PyObject* maxpool2d_bwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    TBN_ARGS(10);
    const at::Tensor *dy = dense(v[0], at::kBFloat16), *arg = dense(v[1], at::kInt);
    tbn_pool_desc d;
    at::ScalarType xt;
    if (!dy || !arg || !integer(v[2], &d.n) || !integer(v[3], &d.h) || !integer(v[4], &d.w) || !integer(v[5], &d.c) ||
        !integer(v[6], &d.k) || !integer(v[7], &d.stride) || !integer(v[8], &d.pad) || !float_type(v[9], &xt))
        return declined();
    int32_t p, q;
    if (tbn_pool_out_dims(&d, &p, &q) != TBN_OK) return declined();
    const int64_t windows = (int64_t)d.n * p * q * d.c;
    if (dy->numel() < windows || arg->numel() < windows) return declined();
    Out dx;
    dx.make({d.n, d.h, d.w, d.c}, xt, *dy);
    void *dyp = dy->data_ptr(), *dxp = dx.t.data_ptr();
    if (!call("tbn_maxpool2d_bwd", [&] { return tbn_maxpool2d_bwd(&d, dyp, i32(*arg), dxp, code(xt), stream()); }))
        return nullptr;
    return dx.object();
    END_HANDLE_TH_ERRORS
}

// (ConvDesc, TbnError): the Python types that the calls above know
PyObject* bind_types(PyObject*, PyObject* const* v, Py_ssize_t n) {
    TBN_ARGS(2);
    Py_INCREF(v[0]);
    Py_INCREF(v[1]);
    Py_XSETREF(g_desc_type, v[0]);
    Py_XSETREF(g_error_type, v[1]);
    Py_RETURN_NONE;
}

#define TBN_FN(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    TBN_FN(conv2d_fwd),       TBN_FN(conv2d_fwd_dense),    TBN_FN(conv2d_fwd_i8),       TBN_FN(conv2d_fwd_fp8),
    TBN_FN(conv2d_bwd_data),  TBN_FN(conv2d_bwd_weight),   TBN_FN(quantize),            TBN_FN(sgd_step),
    TBN_FN(sgd_step_quantize), TBN_FN(quantize_act_i8),    TBN_FN(quantize_act_fp8),    TBN_FN(maxpool2d_fwd),
    TBN_FN(maxpool2d_bwd),    TBN_FN(avgpool_global),      TBN_FN(batchnorm_train_fwd), TBN_FN(batchnorm_train_bwd),
    TBN_FN(relu_bwd),         TBN_FN(softmax_xent),        TBN_FN(bind_types),          {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tbn_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define TBN_STR2(x) #x
#define TBN_STR(x) TBN_STR2(x)

PyMODINIT_FUNC PyInit__tbn_torch(void) {
    PyObject* m = PyModule_Create(&module);
    // the module uses torch's and Python's C++ types directly: the package looks at this before any call
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", "torch " TBN_TORCH_VERSION ", Python " TBN_STR(PY_MAJOR_VERSION) "."
                                                        TBN_STR(PY_MINOR_VERSION)) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
