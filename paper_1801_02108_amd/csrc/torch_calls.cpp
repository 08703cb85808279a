// The binding's calls on torch tensors: argument checks and marshalling from Python objects to the C ABI of
// include/sbnet.h, nothing else (no arithmetic, no launch of its own).  Every function of this module is the body of the
// function of the same name in __init__.py, which holds its documentation and defaults and passes all arguments in order.
//
// Why native: a fused convolution is 10 us of device time, and the same checks through Python and ctypes (shape tuples,
// 25 converted arguments, a stream object) took 9 us of host time per call, so that most programs of small and middle
// layers ran at the speed of their host.  A call with one launch: 10.2 us of host time before, 3.9 now, the launch included;
// the benchmark stage of six units and a reduction (13 launches) 103 us a pass -> 71, which is its device time.
#include <Python.h>

#include <optional>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sbnet.h"

namespace {

PyObject *g_error = nullptr;                       // SbnetError(code, text)
PyObject *g_geom = nullptr;                        // Geom
PyObject *s_buf, *s_shape, *s_dtype;               // attribute names of PackedWeights
PyObject *s_contents, *s_obj;                      // ... of ctypes.pointer(geom) and ctypes.byref(geom)

[[noreturn]] void raise(PyObject *type, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
[[noreturn]] void raise(PyObject *type, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    PyErr_FormatV(type, fmt, ap);
    va_end(ap);
    throw python_error();
}

void require(bool ok, const char *what) {
    if (!ok) raise(PyExc_AssertionError, "%s", what);
}

using at::Tensor;

const Tensor &dev(PyObject *o, const char *name) {
    if (THPVariable_Check(o)) {
        const Tensor &t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.is_contiguous()) return t;
    }
    raise(PyExc_TypeError, "%s must be a contiguous device tensor", name);
}
const Tensor &dev(PyObject *o, const char *name, at::ScalarType dt) {
    const Tensor &t = dev(o, name);
    if (t.scalar_type() != dt) raise(PyExc_TypeError, "%s must be %s", name, c10::toString(dt));
    return t;
}
bool none(PyObject *o) { return o == Py_None; }

sbnet_dtype dt_of(const Tensor &t) {
    switch (t.scalar_type()) {
        case at::kFloat: return SBNET_F32;
        case at::kBFloat16: return SBNET_BF16;
        case at::kHalf: return SBNET_F16;
        case at::kByte: return SBNET_U8;
        default: raise(PyExc_TypeError, "unsupported dtype %s", c10::toString(t.scalar_type()));
    }
}

void *ptr(const Tensor &t) { return t.data_ptr(); }
float *vec(PyObject *o, const char *name, int64_t n) {           // float32 [n] or None
    if (none(o)) return nullptr;
    const Tensor &t = dev(o, name, at::kFloat);
    require(t.dim() == 1 && t.size(0) == n, name);
    return (float *)ptr(t);
}
float *bias_of(PyObject *o, const char *name = "bias") {
    return none(o) ? nullptr : (float *)ptr(dev(o, name, at::kFloat));
}

int64_t i64(PyObject *o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}
int i32(PyObject *o) { return (int)i64(o); }
float f32(PyObject *o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw python_error();
    return (float)v;
}
int flag(PyObject *o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw python_error();
    return v;
}

// output extent of a valid convolution, floor((t - k) / stride) + 1; zero or less for a tile smaller than the kernel, which the
// library refuses
int64_t extent(int64_t t, int64_t k, int64_t stride) {
    if (stride == 0) raise(PyExc_ZeroDivisionError, "stride must not be zero");
    const int64_t d = t - k, q = d / stride;
    return q - (d % stride != 0 && (d < 0) != (stride < 0)) + 1;
}

[[noreturn]] void raise_status(int status, const char *text) {
    PyObject *e = PyObject_CallFunction(g_error, "is", status, text);
    if (e) PyErr_SetObject(g_error, e);
    Py_XDECREF(e);
    throw python_error();
}

struct Geo : sbnet_geom {                           // a Geom, or a ctypes pointer to one
    explicit Geo(PyObject *o) {
        if (none(o)) raise_status(SBNET_EINVAL, "no geometry");
        if (read(o)) return;
        for (PyObject *name : {s_contents, s_obj}) {
            PyObject *g = PyObject_GetAttr(o, name);
            if (!g) {
                if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw python_error();
                PyErr_Clear();
                continue;
            }
            const bool ok = read(g);
            Py_DECREF(g);
            if (ok) return;
        }
        raise(PyExc_TypeError, "a geometry (Geom) is expected");
    }

private:
    bool read(PyObject *o) {
        const int is = PyObject_IsInstance(o, g_geom);
        if (is < 0) throw python_error();
        if (!is) return false;
        Py_buffer v;
        if (PyObject_GetBuffer(o, &v, PyBUF_SIMPLE) < 0) throw python_error();
        memcpy(static_cast<sbnet_geom *>(this), v.buf, sizeof(sbnet_geom));
        PyBuffer_Release(&v);
        return true;
    }
};

struct Dims4 {
    int a, b, c, d;
    Dims4(const Tensor &t, const char *name) {
        if (t.dim() != 4) raise(PyExc_ValueError, "%s must have four dimensions", name);
        a = (int)t.size(0); b = (int)t.size(1); c = (int)t.size(2); d = (int)t.size(3);
    }
    bool is(int64_t p, int64_t q, int64_t r, int64_t s) const { return a == p && b == q && c == r && d == s; }
};

// The n objects of an argument that holds several (weights with their biases and the like), kept until the call is over: an
// iterator's objects may have no other owner, and another thread may change a list while the interpreter lock is released.
struct Several {
    PyObject *item[6] = {};
    Several(PyObject *o, int n, const char *what) {
        PyObject *it = PyObject_GetIter(o), *x = nullptr;
        if (!it) throw python_error();
        int k = 0;
        while ((x = PyIter_Next(it)) && k < n) item[k++] = x;
        const bool ok = !x && k == n && !PyErr_Occurred();
        Py_XDECREF(x);
        Py_DECREF(it);
        if (ok) return;
        drop();
        if (PyErr_Occurred()) throw python_error();
        raise(PyExc_ValueError, "%s", what);
    }
    ~Several() { drop(); }
    Several(const Several &) = delete;
    void drop() {
        for (PyObject *&x : item) Py_CLEAR(x);
    }
    PyObject *operator[](int i) const { return item[i]; }
};

struct Packed {                                     // a PackedWeights object
    void *buf;
    int kh, kw, cin, cout;
    at::ScalarType dtype;
    explicit Packed(PyObject *o) {
        PyObject *b = PyObject_GetAttr(o, s_buf), *s = b ? PyObject_GetAttr(o, s_shape) : nullptr,
                 *d = s ? PyObject_GetAttr(o, s_dtype) : nullptr;
        bool ok = d && THPVariable_Check(b) && PyTuple_Check(s) && PyTuple_GET_SIZE(s) == 4 && THPDtype_Check(d);
        if (ok) {
            buf = THPVariable_Unpack(b).data_ptr();
            kh = (int)PyLong_AsLong(PyTuple_GET_ITEM(s, 0)); kw = (int)PyLong_AsLong(PyTuple_GET_ITEM(s, 1));
            cin = (int)PyLong_AsLong(PyTuple_GET_ITEM(s, 2)); cout = (int)PyLong_AsLong(PyTuple_GET_ITEM(s, 3));
            dtype = reinterpret_cast<THPDtype *>(d)->scalar_type;
        }
        Py_XDECREF(b); Py_XDECREF(s); Py_XDECREF(d);                // the caller, or Several, keeps the object, and the buffer with it
        if (PyErr_Occurred()) throw python_error();
        if (!ok) raise(PyExc_TypeError, "packed weights (PackedWeights) are expected");
    }
    bool is(int a, int b, int c, int d) const { return kh == a && kw == b && cin == c && cout == d; }
};

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// The interpreter lock is given back where a call may wait for the device: in the library (room in the device's queue), and in
// an allocation (the allocator may free its cache or wait for events), which would otherwise stop every thread, and for
// good if what the device waits for is a host callback that needs the lock.
struct Unlocked {
    PyThreadState *s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};

Tensor empty(at::IntArrayRef size, const Tensor &like, at::ScalarType dt) {
    const Unlocked u;
    return at::empty(size, like.options().dtype(dt));
}
Tensor zeros_of(const Tensor &like) {
    const Unlocked u;
    return at::zeros_like(like);
}
// a workspace of at least `need` bytes (never empty): the caller's, or a new one kept in `own`
void *space(PyObject *o, const Tensor &like, size_t need, size_t least, Tensor &own, size_t *bytes, bool any_type = false) {
    if (none(o)) {
        own = empty({(int64_t)std::max(need, least)}, like, at::kByte);
        *bytes = (size_t)own.numel();
        return ptr(own);
    }
    const Tensor &t = any_type ? dev(o, "workspace") : dev(o, "workspace", at::kByte);
    *bytes = (size_t)t.numel() * t.element_size();
    return ptr(t);
}
// an output tensor: the caller's, or a new one kept in `own`
const Tensor &output(PyObject *o, const char *name, at::IntArrayRef size, const Tensor &like, at::ScalarType dt, Tensor &own) {
    if (none(o)) {
        own = empty(size, like, dt);
        return own;
    }
    return dev(o, name, dt);
}

PyObject *same(PyObject *o) {
    Py_INCREF(o);
    return o;
}
PyObject *give(PyObject *o, const Tensor &own) { return none(o) ? THPVariable_Wrap(own) : same(o); }
template <typename... O> PyObject *tuple(O... o) {
    PyObject *items[] = {o...};
    PyObject *t = PyTuple_New(sizeof...(o));
    for (size_t i = 0; i < sizeof...(o); ++i)
        if (t) PyTuple_SET_ITEM(t, i, items[i]);
    return t;
}

// a call of the C ABI
template <typename F, typename... A> void call(F f, A... a) {
    sbnet_status st;
    {
        const Unlocked u;
        st = f(a...);
    }
    if (st != SBNET_OK) raise_status((int)st, sbnet_last_error());
}

struct List {                                       // index list and count
    const int32_t *idx, *cnt;
    int cap;
    List(PyObject *i, PyObject *c) {
        const Tensor &ti = dev(i, "indices", at::kInt), &tc = dev(c, "count", at::kInt);
        idx = (const int32_t *)ptr(ti);
        cnt = (const int32_t *)ptr(tc);
        cap = (int)ti.size(0);
    }
};

typedef PyObject *const *Args;

// ---- the calls, arguments in the order of __init__.py ----------------------------------------------------------------
PyObject *reduce_mask(Args a) {                     // mask, g, pool, threshold, indices, count, workspace
    const Tensor &mask = dev(a[0], "mask");
    if (mask.dim() != 3) raise(PyExc_ValueError, "mask must have three dimensions");
    const Geo g(a[1]);
    const int N = (int)mask.size(0);
    Tensor oi, oc, ow;
    const Tensor &idx = output(a[4], "indices", {(int64_t)N * g.bcount_h * g.bcount_w, 3}, mask, at::kInt, oi);
    const Tensor &cnt = output(a[5], "count", {1}, mask, at::kInt, oc);
    size_t wb;
    void *ws = space(a[6], mask, none(a[6]) ? sbnet_workspace_bytes(N, &g) : 0, 0, ow, &wb, true);
    call(sbnet_reduce_mask, ptr(mask), dt_of(mask), N, (int)mask.size(1), (int)mask.size(2), &g, (sbnet_pool)i32(a[2]), f32(a[3]),
         (int32_t *)ptr(idx), (int32_t *)ptr(cnt), (int)idx.size(0), ws, wb, stream());
    return tuple(give(a[4], oi), give(a[5], oc));
}

PyObject *reduce_mask_static(Args a) {              // mask, g, indices, count, pool, threshold
    const Tensor &mask = dev(a[0], "mask"), &idx = dev(a[2], "indices", at::kInt), &cnt = dev(a[3], "count", at::kInt);
    if (mask.dim() != 3) raise(PyExc_ValueError, "mask must have three dimensions");
    const Geo g(a[1]);
    call(sbnet_reduce_mask_static, ptr(mask), dt_of(mask), (int)mask.size(0), (int)mask.size(1), (int)mask.size(2), &g,
         (sbnet_pool)i32(a[4]), f32(a[5]), (int32_t *)ptr(idx), (int32_t *)ptr(cnt), (int)idx.size(0), stream());
    return tuple(same(a[2]), same(a[3]));
}

template <bool CHW> PyObject *gather(Args a) {      // x, indices, count, g, tiles
    const Tensor &x = dev(a[0], "x");
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(x, "x");
    Tensor own;
    const int64_t sz[4] = {l.cap, CHW ? s.d : g.bsize_h, CHW ? g.bsize_h : g.bsize_w, CHW ? g.bsize_w : s.d};
    const Tensor &tiles = output(a[4], "tiles", sz, x, x.scalar_type(), own);
    require(tiles.sizes() == at::IntArrayRef(sz), "shape of tiles");
    call(CHW ? sbnet_sparse_gather_chw : sbnet_sparse_gather, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, l.idx, l.cnt, l.cap, &g, ptr(tiles),
         stream());
    return give(a[4], own);
}

template <bool CHW> PyObject *scatter(Args a) {     // tiles, indices, count, g, y, add
    const Tensor &tiles = dev(a[0], "tiles"), &y = dev(a[4], "y", tiles.scalar_type());
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(y, "y");
    const int64_t sz[4] = {l.cap, CHW ? s.d : g.bsize_h, CHW ? g.bsize_h : g.bsize_w, CHW ? g.bsize_w : s.d};
    require(tiles.sizes() == at::IntArrayRef(sz), "shape of tiles");
    call(CHW ? sbnet_sparse_scatter_chw : sbnet_sparse_scatter, ptr(tiles), dt_of(tiles), l.idx, l.cnt, l.cap, &g, ptr(y), s.a, s.b, s.c,
         s.d, flag(a[5]), stream());
    return same(a[4]);
}

PyObject *gather_backward(Args a) {                 // dtiles, indices, count, g, dx, workspace
    const Tensor &t = dev(a[0], "dtiles"), &dx = dev(a[4], "dx", t.scalar_type());
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(dx, "dx");
    require(Dims4(t, "dtiles").is(l.cap, g.bsize_h, g.bsize_w, s.d), "shape of dtiles");
    Tensor own;
    size_t wb;
    void *ws = space(a[5], dx, sbnet_gather_backward_workspace_bytes(s.a, &g), 4, own, &wb);
    call(sbnet_sparse_gather_backward, ptr(t), dt_of(t), l.idx, l.cnt, l.cap, &g, ptr(dx), s.a, s.b, s.c, s.d, ws, wb, stream());
    return same(a[4]);
}

PyObject *bn_stats(Args a) {                        // x, indices, count, g, workspace
    const Tensor &x = dev(a[0], "x");
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(x, "x");
    Tensor own, mean = empty({s.d}, x, at::kFloat), var = empty({s.d}, x, at::kFloat);
    size_t wb;
    void *ws = space(a[4], x, sbnet_bn_stats_workspace_bytes(l.cap, s.d), 4, own, &wb);
    call(sbnet_sparse_bn_stats, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, l.idx, l.cnt, l.cap, &g, (float *)ptr(mean), (float *)ptr(var), ws, wb,
         stream());
    return tuple(THPVariable_Wrap(mean), THPVariable_Wrap(var));
}

PyObject *bn_apply(Args a) {                        // x, indices, count, g, mean, var, gamma, beta, eps, relu, y
    const Tensor &x = dev(a[0], "x");
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(x, "x");
    PyObject *out = none(a[10]) ? a[0] : a[10];
    const Tensor &y = dev(out, "y", x.scalar_type());
    require(y.sizes() == x.sizes(), "shape of y");
    call(sbnet_sparse_bn_apply, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, l.idx, l.cnt, l.cap, &g, vec(a[4], "mean", s.d), vec(a[5], "var", s.d),
         vec(a[6], "gamma", s.d), vec(a[7], "beta", s.d), f32(a[8]), flag(a[9]), ptr(y), stream());
    return same(out);
}

PyObject *bn_backward(Args a) {                     // x, dy, indices, count, g, mean, var, gamma, beta, eps, relu, dx, workspace
    const Tensor &x = dev(a[0], "x"), &dy = dev(a[1], "dy", x.scalar_type());
    const List l(a[2], a[3]);
    const Geo g(a[4]);
    const Dims4 s(x, "x");
    Tensor fresh;
    if (none(a[11])) fresh = zeros_of(x);
    const Tensor &dx = none(a[11]) ? fresh : dev(a[11], "dx", x.scalar_type());
    require(dy.sizes() == x.sizes() && dx.sizes() == x.sizes(), "shape of dy or dx");
    Tensor own, dgamma = empty({s.d}, x, at::kFloat), dbeta = empty({s.d}, x, at::kFloat);
    size_t wb;
    void *ws = space(a[12], x, sbnet_bn_backward_workspace_bytes(l.cap, s.d), 4, own, &wb);
    call(sbnet_sparse_bn_backward, ptr(x), ptr(dy), dt_of(x), s.a, s.b, s.c, s.d, l.idx, l.cnt, l.cap, &g, vec(a[5], "mean", s.d),
         vec(a[6], "var", s.d), vec(a[7], "gamma", s.d), vec(a[8], "beta", s.d), f32(a[9]), flag(a[10]), ptr(dx), (float *)ptr(dgamma),
         (float *)ptr(dbeta), ws, wb, stream());
    return tuple(give(a[11], fresh), THPVariable_Wrap(dgamma), THPVariable_Wrap(dbeta));
}

PyObject *relu_backward(Args a) {                   // y_tiles, dy_tiles, count, out
    const Tensor &y = dev(a[0], "y_tiles"), &dy = dev(a[1], "dy_tiles", y.scalar_type()), &cnt = dev(a[2], "count", at::kInt);
    require(y.sizes() == dy.sizes(), "shape of dy_tiles");
    Tensor own;
    const Tensor &out = output(a[3], "out", dy.sizes(), dy, y.scalar_type(), own);
    const int cap = (int)y.size(0);
    call(sbnet_relu_backward_on_tiles, ptr(y), ptr(dy), dt_of(y), (const int32_t *)ptr(cnt), cap,
         (size_t)(cap ? y.numel() / cap : 1), ptr(out), stream());
    return give(a[3], own);
}

PyObject *bias_backward(Args a) {                   // dy_tiles, count, workspace
    const Tensor &dy = dev(a[0], "dy_tiles"), &cnt = dev(a[1], "count", at::kInt);
    const Dims4 s(dy, "dy_tiles");
    Tensor own, db = empty({s.d}, dy, at::kFloat);
    size_t wb;
    void *ws = space(a[2], dy, sbnet_bias_backward_workspace_bytes(s.a, s.d), 4, own, &wb);
    call(sbnet_bias_backward_on_tiles, ptr(dy), dt_of(dy), (const int32_t *)ptr(cnt), s.a, s.b * s.c, s.d, (float *)ptr(db), ws, wb, stream());
    return THPVariable_Wrap(db);
}

PyObject *relu_bias_backward(Args a) {              // y_tiles, dy_tiles, count, out, workspace
    const Tensor &y = dev(a[0], "y_tiles"), &dy = dev(a[1], "dy_tiles", y.scalar_type()), &cnt = dev(a[2], "count", at::kInt);
    require(y.sizes() == dy.sizes(), "shape of dy_tiles");
    const Dims4 s(dy, "dy_tiles");
    Tensor oo, own, db = empty({s.d}, dy, at::kFloat);
    const Tensor &out = output(a[3], "out", dy.sizes(), dy, dy.scalar_type(), oo);
    require(out.sizes() == dy.sizes(), "shape of out");
    size_t wb;
    void *ws = space(a[4], dy, sbnet_bias_backward_workspace_bytes(s.a, s.d), 4, own, &wb);
    call(sbnet_relu_bias_backward_on_tiles, ptr(y), ptr(dy), dt_of(y), (const int32_t *)ptr(cnt), s.a, s.b * s.c, s.d, ptr(out),
         (float *)ptr(db), ws, wb, stream());
    return tuple(give(a[3], oo), THPVariable_Wrap(db));
}

PyObject *quantize_f8(Args a) {                     // x, scale, out
    const Tensor &x = dev(a[0], "x");
    Tensor own;
    const Tensor &out = output(a[2], "out", x.sizes(), x, at::kByte, own);
    require(out.sizes() == x.sizes(), "shape of out");
    call(sbnet_quantize_f8, ptr(x), dt_of(x), (size_t)x.numel(), f32(a[1]), (uint8_t *)ptr(out), stream());
    return give(a[2], own);
}

PyObject *conv_f8(Args a) {                         // tiles_f8, count, w_packed, bias, stride, relu, out_scale, out
    const Tensor &t = dev(a[0], "tiles_f8", at::kByte), &cnt = dev(a[1], "count", at::kInt);
    const Packed w(a[2]);
    const Dims4 s(t, "tiles_f8");
    require(s.d == w.cin && w.dtype == at::kByte, "channels or type of the packed weights");
    const int64_t st = i64(a[4]);
    const int64_t sz[4] = {s.a, extent(s.b, w.kh, st), extent(s.c, w.kw, st), w.cout};
    Tensor own;
    const Tensor &out = output(a[7], "out", sz, t, at::kBFloat16, own);
    call(sbnet_conv_on_tiles_f8, (const uint8_t *)ptr(t), (const int32_t *)ptr(cnt), s.a, s.b, s.c, s.d, (const void *)w.buf, bias_of(a[3]),
         w.kh, w.kw, (int)st, (int)st, w.cout, flag(a[5]), f32(a[6]), ptr(out), stream());
    return give(a[7], own);
}

PyObject *conv_on_tiles(Args a) {                   // tiles, count, w_packed, bias, stride, relu, out
    const Tensor &t = dev(a[0], "tiles"), &cnt = dev(a[1], "count", at::kInt);
    const Packed w(a[2]);
    const Dims4 s(t, "tiles");
    require(s.d == w.cin && w.dtype == t.scalar_type(), "channels or type of the packed weights");
    const int64_t st = i64(a[4]);
    const int64_t sz[4] = {s.a, extent(s.b, w.kh, st), extent(s.c, w.kw, st), w.cout};
    Tensor own;
    const Tensor &out = output(a[6], "out", sz, t, t.scalar_type(), own);
    call(sbnet_conv_on_tiles, ptr(t), dt_of(t), (const int32_t *)ptr(cnt), s.a, s.b, s.c, s.d, (const void *)w.buf, bias_of(a[3]), w.kh, w.kw,
         (int)st, (int)st, w.cout, flag(a[5]), ptr(out), stream());
    return give(a[6], own);
}

PyObject *backward_data(Args a) {                   // dout_tiles, count, w_packed_t, th, tw, stride, out, workspace
    const Tensor &d = dev(a[0], "dout_tiles"), &cnt = dev(a[1], "count", at::kInt);
    const Packed w(a[2]);
    const Dims4 s(d, "dout_tiles");
    const int64_t h = i64(a[3]), wd = i64(a[4]), stride = i64(a[5]);
    require(s.d == w.cout && w.dtype == d.scalar_type(), "channels or type of the packed weights");
    require(s.b == extent(h, w.kh, stride) && s.c == extent(wd, w.kw, stride), "shape of dout_tiles");
    const int th = (int)h, tw = (int)wd, st = (int)stride;
    Tensor oo, own;
    const Tensor &out = output(a[6], "out", {s.a, th, tw, w.cin}, d, d.scalar_type(), oo);
    size_t wb;
    void *ws = space(a[7], d, sbnet_conv_backward_data_workspace_bytes(dt_of(d), s.a, th, tw, w.kh, w.kw, st, st, w.cout), 16, own, &wb);
    call(sbnet_conv_on_tiles_backward_data, ptr(d), dt_of(d), (const int32_t *)ptr(cnt), s.a, th, tw, w.cin, (const void *)w.buf, w.kh, w.kw,
         st, st, w.cout, ptr(out), ws, wb, stream());
    return give(a[6], oo);
}

PyObject *backward_weights(Args a) {                // tiles, dout_tiles, count, k, stride, out, workspace
    const Tensor &t = dev(a[0], "tiles"), &d = dev(a[1], "dout_tiles", t.scalar_type()), &cnt = dev(a[2], "count", at::kInt);
    const Dims4 s(t, "tiles"), o(d, "dout_tiles");
    const int64_t side = i64(a[3]), stride = i64(a[4]);
    require(o.a == s.a && o.b == extent(s.b, side, stride) && o.c == extent(s.c, side, stride), "shape of dout_tiles");
    const int k = (int)side, st = (int)stride;
    Tensor oo, own;
    const Tensor &out = output(a[5], "out", {k, k, s.d, o.d}, t, at::kFloat, oo);
    require(Dims4(out, "out").is(k, k, s.d, o.d), "shape of out");
    size_t wb;
    void *ws = space(a[6], t, sbnet_conv_backward_weights_workspace_bytes(dt_of(t), s.a, s.b, s.c, s.d, k, k, st, st, o.d), 16, own, &wb);
    call(sbnet_conv_on_tiles_backward_weights, ptr(t), ptr(d), dt_of(t), (const int32_t *)ptr(cnt), s.a, s.b, s.c, s.d, k, k, st, st, o.d,
         (float *)ptr(out), ws, wb, stream());
    return give(a[5], oo);
}

PyObject *sparse_conv(Args a) {                     // x, indices, count, g_in, g_out, w_packed, bias, y, stride, relu, add
    const Tensor &x = dev(a[0], "x"), &y = dev(a[7], "y", x.scalar_type());
    const List l(a[1], a[2]);
    const Geo gi(a[3]), go(a[4]);
    const Packed w(a[5]);
    const Dims4 s(x, "x"), o(y, "y");
    require(s.d == w.cin && w.dtype == x.scalar_type(), "channels or type of the packed weights");
    require(o.a == s.a && o.d == w.cout, "shape of y");
    const int st = i32(a[8]);
    call(sbnet_sparse_conv, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, l.idx, l.cnt, l.cap, &gi, &go, (const void *)w.buf, bias_of(a[6]), w.kh, w.kw,
         st, st, w.cout, flag(a[9]), ptr(y), o.b, o.c, flag(a[10]), stream());
    return same(a[7]);
}

PyObject *block_flags(Args a) {                     // mask, g, pool, threshold, flags
    const Tensor &mask = dev(a[0], "mask");
    if (mask.dim() != 3) raise(PyExc_ValueError, "mask must have three dimensions");
    const Geo g(a[1]);
    Tensor own;
    const Tensor &f = output(a[4], "flags", {(int64_t)sbnet_block_flags_bytes((int)mask.size(0), &g)}, mask, at::kByte, own);
    call(sbnet_block_flags, ptr(mask), dt_of(mask), (int)mask.size(0), (int)mask.size(1), (int)mask.size(2), &g, (sbnet_pool)i32(a[2]),
         f32(a[3]), (uint8_t *)ptr(f), (size_t)f.numel(), stream());
    return give(a[4], own);
}

PyObject *conv_from_flags(Args a) {                 // flags, x, g_in, g_out, w_packed, bias, y, indices, count, stride, relu, add
    const Tensor &f = dev(a[0], "flags", at::kByte), &x = dev(a[1], "x"), &y = dev(a[6], "y", x.scalar_type());
    const List l(a[7], a[8]);
    const Geo gi(a[2]), go(a[3]);
    const Packed w(a[4]);
    const Dims4 s(x, "x"), o(y, "y");
    require(s.d == w.cin && w.dtype == x.scalar_type(), "channels or type of the packed weights");
    require(o.a == s.a && o.d == w.cout && (size_t)f.numel() >= sbnet_block_flags_bytes(s.a, &gi), "shape of y or flags");
    const int st = i32(a[9]);
    call(sbnet_sparse_conv_from_flags, (const uint8_t *)ptr(f), ptr(x), dt_of(x), s.a, s.b, s.c, s.d, (int32_t *)l.idx, (int32_t *)l.cnt, l.cap,
         &gi, &go, (const void *)w.buf, bias_of(a[5]), w.kh, w.kw, st, st, w.cout, flag(a[10]), ptr(y), o.b, o.c, flag(a[11]), stream());
    return same(a[6]);
}

// mask, g_mask, x, g_in, g_out, w_packed, bias, y, indices, count, workspace, pool, threshold, stride, relu, add
PyObject *conv_from_mask(Args a) {
    const Tensor &m = dev(a[0], "mask"), &x = dev(a[2], "x"), &y = dev(a[7], "y", x.scalar_type()), &ws = dev(a[10], "workspace");
    if (m.dim() != 3) raise(PyExc_ValueError, "mask must have three dimensions");
    const List l(a[8], a[9]);
    const Geo gm(a[1]), gi(a[3]), go(a[4]);
    const Packed w(a[5]);
    const Dims4 s(x, "x"), o(y, "y");
    require(s.d == w.cin && w.dtype == x.scalar_type() && m.size(0) == s.a, "channels or type of the packed weights, or samples of the mask");
    require(o.a == s.a && o.d == w.cout, "shape of y");
    const int st = i32(a[13]);
    call(sbnet_sparse_conv_from_mask, ptr(m), dt_of(m), (int)m.size(1), (int)m.size(2), &gm, (sbnet_pool)i32(a[11]), f32(a[12]), ptr(x),
         dt_of(x), s.a, s.b, s.c, s.d, (int32_t *)l.idx, (int32_t *)l.cnt, l.cap, &gi, &go, (const void *)w.buf, bias_of(a[6]), w.kh, w.kw, st, st,
         w.cout, flag(a[14]), ptr(y), o.b, o.c, flag(a[15]), ptr(ws), (size_t)ws.numel() * ws.element_size(), stream());
    return same(a[7]);
}

// (w1, b1, w2, b2, w3, b3) of a residual unit; biases of the widths given
struct Unit {
    Several it;
    void *w[3];
    float *b[3];
    int cin, cm, cout;
    Unit(PyObject *o, bool need_bias) : it(o, 6, "weights must be (w1, b1, w2, b2, w3, b3)") {
        const Packed w1(it[0]), w2(it[2]), w3(it[4]);
        cin = w1.cin; cm = w1.cout; cout = w3.cout;
        require(w2.is(3, 3, cm, cm) && w3.kh == 1 && w3.kw == 1 && w3.cin == cm, "shapes of the unit's weights");
        w[0] = w1.buf; w[1] = w2.buf; w[2] = w3.buf;
        const int n[3] = {cm, cm, cout};
        for (int i = 0; i < 3; ++i) {
            if (!need_bias && none(it[2 * i + 1])) { b[i] = nullptr; continue; }
            const Tensor &t = dev(it[2 * i + 1], "bias", at::kFloat);
            require(!need_bias || t.numel() == n[i], "bias");
            b[i] = (float *)ptr(t);
        }
    }
};

struct Pre {                                        // (scale, shift) or None
    std::optional<Several> it;
    const float *scale = nullptr, *shift = nullptr;
    Pre(PyObject *o, int C) {
        if (none(o)) return;
        it.emplace(o, 2, "pre must be (scale, shift)");
        const Tensor &a = dev((*it)[0], "pre_scale", at::kFloat);
        const Tensor &b = dev((*it)[1], "pre_shift", at::kFloat);
        require(a.numel() == C && b.numel() == C, "pre_scale or pre_shift");
        scale = (const float *)ptr(a);
        shift = (const float *)ptr(b);
    }
};

PyObject *bottleneck_on_tiles(Args a) {             // tiles, indices, count, g_in, g_out, H, W, weights, out, pre
    const Tensor &t = dev(a[0], "tiles");
    const List l(a[1], a[2]);
    const Geo gi(a[3]), go(a[4]);
    const Unit u(a[7], true);
    require(u.cout == u.cin, "shapes of the unit's weights");
    require(Dims4(t, "tiles").is(l.cap, gi.bsize_h, gi.bsize_w, u.cin), "shape of tiles");
    const Pre pre(a[9], u.cin);
    Tensor own;
    const Tensor &out = output(a[8], "out", {l.cap, go.bsize_h, go.bsize_w, u.cin}, t, t.scalar_type(), own);
    const int H = i32(a[5]), W = i32(a[6]);
    if (pre.scale)
        call(sbnet_bottleneck_on_tiles_preact, ptr(t), dt_of(t), H, W, u.cin, u.cm, l.idx, l.cnt, l.cap, &gi, &go, pre.scale, pre.shift,
             (const void *)u.w[0], u.b[0], (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], ptr(out), stream());
    else
        call(sbnet_bottleneck_on_tiles, ptr(t), dt_of(t), H, W, u.cin, u.cm, l.idx, l.cnt, l.cap, &gi, &go, (const void *)u.w[0], u.b[0],
             (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], ptr(out), stream());
    return give(a[8], own);
}

PyObject *sparse_bottleneck(Args a) {               // x, indices, count, g_in, g_out, weights, y, pre
    const Tensor &x = dev(a[0], "x"), &y = dev(a[6], "y", x.scalar_type());
    const List l(a[1], a[2]);
    const Geo gi(a[3]), go(a[4]);
    const Unit u(a[5], true);
    const Dims4 s(x, "x");
    require(u.cout == u.cin && s.d == u.cin && y.sizes() == x.sizes(), "shapes of the unit's weights or of y");
    const Pre pre(a[7], u.cin);
    if (pre.scale)
        call(sbnet_sparse_bottleneck_preact, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, u.cm, l.idx, l.cnt, l.cap, &gi, &go, pre.scale, pre.shift,
             (const void *)u.w[0], u.b[0], (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], ptr(y), stream());
    else
        call(sbnet_sparse_bottleneck, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, u.cm, l.idx, l.cnt, l.cap, &gi, &go, (const void *)u.w[0], u.b[0],
             (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], ptr(y), stream());
    return same(a[6]);
}

PyObject *sparse_unit(Args a) {                     // x, indices, count, g_in, g_out, weights, y, stride, shortcut, workspace
    const Tensor &x = dev(a[0], "x"), &y = dev(a[6], "y", x.scalar_type());
    const List l(a[1], a[2]);
    const Geo gi(a[3]), go(a[4]);
    const Unit u(a[5], true);
    const Dims4 s(x, "x"), o(y, "y");
    require(s.d == u.cin && o.d == u.cout && o.a == s.a, "shapes of the unit's weights, x or y");
    void *ws = nullptr;
    float *bs = nullptr;
    std::optional<Several> sc;
    if (!none(a[8])) {
        sc.emplace(a[8], 2, "shortcut must be (weights, bias)");
        if (!none((*sc)[0])) {
            const Packed p((*sc)[0]);
            const Tensor &b = dev((*sc)[1], "shortcut bias", at::kFloat);
            require(p.is(1, 1, u.cin, u.cout) && b.numel() == u.cout, "shapes of the shortcut");
            ws = p.buf;
            bs = (float *)ptr(b);
        }
    }
    Tensor own;
    size_t wb;
    void *work = space(a[9], x, none(a[9]) ? sbnet_sparse_unit_workspace_bytes(dt_of(x), l.cap, &gi, &go, u.cin, u.cm, u.cout) : 0, 256, own,
                       &wb, true);
    call(sbnet_sparse_unit, ptr(x), dt_of(x), s.a, s.b, s.c, s.d, u.cm, u.cout, i32(a[7]), l.idx, l.cnt, l.cap, &gi, &go, (const void *)u.w[0],
         u.b[0], (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], (const void *)ws, bs, ptr(y), o.b, o.c, work, wb, stream());
    return same(a[6]);
}

PyObject *zero_outside(Args a) {                    // tiles, indices, count, g, H, W
    const Tensor &t = dev(a[0], "tiles");
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Dims4 s(t, "tiles");
    require(s.is(l.cap, g.bsize_h, g.bsize_w, s.d), "shape of tiles");
    call(sbnet_zero_outside, ptr(t), dt_of(t), i32(a[4]), i32(a[5]), s.d, l.idx, l.cnt, l.cap, &g, stream());
    return same(a[0]);
}

PyObject *forward_keep(Args a) {                    // tiles, indices, count, g_in, H, W, weights
    const Tensor &t = dev(a[0], "tiles");
    const List l(a[1], a[2]);
    const Geo g(a[3]);
    const Unit u(a[6], false);
    const Dims4 s(t, "tiles");
    require(s.b == g.bsize_h && s.c == g.bsize_w && s.a == l.cap, "shape of tiles");
    Tensor t1 = empty({s.a, s.b, s.c, u.cm}, t, t.scalar_type()), t2 = empty({s.a, s.b - 2, s.c - 2, u.cm}, t, t.scalar_type()),
           t3 = empty({s.a, s.b - 2, s.c - 2, s.d}, t, t.scalar_type());
    call(sbnet_bottleneck_forward_keep_on_tiles, ptr(t), dt_of(t), i32(a[4]), i32(a[5]), s.d, u.cm, l.idx, l.cnt, l.cap, &g,
         (const void *)u.w[0], u.b[0], (const void *)u.w[1], u.b[1], (const void *)u.w[2], u.b[2], ptr(t1), ptr(t2), ptr(t3), stream());
    return tuple(THPVariable_Wrap(t1), THPVariable_Wrap(t2), THPVariable_Wrap(t3));
}

PyObject *unit_backward(Args a) {                   // tiles, t1, t2, dt3, count, weights_t, workspace
    const Tensor &t = dev(a[0], "tiles"), &t1 = dev(a[1], "t1", t.scalar_type()), &t2 = dev(a[2], "t2", t.scalar_type()),
                 &d = dev(a[3], "dt3", t.scalar_type()), &cnt = dev(a[4], "count", at::kInt);
    const Dims4 s(t, "tiles");
    const int Cm = (int)Dims4(t1, "t1").d;
    require(Dims4(t1, "t1").is(s.a, s.b, s.c, Cm) && Dims4(t2, "t2").is(s.a, s.b - 2, s.c - 2, Cm) &&
                Dims4(d, "dt3").is(s.a, s.b - 2, s.c - 2, s.d), "shape of t1, t2 or dt3");
    const Several it(a[5], 3, "weights_t must be (w1_t, w2_t, w3_t)");
    const Packed w1(it[0]), w2(it[1]), w3(it[2]);
    require(w1.is(1, 1, s.d, Cm) && w2.is(3, 3, Cm, Cm) && w3.is(1, 1, Cm, s.d), "shapes of the transposed weights");
    Tensor own, dx = empty(t.sizes(), t, t.scalar_type());
    size_t wb;
    void *ws = space(a[6], t, sbnet_bottleneck_backward_workspace_bytes(dt_of(t), s.a, s.b, s.c, s.d, Cm), 256, own, &wb);
    Tensor dw1 = empty({1, 1, s.d, Cm}, t, at::kFloat), db1 = empty({Cm}, t, at::kFloat), dw2 = empty({3, 3, Cm, Cm}, t, at::kFloat),
           db2 = empty({Cm}, t, at::kFloat), dw3 = empty({1, 1, Cm, s.d}, t, at::kFloat), db3 = empty({s.d}, t, at::kFloat);
    auto f = [](const Tensor &x) { return (float *)ptr(x); };
    call(sbnet_bottleneck_backward_on_tiles, ptr(t), ptr(t1), ptr(t2), ptr(d), dt_of(t), (const int32_t *)ptr(cnt), s.a, s.b, s.c, s.d, Cm,
         (const void *)w1.buf, (const void *)w2.buf, (const void *)w3.buf, ptr(dx), f(dw1), f(db1), f(dw2), f(db2), f(dw3), f(db3), ws, wb,
         stream());
    return tuple(THPVariable_Wrap(dx), THPVariable_Wrap(dw1), THPVariable_Wrap(db1), THPVariable_Wrap(dw2), THPVariable_Wrap(db2),
                 THPVariable_Wrap(dw3), THPVariable_Wrap(db3));
}

PyObject *set_types(Args a) {                       // SbnetError, Geom
    Py_XSETREF(g_error, same(a[0]));
    Py_XSETREF(g_geom, same(a[1]));
    Py_RETURN_NONE;
}

// ---- module ------------------------------------------------------------------------------------------------------
template <PyObject *(*F)(Args), int N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (python_error &e) {
        e.restore();
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

#define CALL(name, fn, n) {name, (PyCFunction)(void (*)(void))entry<fn, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    CALL("set_types", set_types, 2),
    CALL("reduce_mask", reduce_mask, 7),
    CALL("reduce_mask_static", reduce_mask_static, 6),
    CALL("sparse_gather", gather<false>, 5),
    CALL("sparse_gather_chw", gather<true>, 5),
    CALL("sparse_scatter", scatter<false>, 6),
    CALL("sparse_scatter_chw", scatter<true>, 6),
    CALL("sparse_gather_backward", gather_backward, 6),
    CALL("sparse_bn_stats", bn_stats, 5),
    CALL("sparse_bn_apply", bn_apply, 11),
    CALL("sparse_bn_backward", bn_backward, 13),
    CALL("relu_backward_on_tiles", relu_backward, 4),
    CALL("bias_backward_on_tiles", bias_backward, 3),
    CALL("relu_bias_backward_on_tiles", relu_bias_backward, 5),
    CALL("quantize_f8", quantize_f8, 3),
    CALL("conv_on_tiles_f8", conv_f8, 8),
    CALL("conv_on_tiles", conv_on_tiles, 7),
    CALL("conv_on_tiles_backward_data", backward_data, 8),
    CALL("conv_on_tiles_backward_weights", backward_weights, 7),
    CALL("sparse_conv", sparse_conv, 11),
    CALL("block_flags", block_flags, 5),
    CALL("sparse_conv_from_flags", conv_from_flags, 12),
    CALL("sparse_conv_from_mask", conv_from_mask, 16),
    CALL("bottleneck_on_tiles", bottleneck_on_tiles, 10),
    CALL("sparse_bottleneck", sparse_bottleneck, 8),
    CALL("sparse_unit", sparse_unit, 10),
    CALL("zero_outside", zero_outside, 6),
    CALL("bottleneck_forward_keep_on_tiles", forward_keep, 7),
    CALL("bottleneck_backward_on_tiles", unit_backward, 7),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", "Calls of the library on torch tensors.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__torch_calls() {
    s_buf = PyUnicode_InternFromString("buf");
    s_shape = PyUnicode_InternFromString("shape");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_contents = PyUnicode_InternFromString("contents");
    s_obj = PyUnicode_InternFromString("_obj");
    return PyModule_Create(&module);
}
