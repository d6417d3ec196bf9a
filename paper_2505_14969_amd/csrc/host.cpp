// The binding's work on a call: arguments checked, results allocated, sizes and pointers handed to the C ABI of
// include/stree.h.  Nothing of the path is computed here.
//
// A decoding step on a small tree takes the GPU 15 us, and the same work in Python (some thirty attribute look-ups and
// conversions a call) took the CPU 14 us of it beside 10 us in the library: a step of 15 nodes with its gate 25.7 us a
// pass, now 16.4, verification of 15 fp32 nodes in three calls 26.8 -> 15.7.  binding.py keeps the functions, their arguments and defaults; each passes its arguments here by
// position.  The library stays the one that binding.load() opened: bind() takes the entry points' addresses from it.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <memory>
#include <vector>

#include "../../include/stree.h"

namespace {

struct Entry {
    decltype(&stree_tree_conv) tree_conv;
    decltype(&stree_tree_ssd) tree_ssd;
    decltype(&stree_commit_state) commit_state;
    decltype(&stree_tree_ssd_replay) tree_ssd_replay;
    decltype(&stree_tree_conv_replay) tree_conv_replay;
    decltype(&stree_tree_step) tree_step;
    decltype(&stree_gate_norm) gate_norm;
    decltype(&stree_linear_ssd) linear_ssd;
};

// A Python exception is set: leave the call.
struct Raised {};
[[noreturn]] void raise(PyObject *type, const char *text) {
    PyErr_SetString(type, text);
    throw Raised{};
}
void require(bool ok, const char *text) {
    if (!ok) raise(PyExc_AssertionError, text);
}

bool truth(PyObject *o) {
    const int t = PyObject_IsTrue(o);
    if (t < 0) throw Raised{};
    return t != 0;
}
// A Python object of our own.
struct Owned {
    PyObject *o;
    explicit Owned(PyObject *made) : o(made) {
        if (!o) throw Raised{};
    }
    Owned(const Owned &) = delete;
    ~Owned() { Py_DECREF(o); }
};
// The arguments of a call, and whether somebody listens to what is called on tensors (asked for once a call: it costs as much
// as reading a size).
struct Arg {
    PyObject *o;
    bool heard;
    operator PyObject *() const { return o; }
    // A tensor that is read, and results made like it, without a detour through Python: no subclass, whose methods may be
    // somebody's own.
    bool plain() const { return THPVariable_CheckExact(o) && !heard; }
};
struct Args {
    PyObject *const *v;
    bool heard;
    Arg operator[](int i) const { return {v[i], heard}; }
    Arg none() const { return {Py_None, heard}; }
};

// An array argument: a plain tensor, or whatever its Python attributes say it is (shape, stride(), dtype, is_contiguous(),
// numel(), element_size(), data_ptr()).
class Array {
  public:
    explicit Array(Arg a) : o(a.o), t(a.plain() ? &THPVariable_Unpack(a.o) : nullptr) {}
    at::IntArrayRef sizes() const {
        if (t) return t->sizes();
        if (!size_) size_ = numbers(Owned(PyObject_GetAttrString(o, "shape")).o);
        return *size_;
    }
    at::IntArrayRef strides() const {
        if (t) return t->strides();
        if (!stride_) stride_ = numbers(Owned(PyObject_CallMethod(o, "stride", nullptr)).o);
        return *stride_;
    }
    int64_t dim() const { return (int64_t)sizes().size(); }
    int64_t size(int64_t i) const {
        if (i >= dim()) raise(PyExc_IndexError, "tuple index out of range");
        return sizes()[i];
    }
    bool shaped(std::initializer_list<int64_t> size) const { return sizes() == at::IntArrayRef(size); }
    bool is_contiguous() const { return t ? t->is_contiguous() : truth(Owned(PyObject_CallMethod(o, "is_contiguous", nullptr)).o); }
    int64_t numel() const { return t ? t->numel() : number("numel"); }
    int64_t element_size() const { return t ? t->element_size() : number("element_size"); }
    void *data_ptr() const {
        if (t) return t->data_ptr();
        const Owned p(PyObject_CallMethod(o, "data_ptr", nullptr));
        void *v = p.o == Py_None ? nullptr : PyLong_AsVoidPtr(p.o);
        if (!v && PyErr_Occurred()) throw Raised{};
        return v;
    }
    // (Undefined: a type that torch does not know)
    at::ScalarType type() const {
        if (t) return t->scalar_type();
        const Owned d(PyObject_GetAttrString(o, "dtype"));
        return THPDtype_Check(d.o) ? reinterpret_cast<THPDtype *>(d.o)->scalar_type : at::ScalarType::Undefined;
    }
    bool same_type(const Array &b) const { return type() == b.type() && type() != at::ScalarType::Undefined; }

  private:
    typedef std::unique_ptr<std::vector<int64_t>> Numbers;
    static Numbers numbers(PyObject *sequence) {
        const Owned f(PySequence_Fast(sequence, "a sequence of sizes"));
        Numbers v(new std::vector<int64_t>(PySequence_Fast_GET_SIZE(f.o)));
        for (size_t i = 0; i < v->size(); ++i) {
            (*v)[i] = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(f.o, (Py_ssize_t)i));
            if ((*v)[i] == -1 && PyErr_Occurred()) throw Raised{};
        }
        return v;
    }
    int64_t number(const char *method) const {
        const int64_t v = PyLong_AsLongLong(Owned(PyObject_CallMethod(o, method, nullptr)).o);
        if (v == -1 && PyErr_Occurred()) throw Raised{};
        return v;
    }
    PyObject *o;
    const at::Tensor *t;
    mutable Numbers size_, stride_;
};
void *pointer(Arg a) { return a.o == Py_None ? nullptr : a.plain() ? THPVariable_Unpack(a.o).data_ptr() : Array(a).data_ptr(); }
// An int, or what gives one as an index (numpy's), as far as 64 bits reach: the checks see the whole value.
int64_t integer(PyObject *o) {
    PyObject *i = PyNumber_Index(o);
    if (!i) throw Raised{};
    int beyond = 0;
    const long long v = PyLong_AsLongLongAndOverflow(i, &beyond);
    Py_DECREF(i);
    return beyond > 0 ? INT64_MAX : beyond < 0 ? INT64_MIN : v;
}
// channels of a row: x, then B and C of every group
bool channels_are(int64_t channels, int64_t heads, int64_t headdim, int64_t dstate, int64_t groups) {
    int64_t x, bc;
    return !__builtin_mul_overflow(heads, headdim, &x) && !__builtin_mul_overflow(groups, dstate, &bc) &&
           !__builtin_mul_overflow(bc, (int64_t)2, &bc) && !__builtin_add_overflow(x, bc, &x) && x == channels;
}
void dimensions(const Array &t, int n) {
    if (t.dim() != n) {
        PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions is expected, not %d", n, (int)t.dim());
        throw Raised{};
    }
}
int type_code(const Array &t) {
    const auto type = t.type();
    if (type == at::kFloat) return STREE_F32;
    if (type == at::kBFloat16) return STREE_BF16;
    raise(PyExc_TypeError, "unsupported dtype");
}
// ... of the rows, which are torch's
int rows_code(Arg a) {
    if (!a.plain() && !THPVariable_Check(a.o)) raise(PyExc_TypeError, "unsupported dtype");
    return type_code(Array(a));
}
// type of the SSM state from the state tensors of a call (those that are given must agree)
int state_code(Arg h0, Arg h_out) {
    if (h0.o == Py_None) return h_out.o == Py_None ? STREE_F32 : type_code(Array(h_out));
    const Array h(h0);
    require(h_out.o == Py_None || h_out.o == h0.o || Array(h_out).same_type(h), "h0 and h_out must have the same dtype");
    return type_code(h);
}
// Element stride between tokens of a [B,N,a,b] view whose last two dims are dense and whose batch stride is N * token
// stride.
int64_t token_stride(const Array &t, int64_t nnodes) {
    require(t.dim() == 4, "inner dims must be dense");
    const at::IntArrayRef size = t.sizes(), stride = t.strides();
    require(stride.size() == 4, "inner dims must be dense");
    require(stride[3] == 1 && stride[2] == size[3], "inner dims must be dense");
    // (the stride torch keeps for a dimension of size 1 means nothing)
    const int64_t sn = nnodes == 1 && size[0] > 1 ? stride[0] : stride[1];
    require(size[0] == 1 || stride[0] == nnodes * sn, "batch stride must be N * token stride");
    return sn;
}

stree_dims make_dims(int64_t batch, int64_t nnodes, int64_t heads, int64_t headdim, int64_t dstate, int64_t groups, int64_t width,
                     int io, int state, int flags, Arg dt_bias) {
    stree_dims d = {};
    d.batch = (int32_t)batch, d.nnodes = (int32_t)nnodes, d.nheads = (int32_t)heads, d.headdim = (int32_t)headdim;
    d.dstate = (int32_t)dstate, d.ngroups = (int32_t)groups, d.conv_width = (int32_t)width;
    d.io_dtype = io, d.state_dtype = state, d.flags = flags;
    if (dt_bias.o != Py_None) {
        const Array b(dt_bias);
        require(b.type() == at::kFloat && b.is_contiguous() && b.numel() == heads, "dt_bias must be fp32 [H], contiguous");
        d.flags |= STREE_FLAG_DT_SOFTPLUS;
        d.dt_bias = static_cast<const float *>(b.data_ptr());
    }
    return d;
}

// A result: `given`, or what torch.empty_like(o) makes (through Python where something there may want to see it).
struct Result {
    PyObject *o = nullptr;
    bool heard = false;
    ~Result() { Py_XDECREF(o); }
    Arg arg() const { return {o, heard}; }
    Array t() const { return Array(arg()); }
    void *ptr() const { return pointer(arg()); }
    bool keep(Arg given) {
        heard = given.heard;
        if (given.o == Py_None) return false;
        Py_INCREF(given.o);
        o = given.o;
        return true;
    }
    void none() { keep_none(); }
    PyObject *release() {
        PyObject *r = o;
        o = nullptr;
        return r;
    }

  private:
    void keep_none() {
        Py_INCREF(Py_None);
        o = Py_None;
    }
};
void like(Result &r, Arg given, Arg model) {
    if (r.keep(given)) return;
    if (model.plain()) {
        r.o = THPVariable_Wrap(at::empty_like(THPVariable_Unpack(model.o)));
    } else {
        PyObject *torch = PyImport_ImportModule("torch");
        r.o = torch ? PyObject_CallMethod(torch, "empty_like", "O", model.o) : nullptr;
        Py_XDECREF(torch);
    }
    if (!r.o) throw Raised{};
}
// ... what model.new_empty(size) makes, in the type of `typed` (fp32 where that is None)
void sized(Result &r, Arg given, Arg model, std::initializer_list<int64_t> size, Arg typed) {
    if (r.keep(given)) return;
    const auto type = typed.o == Py_None ? at::kFloat : Array(typed).type();
    if (model.plain() && type != at::ScalarType::Undefined) {
        r.o = THPVariable_Wrap(at::empty(at::IntArrayRef(size), THPVariable_Unpack(model.o).options().dtype(type).requires_grad(false)));
    } else {
        PyObject *torch = PyImport_ImportModule("torch"), *dtype = nullptr, *shape = nullptr, *kw = nullptr, *args = nullptr, *f = nullptr;
        if (torch) dtype = typed.o == Py_None ? PyObject_GetAttrString(torch, "float32") : PyObject_GetAttrString(typed.o, "dtype");
        shape = PyTuple_New((Py_ssize_t)size.size());
        Py_ssize_t i = 0;
        for (int64_t n : size) PyTuple_SET_ITEM(shape, i++, PyLong_FromLongLong(n));
        if (dtype) kw = Py_BuildValue("{s:O}", "dtype", dtype);
        args = Py_BuildValue("(O)", shape);
        if (kw) f = PyObject_GetAttrString(model.o, "new_empty");
        if (f) r.o = PyObject_Call(f, args, kw);
        Py_XDECREF(f), Py_XDECREF(args), Py_XDECREF(kw), Py_XDECREF(shape), Py_XDECREF(dtype), Py_XDECREF(torch);
    }
    if (!r.o) throw Raised{};
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

PyObject *g_error = nullptr;           // binding.StreeError
Entry g_entry = {};

template <typename Call>
void run(const char *where, Call &&call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    if (rc == STREE_OK) return;
    PyObject *e = PyObject_CallFunction(g_error, "is", rc, where);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Raised{};
}
PyObject *pair(Result &a, Result &b) {
    PyObject *t = PyTuple_Pack(2, a.o, b.o);
    return t;
}

PyObject *conv(const Args &a) {
    enum { parent, xbc_pre, conv_state, conv_w, conv_b, nheads, headdim, dstate, ngroups, silu, out, status };
    const Array x(a[xbc_pre]), w(a[conv_w]);
    dimensions(x, 3);
    const int64_t B = x.size(0), N = x.size(1), Cc = x.size(2), W = w.size(1);
    const int64_t H = integer(a[nheads]), P = integer(a[headdim]), S = integer(a[dstate]), G = integer(a[ngroups]);
    require(channels_are(Cc, H, P, S, G), "channels of xbc_pre");
    require(x.is_contiguous() && Array(a[conv_state]).is_contiguous() && w.is_contiguous(), "contiguous rows");
    Result y;
    like(y, a[out], a[xbc_pre]);
    const stree_dims d = make_dims(B, N, H, P, S, G, W, rows_code(a[xbc_pre]), STREE_F32, truth(a[silu]) ? STREE_FLAG_CONV_SILU : 0, a.none());
    const auto p0 = (const int32_t *)pointer(a[parent]);
    const void *p1 = pointer(a[xbc_pre]), *p2 = pointer(a[conv_state]), *p3 = pointer(a[conv_w]), *p4 = pointer(a[conv_b]);
    void *p5 = y.ptr(), *st = stream();
    const auto p6 = (int32_t *)pointer(a[status]);
    run("stree_tree_conv", [&] { return g_entry.tree_conv(&d, p0, p1, p2, p3, p4, p5, p6, st); });
    return y.release();
}

PyObject *ssd(const Args &a) {
    enum { parent, x, dt, A, Bm, Cm, D, h0, out, status, force_fma, general_mfma, dt_bias };
    const Array tx(a[x]), tb(a[Bm]), tc(a[Cm]);
    dimensions(tx, 4);
    require(tb.dim() == 4, "inner dims must be dense");
    const int64_t B = tx.size(0), N = tx.size(1), H = tx.size(2), P = tx.size(3), G = tb.size(2), S = tb.size(3);
    Result y;
    sized(y, a[out], a[x], {B, N, H, P}, a[x]);
    stree_dims d = make_dims(B, N, H, P, S, G, 0, rows_code(a[x]), state_code(a[h0], a.none()),
                             (truth(a[force_fma]) ? STREE_FLAG_FORCE_FMA : 0) | (truth(a[general_mfma]) ? STREE_FLAG_GENERAL_MFMA : 0), a[dt_bias]);
    d.x_stride_n = token_stride(tx, N), d.b_stride_n = token_stride(tb, N), d.c_stride_n = token_stride(tc, N);
    const Array td(a[dt]);
    require(td.is_contiguous() && td.type() == at::kFloat && y.t().is_contiguous(), "dt fp32, dense; out dense");
    const auto p0 = (const int32_t *)pointer(a[parent]);
    const void *p1 = pointer(a[x]), *p4 = pointer(a[Bm]), *p5 = pointer(a[Cm]), *p7 = pointer(a[h0]);
    const auto p2 = (const float *)pointer(a[dt]), p3 = (const float *)pointer(a[A]), p6 = (const float *)pointer(a[D]);
    void *p8 = y.ptr(), *st = stream();
    const auto p9 = (int32_t *)pointer(a[status]);
    run("stree_tree_ssd", [&] { return g_entry.tree_ssd(&d, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, st); });
    return y.release();
}

PyObject *commit(const Args &a) {
    enum { parent, accepted, x, dt, A, Bm, h0, h_out, xbc_pre, conv_state, conv_state_out, status, dims, dt_bias };
    Result h, cs;
    stree_dims d;
    if (a[x] == Py_None) {                            // the conv tail alone; `dims` names the head shapes
        const Array tp(a[parent]);
        dimensions(tp, 2);
        int64_t shape[4];
        Result s;
        s.o = PySequence_Fast(a[dims], "dims = (H, P, S, G)");
        if (!s.o) throw Raised{};
        if (PySequence_Fast_GET_SIZE(s.o) != 4) raise(PyExc_ValueError, "dims = (H, P, S, G)");
        for (int i = 0; i < 4; ++i) shape[i] = integer(PySequence_Fast_GET_ITEM(s.o, i));
        like(cs, a[conv_state_out], a[conv_state]);
        d = make_dims(tp.size(0), tp.size(1), shape[0], shape[1], shape[2], shape[3], Array(a[conv_state]).size(1) + 1,
                      rows_code(a[xbc_pre]), STREE_F32, 0, a.none());
        h.none();
        const auto p0 = (const int32_t *)pointer(a[parent]), p1 = (const int32_t *)pointer(a[accepted]);
        const void *p2 = pointer(a[xbc_pre]), *p3 = pointer(a[conv_state]);
        void *p4 = cs.ptr(), *st = stream();
        const auto p5 = (int32_t *)pointer(a[status]);
        run("stree_commit_state", [&] {
            return g_entry.commit_state(&d, p0, p1, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, p2, p3, p4, p5, st);
        });
        return pair(h, cs);
    }
    const Array tx(a[x]), tb(a[Bm]);
    dimensions(tx, 4);
    require(tb.dim() == 4, "inner dims must be dense");
    const int64_t B = tx.size(0), N = tx.size(1), H = tx.size(2), P = tx.size(3), G = tb.size(2), S = tb.size(3);
    sized(h, a[h_out], a[x], {B, H, P, S}, a[h0]);
    int64_t W = 0;
    if (a[xbc_pre] != Py_None) {
        W = Array(a[conv_state]).size(1) + 1;
        like(cs, a[conv_state_out], a[conv_state]);
    } else if (!cs.keep(a[conv_state_out])) {
        cs.none();
    }
    d = make_dims(B, N, H, P, S, G, W, rows_code(a[x]), state_code(a[h0], h.arg()), 0, a[dt_bias]);
    d.x_stride_n = token_stride(tx, N), d.b_stride_n = token_stride(tb, N);
    const auto p0 = (const int32_t *)pointer(a[parent]), p1 = (const int32_t *)pointer(a[accepted]);
    const void *p2 = pointer(a[x]), *p5 = pointer(a[Bm]), *p6 = pointer(a[h0]), *p8 = pointer(a[xbc_pre]), *p9 = pointer(a[conv_state]);
    const auto p3 = (const float *)pointer(a[dt]), p4 = (const float *)pointer(a[A]);
    void *p7 = h.ptr(), *p10 = cs.ptr(), *st = stream();
    const auto p11 = (int32_t *)pointer(a[status]);
    run("stree_commit_state", [&] { return g_entry.commit_state(&d, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, p10, p11, st); });
    return pair(h, cs);
}

PyObject *ssd_replay(const Args &a) {
    enum { pparent, paccepted, px, pdt, pBm, parent, x, dt, A, Bm, Cm, D, h0, h_out, out, status, rstatus, force_fma, dt_bias };
    const Array tx(a[x]), tb(a[Bm]), tc(a[Cm]), tpx(a[px]), tpb(a[pBm]);
    const Array tpd(a[pdt]), td(a[dt]), th(a[h0]);
    dimensions(tx, 4);
    require(tb.dim() == 4 && tpx.dim() == 4, "inner dims must be dense");
    const int64_t B = tx.size(0), N = tx.size(1), H = tx.size(2), P = tx.size(3), G = tb.size(2), S = tb.size(3), Np = tpx.size(1);
    require(tpx.shaped({B, Np, H, P}) && tpb.shaped({B, Np, G, S}) && tpx.same_type(tx), "rows of the previous tree");
    require(tpd.is_contiguous() && tpd.type() == at::kFloat && tpd.shaped({B, Np, H}), "prev_dt fp32 [B,Np,H], dense");
    require(td.is_contiguous() && td.type() == at::kFloat && th.is_contiguous(), "dt fp32, dense; h0 dense");
    Result y, h;
    sized(y, a[out], a[x], {B, N, H, P}, a[x]);
    like(h, a[h_out], a[h0]);
    stree_dims d = make_dims(B, N, H, P, S, G, 0, rows_code(a[x]), state_code(a[h0], h.arg()), truth(a[force_fma]) ? STREE_FLAG_FORCE_FMA : 0, a[dt_bias]);
    d.x_stride_n = token_stride(tx, N), d.b_stride_n = token_stride(tb, N), d.c_stride_n = token_stride(tc, N);
    stree_replay r = {};
    r.nnodes = (int32_t)Np, r.parent = (const int32_t *)Array(a[pparent]).data_ptr();
    r.accepted = (const int32_t *)Array(a[paccepted]).data_ptr(), r.x = tpx.data_ptr(), r.dt = (const float *)tpd.data_ptr();
    r.Bm = tpb.data_ptr(), r.x_stride_n = token_stride(tpx, Np), r.b_stride_n = token_stride(tpb, Np);
    const auto p0 = (const int32_t *)pointer(a[parent]);
    const void *p1 = pointer(a[x]), *p4 = pointer(a[Bm]), *p5 = pointer(a[Cm]), *p7 = pointer(a[h0]);
    const auto p2 = (const float *)pointer(a[dt]), p3 = (const float *)pointer(a[A]), p6 = (const float *)pointer(a[D]);
    void *p8 = h.ptr(), *p9 = y.ptr(), *st = stream();
    const auto p10 = (int32_t *)pointer(a[status]), p11 = (int32_t *)pointer(a[rstatus]);
    run("stree_tree_ssd_replay", [&] { return g_entry.tree_ssd_replay(&d, &r, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, p10, p11, st); });
    return pair(y, h);
}

PyObject *conv_replay(const Args &a) {
    enum { pparent, paccepted, pxbc_pre, parent, xbc_pre, conv_state, conv_w, conv_b, nheads, headdim, dstate, ngroups, silu, out,
           conv_state_out, status, rstatus };
    const Array x(a[xbc_pre]), w(a[conv_w]), px(a[pxbc_pre]), cs(a[conv_state]);
    dimensions(x, 3);
    require(px.dim() >= 2, "rows of the previous tree");
    const int64_t B = x.size(0), N = x.size(1), Cc = x.size(2), W = w.size(1), Np = px.size(1);
    const int64_t H = integer(a[nheads]), P = integer(a[headdim]), S = integer(a[dstate]), G = integer(a[ngroups]);
    require(channels_are(Cc, H, P, S, G) && px.shaped({B, Np, Cc}), "channels of xbc_pre and prev_xbc_pre");
    require(x.is_contiguous() && cs.is_contiguous() && w.is_contiguous() && px.is_contiguous(), "contiguous rows");
    Result y, c;
    like(y, a[out], a[xbc_pre]);
    like(c, a[conv_state_out], a[conv_state]);
    require(c.t().data_ptr() != cs.data_ptr(), "conv_state_out must not be conv_state");
    const stree_dims d = make_dims(B, N, H, P, S, G, W, rows_code(a[xbc_pre]), STREE_F32, truth(a[silu]) ? STREE_FLAG_CONV_SILU : 0, a.none());
    stree_replay r = {};
    r.nnodes = (int32_t)Np, r.parent = (const int32_t *)Array(a[pparent]).data_ptr();
    r.accepted = (const int32_t *)Array(a[paccepted]).data_ptr();
    const void *p0 = pointer(a[pxbc_pre]), *p2 = pointer(a[xbc_pre]), *p3 = pointer(a[conv_state]), *p4 = pointer(a[conv_w]), *p5 = pointer(a[conv_b]);
    const auto p1 = (const int32_t *)pointer(a[parent]);
    void *p6 = y.ptr(), *p7 = c.ptr(), *st = stream();
    const auto p8 = (int32_t *)pointer(a[status]), p9 = (int32_t *)pointer(a[rstatus]);
    run("stree_tree_conv_replay", [&] { return g_entry.tree_conv_replay(&d, &r, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, st); });
    return pair(y, c);
}

PyObject *step(const Args &a) {
    enum { pparent, paccepted, pxbc_pre, pxbc_out, pdt, parent, xbc_pre, conv_state, conv_w, conv_b, dt, A, D, h0, nheads, headdim, dstate,
           ngroups, silu, xbc_out, conv_state_out, h_out, out, status, rstatus, force_fma, dt_bias };
    const Array x(a[xbc_pre]), w(a[conv_w]), px(a[pxbc_pre]), po(a[pxbc_out]);
    const Array cs(a[conv_state]), tpd(a[pdt]), td(a[dt]), th(a[h0]);
    dimensions(x, 3);
    require(px.dim() >= 2, "rows of the previous tree");
    const int64_t B = x.size(0), N = x.size(1), Cc = x.size(2), W = w.size(1), Np = px.size(1);
    const int64_t H = integer(a[nheads]), P = integer(a[headdim]), S = integer(a[dstate]), G = integer(a[ngroups]);
    require(channels_are(Cc, H, P, S, G) && px.shaped({B, Np, Cc}) && po.shaped({B, Np, Cc}), "channels of the rows of both trees");
    for (const Array *t : {&x, &cs, &w, &px, &po, &tpd, &td, &th}) require(t->is_contiguous(), "dense tensors");
    require(td.type() == at::kFloat && tpd.type() == at::kFloat && tpd.shaped({B, Np, H}), "dt fp32, prev_dt fp32 [B,Np,H]");
    Result xo, c, h, y;
    like(xo, a[xbc_out], a[xbc_pre]);
    like(c, a[conv_state_out], a[conv_state]);
    like(h, a[h_out], a[h0]);
    sized(y, a[out], a[xbc_pre], {B, N, H, P}, a[xbc_pre]);
    require(xo.t().is_contiguous() && y.t().is_contiguous() && h.t().is_contiguous(), "dense results");
    require(c.t().data_ptr() != cs.data_ptr(), "conv_state_out must not be conv_state");
    const stree_dims d = make_dims(B, N, H, P, S, G, W, rows_code(a[xbc_pre]), state_code(a[h0], h.arg()),
                                   (truth(a[silu]) ? STREE_FLAG_CONV_SILU : 0) | (truth(a[force_fma]) ? STREE_FLAG_FORCE_FMA : 0), a[dt_bias]);
    stree_replay r = {};
    r.nnodes = (int32_t)Np, r.parent = (const int32_t *)Array(a[pparent]).data_ptr();
    r.accepted = (const int32_t *)Array(a[paccepted]).data_ptr(), r.x = po.data_ptr(), r.dt = (const float *)tpd.data_ptr();
    r.Bm = static_cast<const char *>(po.data_ptr()) + H * P * po.element_size();             // the B columns behind x's
    r.x_stride_n = r.b_stride_n = Cc;
    const void *p0 = pointer(a[pxbc_pre]), *p2 = pointer(a[xbc_pre]), *p3 = pointer(a[conv_state]), *p4 = pointer(a[conv_w]), *p5 = pointer(a[conv_b]);
    const auto p1 = (const int32_t *)pointer(a[parent]);
    void *p6 = xo.ptr(), *p7 = c.ptr(), *p12 = h.ptr(), *p13 = y.ptr();
    const auto p8 = (const float *)pointer(a[dt]), p9 = (const float *)pointer(a[A]), p10 = (const float *)pointer(a[D]);
    const void *p11 = pointer(a[h0]);
    const auto p14 = (int32_t *)pointer(a[status]), p15 = (int32_t *)pointer(a[rstatus]);
    void *st = stream();
    run("stree_tree_step", [&] {
        return g_entry.tree_step(&d, &r, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, p10, p11, p12, p13, p14, p15, st);
    });
    return PyTuple_Pack(4, y.o, h.o, xo.o, c.o);
}

PyObject *gate(const Args &a) {
    enum { y, z, norm_w, ngroups, eps, out };
    const Array ty(a[y]), tz(a[z]), tw(a[norm_w]);
    dimensions(ty, 4);
    const int64_t B = ty.size(0), N = ty.size(1), H = ty.size(2), P = ty.size(3);
    require(ty.is_contiguous() && tz.sizes() == ty.sizes() && tz.same_type(ty) && tw.numel() == H * P, "y, z and norm_w agree");
    Result o;
    like(o, a[out], a[y]);
    const stree_dims d = make_dims(B, N, H, P, 1, integer(a[ngroups]), 0, rows_code(a[y]), STREE_F32, 0, a.none());
    const int64_t zs = token_stride(tz, N);
    const float e = (float)PyFloat_AsDouble(a[eps]);
    if (PyErr_Occurred()) throw Raised{};
    const void *p0 = ty.data_ptr(), *p1 = tz.data_ptr(), *p2 = tw.data_ptr();
    void *p3 = o.ptr(), *st = stream();
    run("stree_gate_norm", [&] { return g_entry.gate_norm(&d, p0, p1, zs, p2, e, p3, st); });
    return o.release();
}

PyObject *linear(const Args &a) {
    enum { x, dt, A, Bm, Cm, D, h0, want_y, out, h_out, dt_bias };
    const Array tx(a[x]), tb(a[Bm]), td(a[dt]);
    dimensions(tx, 4);
    require(tb.dim() == 4, "inner dims must be dense");
    const int64_t B = tx.size(0), T = tx.size(1), H = tx.size(2), P = tx.size(3), G = tb.size(2), S = tb.size(3);
    require(td.is_contiguous() && td.type() == at::kFloat && td.shaped({B, T, H}), "dt fp32 [B,T,H], dense");
    const bool wanted = truth(a[want_y]);
    Result y, h;
    if (wanted) sized(y, a[out], a[x], {B, T, H, P}, a[x]);
    else y.none();
    sized(h, a[h_out], a[x], {B, H, P, S}, a[h0]);
    stree_dims d = make_dims(B, T, H, P, S, G, 0, rows_code(a[x]), state_code(a[h0], h.arg()), 0, a[dt_bias]);
    d.x_stride_n = token_stride(tx, T), d.b_stride_n = token_stride(tb, T);
    d.c_stride_n = a[Cm] == Py_None ? 0 : token_stride(Array(a[Cm]), T);
    const void *p0 = pointer(a[x]), *p3 = pointer(a[Bm]), *p4 = pointer(a[Cm]), *p6 = pointer(a[h0]);
    const auto p1 = (const float *)pointer(a[dt]), p2 = (const float *)pointer(a[A]), p5 = (const float *)pointer(a[D]);
    void *p7 = y.ptr(), *p8 = h.ptr(), *st = stream();
    run("stree_linear_ssd", [&] { return g_entry.linear_ssd(&d, p0, p1, p2, p3, p4, p5, p6, p7, p8, st); });
    return pair(y, h);
}

template <PyObject *(*F)(const Args &), int kArgs>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != kArgs) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, not %d", kArgs, (int)n);
        return nullptr;
    }
    try {
        return F(Args{args, at::impl::torch_function_mode_enabled()});
    } catch (const Raised &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// bind(StreeError, addresses in the order of Entry)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    constexpr int kEntries = sizeof(Entry) / sizeof(void *);
    if (n != kEntries + 1) {
        PyErr_SetString(PyExc_TypeError, "bind(error, addresses)");
        return nullptr;
    }
    void *at[kEntries];
    for (int i = 0; i < kEntries; ++i) {
        at[i] = PyLong_AsVoidPtr(args[i + 1]);
        if (!at[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    static_assert(sizeof(at) == sizeof(Entry), "");
    std::memcpy(&g_entry, at, sizeof(at));
    Py_INCREF(args[0]);
    Py_XDECREF(g_error);
    g_error = args[0];
    Py_RETURN_NONE;
}

#define STREE_METHOD(name, f, args) {name, (PyCFunction)(void (*)(void))entry<f, args>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    STREE_METHOD("tree_conv", conv, 12),
    STREE_METHOD("tree_ssd", ssd, 13),
    STREE_METHOD("commit_state", commit, 14),
    STREE_METHOD("tree_ssd_replay", ssd_replay, 19),
    STREE_METHOD("tree_conv_replay", conv_replay, 17),
    STREE_METHOD("tree_step", step, 27),
    STREE_METHOD("gate_norm", gate, 6),
    STREE_METHOD("linear_ssd", linear, 11),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
