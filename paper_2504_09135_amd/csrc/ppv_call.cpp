// The per-step calls of binding.py, from the checks of their tensors to the library call, as a CPython extension.
//
// What bounds it: a per-step call on a small batch is over on the GPU in 4 to 8 us, and the same work done in Python
// (ctypes conversions; device, dtype, shape, contiguity and address of ten tensors, a Stream object for its handle)
// took 10 to 12 us of host time per call, so that the host set the pace of every eager decoding loop.
//
// The extension is not linked against libppv_hip.so: binding.py loads the library and hands over the addresses of
// its entry points (bind), so that there is one place that finds, or fails to find, the library.  Every function here
// takes its arguments by position, None where an optional one is left out, raises what binding.py documents for
// arguments that do not fit, and returns the ppv_status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ppv.h"

namespace {

struct Entry {
    decltype(&::ppv_next_token_mask) next_token_mask;
    decltype(&::constrained_sample) sample, sample_noalloc;
    decltype(&::ppv_decode_begin) begin;
    decltype(&::ppv_decode_begin_empty) begin_empty;
    decltype(&::ppv_decode_step) step, first_step;
    decltype(&::ppv_decode_loop) loop;
    decltype(&::ppv_topm_mask) topm;
    decltype(&::ppv_disc_select) disc;
    decltype(&::ppv_sample_next) sample_next;
} lib;

PyObject *s_handle, *s_n_words, *s_vocab, *s_cuda_stream;   // interned attribute names

// A Python error has been set; unwinds to the function's entry.
struct Raised {};

[[noreturn]] void raise(PyObject *kind, const char *format, const char *a = "", const char *b = "", const char *c = "") {
    PyErr_Format(kind, format, a, b, c);
    throw Raised();
}

const at::Tensor &tensor(PyObject *o, const char *what) {
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s: need a GPU tensor, got %s", what, Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}

// a contiguous GPU tensor's address
template <typename P> P *address(PyObject *o, at::ScalarType dtype, const char *what) {
    const at::Tensor &t = tensor(o, what);
    if (!(t.is_cuda() && t.scalar_type() == dtype && t.is_contiguous())) {
        PyObject *dt = PyObject_GetAttrString(o, "dtype"), *dev = PyObject_GetAttrString(o, "device");
        if (dt && dev)
            PyErr_Format(PyExc_TypeError, "%s: need a contiguous GPU tensor of torch.%s, got %S on %S", what,
                         dtype == at::kInt ? "int32" : (dtype == at::kFloat ? "float32" : "uint8"), dt, dev);
        Py_XDECREF(dt);
        Py_XDECREF(dev);
        throw Raised();
    }
    return (P *)t.data_ptr();
}

bool has_shape(const at::Tensor &t, int64_t n) { return t.dim() == 1 && t.size(0) == n; }
bool has_shape(const at::Tensor &t, int64_t n, int64_t m) { return t.dim() == 2 && t.size(0) == n && t.size(1) == m; }

constexpr at::ScalarType I32 = at::kInt, F32 = at::kFloat, U8 = at::kByte;

// A tensor argument of the shape [n] (m < 0) or [n, m]; None stands for a null pointer where the argument is optional.
struct Arg {
    PyObject *o;
    const char *name;
    bool none() const { return o == Py_None; }
    bool fits(int64_t n, int64_t m = -1) const {
        const at::Tensor &t = tensor(o, name);
        return m < 0 ? has_shape(t, n) : has_shape(t, n, m);
    }
    bool fits_or_none(int64_t n, int64_t m = -1) const { return none() || fits(n, m); }
    template <typename P> P *get(at::ScalarType dtype) const { return none() ? nullptr : address<P>(o, dtype, name); }
};

// the index's handle and one of its sizes
template <typename H = const ppv_index_t> H *handle(PyObject *index) {
    PyObject *v = PyObject_GetAttr(index, s_handle);
    if (!v) throw Raised();
    if (v == Py_None) {
        Py_DECREF(v);
        raise(PyExc_ValueError, "index already freed");
    }
    void *p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!p && PyErr_Occurred()) throw Raised();
    return (H *)p;
}
int64_t size_of(PyObject *index, PyObject *attr) {
    PyObject *v = PyObject_GetAttr(index, attr);
    if (!v) throw Raised();
    const int64_t n = PyLong_AsLongLong(v);
    Py_DECREF(v);
    if (n == -1 && PyErr_Occurred()) throw Raised();
    return n;
}

void *stream_of(PyObject *o) {
    if (o == Py_None) return (void *)c10::hip::getCurrentHIPStream().stream();
    PyObject *v = PyObject_GetAttr(o, s_cuda_stream);
    if (!v) throw Raised();
    void *p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!p && PyErr_Occurred()) throw Raised();
    return p;
}

float temperature_of(PyObject *o) {
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject *f = PyNumber_Float(o);
    if (!f) throw Raised();
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}

int64_t int_of(PyObject *o) {
    PyObject *n = PyNumber_Long(o);
    if (!n) throw Raised();
    const int64_t v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}

ppv_dtype logits_dtype(const at::Tensor &t) {
    if (t.scalar_type() == at::kFloat) return PPV_F32;
    if (t.scalar_type() == at::kBFloat16) return PPV_BF16;
    raise(PyExc_TypeError, "logits: float32 or bfloat16, got %s", c10::toString(t.scalar_type()));
}

struct Logits {
    const void *ptr;
    ppv_dtype dtype;
    int64_t row_stride;
    int64_t B, V;
    explicit Logits(PyObject *o) {
        const at::Tensor &t = tensor(o, "logits");
        if (t.dim() != 2 || !t.is_cuda() || t.stride(1) != 1)
            raise(PyExc_ValueError, "logits: need a 2-D GPU tensor with unit stride along the vocabulary");
        dtype = logits_dtype(t);
        B = t.size(0);
        V = t.size(1);
        // a single row: torch's stride of a size-1 dimension carries no meaning unless it covers the row (a row cut out
        // of a padded buffer keeps the buffer's stride, which is what says that the padding is there)
        row_stride = t.stride(0);
        if (B <= 1 && row_stride < V) row_stride = V;
        ptr = t.data_ptr();
    }
};

// prefixes as a 2-D matrix (-1 rows if it is not one); the decoding calls also take further dimensions behind the first two
// (a column of size 1, say) and read rows of the second one's size from its start
struct Prefixes {
    int64_t B = -1, stride = 0;
    PyObject *o;
    explicit Prefixes(PyObject *p, bool decoding = false) : o(p) {
        const at::Tensor &t = tensor(p, "prefixes");
        if (decoding && t.dim() < 2) raise(PyExc_IndexError, "prefixes: need a tensor of shape [B, stride]");
        if (!decoding && t.dim() != 2) return;
        B = t.size(0);
        stride = t.size(1);
    }
    int32_t *get() const { return address<int32_t>(o, I32, "prefixes"); }
};

template <typename F> PyObject *status(F call) {
    ppv_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

// runs the body of a function: C++ exceptions (ours, torch's) become Python errors
template <typename F> PyObject *guarded(const char *name, Py_ssize_t n, Py_ssize_t want, F body) {
    if (n != want) return PyErr_Format(PyExc_TypeError, "%s: %zd arguments, %zd expected", name, n, want);
    if (!lib.step) return PyErr_Format(PyExc_RuntimeError, "%s: bind() has not been called", name);
    try {
        return body();
    } catch (const Raised &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// index, prefixes, lens, mask, range_lo, range_hi, member, stream
PyObject *next_token_mask(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("next_token_mask", n, 8, [&] {
        const Prefixes p(a[1]);
        const Arg lens{a[2], "lens"}, mask{a[3], "mask"}, lo{a[4], "range_lo"}, hi{a[5], "range_hi"}, member{a[6], "member"};
        if (p.B < 0 || !lens.fits(p.B) || !mask.fits(p.B, size_of(a[0], s_n_words)))
            raise(PyExc_ValueError, "ppv_next_token_mask: shape mismatch");
        for (const Arg &x : {lo, hi, member})
            if (!x.fits_or_none(p.B)) raise(PyExc_ValueError, "ppv_next_token_mask: %s must have shape [B]", x.name);
        const ppv_index_t *ix = handle(a[0]);
        const int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32);
        uint32_t *mk = mask.get<uint32_t>(I32), *rl = lo.get<uint32_t>(I32), *rh = hi.get<uint32_t>(I32);
        uint8_t *me = member.get<uint8_t>(U8);
        void *s = stream_of(a[7]);
        return status([&] { return lib.next_token_mask(ix, pp, (int32_t)p.stride, ln, (int32_t)p.B, mk, rl, rh, me, s); });
    });
}

// logits, mask, uniforms, ids, logZ_valid, logZ_all, stream, temperature, noalloc
PyObject *sample(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("sample", n, 9, [&] {
        const Logits l(a[0]);
        const Arg mask{a[1], "mask"}, un{a[2], "uniforms"}, ids{a[3], "ids"}, lzv{a[4], "logZ_valid"}, lza{a[5], "logZ_all"};
        if (!mask.fits(l.B, (l.V + 31) / 32) || !un.fits(l.B) || !ids.fits(l.B) || !lzv.fits(l.B) || !lza.fits_or_none(l.B))
            raise(PyExc_ValueError, "constrained_sample: shape mismatch");
        const uint32_t *mk = mask.get<uint32_t>(I32);
        const float *u = un.get<float>(F32);
        int32_t *id = ids.get<int32_t>(I32);
        float *zv = lzv.get<float>(F32), *za = lza.get<float>(F32);
        const float T = temperature_of(a[7]);
        const auto fn = PyObject_IsTrue(a[8]) ? lib.sample_noalloc : lib.sample;
        void *s = stream_of(a[6]);
        return status([&] { return fn(l.ptr, l.dtype, l.row_stride, mk, u, (int32_t)l.B, (int32_t)l.V, id, zv, za, T, s); });
    });
}

// index, prefixes, lens, state, active, logx, stream
PyObject *decode_begin(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("decode_begin", n, 7, [&] {
        const Prefixes p(a[1], true);
        const Arg lens{a[2], "lens"}, state{a[3], "state"}, active{a[4], "active"}, logx{a[5], "logx"};
        if (!lens.fits(p.B) || !state.fits(p.B, PPV_STATE_WORDS) || !active.fits(p.B) || !logx.fits_or_none(p.B))
            raise(PyExc_ValueError, "ppv_decode_begin: shape mismatch");
        const ppv_index_t *ix = handle(a[0]);
        const int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32);
        uint32_t *st = state.get<uint32_t>(I32);
        uint8_t *on = active.get<uint8_t>(U8);
        float *lx = logx.get<float>(F32);
        void *s = stream_of(a[6]);
        return status([&] { return lib.begin(ix, pp, (int32_t)p.stride, ln, (int32_t)p.B, st, on, lx, s); });
    });
}

// index, lens, state, active, logx, stream
PyObject *decode_begin_empty(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("decode_begin_empty", n, 6, [&] {
        const Arg lens{a[1], "lens"}, state{a[2], "state"}, active{a[3], "active"}, logx{a[4], "logx"};
        const at::Tensor &l = tensor(a[1], "lens");
        if (l.dim() < 1) raise(PyExc_IndexError, "lens: need a tensor of shape [B]");
        const int64_t B = l.size(0);
        if (l.dim() != 1 || !state.fits(B, PPV_STATE_WORDS) || !active.fits(B) || !logx.fits_or_none(B))
            raise(PyExc_ValueError, "ppv_decode_begin_empty: shape mismatch");
        const ppv_index_t *ix = handle(a[0]);
        int32_t *ln = lens.get<int32_t>(I32);
        uint32_t *st = state.get<uint32_t>(I32);
        uint8_t *on = active.get<uint8_t>(U8);
        float *lx = logx.get<float>(F32);
        void *s = stream_of(a[5]);
        return status([&] { return lib.begin_empty(ix, (int32_t)B, ln, st, on, lx, s); });
    });
}

// index, prefixes, lens, active, logits, uniforms, ids, logZ_valid, logx, state, stream, temperature, first
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("decode_step", n, 13, [&] {
        const Logits l(a[4]);
        const Prefixes p(a[1], true);
        const Arg lens{a[2], "lens"}, active{a[3], "active"}, un{a[5], "uniforms"}, ids{a[6], "ids"}, lzv{a[7], "logZ_valid"},
            logx{a[8], "logx"}, state{a[9], "state"};
        if (l.B != p.B || l.V != size_of(a[0], s_vocab) || !lens.fits(p.B) || !active.fits(p.B) || !un.fits(p.B) ||
            !state.fits_or_none(p.B, PPV_STATE_WORDS))
            raise(PyExc_ValueError, "ppv_decode_step: shape mismatch");
        for (const Arg &x : {ids, lzv, logx})
            if (!x.fits_or_none(p.B)) raise(PyExc_ValueError, "ppv_decode_step: %s must have shape [B]", x.name);
        const ppv_index_t *ix = handle(a[0]);
        int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32), *id = ids.get<int32_t>(I32);
        uint8_t *on = active.get<uint8_t>(U8);
        uint32_t *st = state.get<uint32_t>(I32);
        const float *u = un.get<float>(F32);
        float *zv = lzv.get<float>(F32), *lx = logx.get<float>(F32);
        const float T = temperature_of(a[11]);
        const auto fn = a[12] == Py_True ? lib.first_step : lib.step;
        void *s = stream_of(a[10]);
        return status([&] {
            return fn(ix, pp, (int32_t)p.stride, ln, on, st, l.ptr, l.dtype, l.row_stride, u, (int32_t)p.B, id, zv, lx, T, s);
        });
    });
}

// index, prefixes, lens, active, logits, uniforms, ids, logZ_valid, logx, state, stream, temperature
PyObject *decode_loop(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("decode_loop", n, 12, [&] {
        const at::Tensor &l = tensor(a[4], "logits");
        if (l.dim() != 3 || !l.is_cuda() || l.stride(2) != 1)
            raise(PyExc_ValueError, "logits: need a 3-D GPU tensor [n_steps, B, V] with unit stride along the vocabulary");
        const int64_t n_steps = l.size(0), B = l.size(1), V = l.size(2);
        const ppv_dtype dt = logits_dtype(l);
        const Prefixes p(a[1], true);
        const Arg lens{a[2], "lens"}, active{a[3], "active"}, un{a[5], "uniforms"}, ids{a[6], "ids"}, lzv{a[7], "logZ_valid"},
            logx{a[8], "logx"}, state{a[9], "state"};
        if (p.B != B || V != size_of(a[0], s_vocab) || !lens.fits(B) || !active.fits(B) || !un.fits(n_steps, B) ||
            !state.fits_or_none(B, PPV_STATE_WORDS) || !logx.fits_or_none(B))
            raise(PyExc_ValueError, "ppv_decode_loop: shape mismatch");
        for (const Arg &x : {ids, lzv})
            if (!x.fits_or_none(n_steps, B)) raise(PyExc_ValueError, "ppv_decode_loop: %s must have shape [n_steps, B]", x.name);
        const ppv_index_t *ix = handle(a[0]);
        int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32), *id = ids.get<int32_t>(I32);
        uint8_t *on = active.get<uint8_t>(U8);
        uint32_t *st = state.get<uint32_t>(I32);
        const float *u = un.get<float>(F32);
        float *zv = lzv.get<float>(F32), *lx = logx.get<float>(F32);
        const void *lp = l.data_ptr();
        const int64_t row_stride = l.stride(1), step_stride = l.stride(0);
        const float T = temperature_of(a[11]);
        void *s = stream_of(a[10]);
        return status([&] {
            return lib.loop(ix, pp, (int32_t)p.stride, ln, on, st, lp, dt, row_stride, step_stride, u, (int32_t)n_steps,
                            (int32_t)B, id, zv, lx, T, s);
        });
    });
}

// index, prefixes, lens, logits, M, mask, top_ids, mask_V, stream
PyObject *topm_mask(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("topm_mask", n, 9, [&] {
        const Logits l(a[3]);
        const Prefixes p(a[1]);
        const int64_t M = int_of(a[4]);
        const Arg lens{a[2], "lens"}, mask{a[5], "mask"}, top{a[6], "top_ids"}, mv{a[7], "mask_V"};
        if (p.B < 0 || l.B != p.B || l.V != size_of(a[0], s_vocab) || !lens.fits(p.B) || !mask.fits(p.B, size_of(a[0], s_n_words)))
            raise(PyExc_ValueError, "ppv_topm_mask: shape mismatch");
        for (const Arg &x : {top, mv})
            if (!x.fits_or_none(p.B, M < 0 ? -2 : M)) raise(PyExc_ValueError, "ppv_topm_mask: %s must have shape [B, M]", x.name);
        const ppv_index_t *ix = handle(a[0]);
        const int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32);
        int32_t *ti = top.get<int32_t>(I32);
        uint8_t *me = mv.get<uint8_t>(U8);
        uint32_t *mk = mask.get<uint32_t>(I32);
        void *s = stream_of(a[8]);
        return status([&] {
            return lib.topm(ix, pp, (int32_t)p.stride, ln, l.ptr, l.dtype, l.row_stride, (int32_t)M, (int32_t)p.B, ti, me, mk, s);
        });
    });
}

// logx, K, accept_u, resample_u, chosen, n_draws, accepted, reuse_rejected, stream
PyObject *disc_select(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("disc_select", n, 9, [&] {
        const Arg logx{a[0], "logx"}, au{a[2], "accept_u"}, ru{a[3], "resample_u"}, ch{a[4], "chosen"}, nd{a[5], "n_draws"},
            ac{a[6], "accepted"};
        const at::Tensor &x = tensor(a[0], "logx");
        const int64_t K = int_of(a[1]);
        if (x.dim() < 2) raise(PyExc_IndexError, "ppv_disc_select: logx must have shape [n_candidates, Q]");
        const int64_t n_cand = x.size(0), Q = x.size(1);
        if (!au.fits(K < 0 ? -2 : K, Q) || !ru.fits(Q) || !ch.fits(Q)) raise(PyExc_ValueError, "ppv_disc_select: shape mismatch");
        const float *lx = logx.get<float>(F32), *u1 = au.get<float>(F32), *u2 = ru.get<float>(F32);
        int32_t *c = ch.get<int32_t>(I32), *d = nd.get<int32_t>(I32);
        uint8_t *acc = ac.get<uint8_t>(U8);
        const int reuse = PyObject_IsTrue(a[7]);
        if (reuse < 0) throw Raised();
        void *s = stream_of(a[8]);
        return status([&] { return lib.disc(lx, (int32_t)n_cand, (int32_t)K, (int32_t)Q, u1, u2, reuse, c, d, acc, s); });
    });
}

// index, prefixes, lens, logits, uniforms, ids, logZ_valid, stream, temperature
PyObject *sample_next(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded("sample_next", n, 9, [&] {
        const Logits l(a[3]);
        const Prefixes p(a[1]);
        const Arg lens{a[2], "lens"}, un{a[4], "uniforms"}, ids{a[5], "ids"}, lzv{a[6], "logZ_valid"};
        if (p.B < 0 || l.B != p.B || l.V != size_of(a[0], s_vocab) || !lens.fits(p.B) || !un.fits(p.B) || !ids.fits(p.B) ||
            !lzv.fits_or_none(p.B))
            raise(PyExc_ValueError, "ppv_sample_next: shape mismatch");
        const ppv_index_t *ix = handle(a[0]);
        const int32_t *pp = p.get(), *ln = lens.get<int32_t>(I32);
        const float *u = un.get<float>(F32);
        int32_t *id = ids.get<int32_t>(I32);
        float *zv = lzv.get<float>(F32);
        const float T = temperature_of(a[8]);
        void *s = stream_of(a[7]);
        return status([&] {
            return lib.sample_next(ix, pp, (int32_t)p.stride, ln, (int32_t)p.B, l.ptr, l.dtype, l.row_stride, u, id, zv, T, s);
        });
    });
}

// bind({entry point's name: its address})
PyObject *bind(PyObject *, PyObject *table) {
    if (!PyDict_Check(table)) return PyErr_Format(PyExc_TypeError, "bind: need a dict of addresses");
    bool fine = true;
    auto find = [&](const char *name) -> void * {
        PyObject *v = PyDict_GetItemString(table, name);   // borrowed
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p && fine) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "bind: no address for %s", name);
            fine = false;
        }
        return p;
    };
    Entry e;
    e.next_token_mask = (decltype(e.next_token_mask))find("ppv_next_token_mask");
    e.sample = (decltype(e.sample))find("constrained_sample");
    e.sample_noalloc = (decltype(e.sample_noalloc))find("constrained_sample_noalloc");
    e.begin = (decltype(e.begin))find("ppv_decode_begin");
    e.begin_empty = (decltype(e.begin_empty))find("ppv_decode_begin_empty");
    e.step = (decltype(e.step))find("ppv_decode_step");
    e.first_step = (decltype(e.first_step))find("ppv_decode_first_step");
    e.loop = (decltype(e.loop))find("ppv_decode_loop");
    e.topm = (decltype(e.topm))find("ppv_topm_mask");
    e.disc = (decltype(e.disc))find("ppv_disc_select");
    e.sample_next = (decltype(e.sample_next))find("ppv_sample_next");
    if (!fine) return nullptr;
    lib = e;
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(next_token_mask), FAST(sample),      FAST(decode_begin), FAST(decode_begin_empty),
                         FAST(decode_step),     FAST(decode_loop), FAST(topm_mask),    FAST(disc_select),
                         FAST(sample_next),     {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ppv_call", "Native argument checks and calls of binding.py.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ppv_call() {
    s_handle = PyUnicode_InternFromString("_address");
    s_n_words = PyUnicode_InternFromString("n_words");
    s_vocab = PyUnicode_InternFromString("vocab");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_handle || !s_n_words || !s_vocab || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
