// Argument marshalling of the Python binding: checks the tensors, collects their addresses and calls the C ABI.
//
// What bounds a call on a short gradient is the host, not the GPU: checking and converting the arguments in Python took
// 4.5 to 6.5 us a call with four workers (10 with sixteen) beside 3.6 to 8 us for the call itself.  Here the same checks
// take well under a microsecond.  Every function takes its arguments by position, raises ValueError where a tensor does not fit the call, and
// returns the library's status code.  The interpreter lock is released around the library; until it returns, the sequences
// that the addresses came from are kept, and nothing beyond.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <stdint.h>

#include "gqsgd.h"

#ifndef GQ_BUILT_FOR
#error "GQ_BUILT_FOR names the torch and the interpreter that this is compiled for"
#endif

namespace {

// the library's entry points, by their addresses in the copy that the binding loaded
#define GQ_ENTRY_POINTS(X)                                                                                              \
    X(gq_global_norm) X(gq_global_norm_static) X(gq_quantize) X(gq_int_aggregate) X(gq_dequantize)                      \
    X(gq_fused_quantize_aggregate) X(gq_bucketed_quantize_aggregate) X(gq_exp_reduce) X(gq_avg_reduce) X(gq_compact)     \
    X(gq_quantize_compact) X(gq_sparse_aggregate) X(gq_tile_starts_len)
struct Library {
#define GQ_FIELD(name) decltype(&name) name##_;
    GQ_ENTRY_POINTS(GQ_FIELD)
#undef GQ_FIELD
} lib;

PyObject *current_device = nullptr, *current_raw_stream = nullptr;     // torch's own functions

struct Refused {};                                                     // a Python error has been set

const at::Tensor &tensor(PyObject *o, const char *what)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", what);
        throw Refused();
    }
    return THPVariable_Unpack(o);
}

// The C ABI takes raw addresses and cannot see buffer sizes: a tensor that is too small, not contiguous or not on the GPU
// is refused here, before any launch.
void *need(const at::Tensor &t, int64_t nbytes, const char *what)
{
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous CUDA tensor", what);
        throw Refused();
    }
    const int64_t have = t.numel() * (int64_t)t.element_size();
    if (have < nbytes) {
        PyErr_Format(PyExc_ValueError, "%s holds %lld bytes, the call needs %lld", what, (long long)have, (long long)nbytes);
        throw Refused();
    }
    return t.data_ptr();
}
void *need(PyObject *o, int64_t nbytes, const char *what) { return o == Py_None ? nullptr : need(tensor(o, what), nbytes, what); }

int64_t integer(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Refused();
    return v;
}

struct Params {                                                        // a ctypes gq_params, read in place
    Py_buffer view;
    explicit Params(PyObject *o)
    {
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Refused();
        if (view.len != (Py_ssize_t)sizeof(gq_params)) {
            PyBuffer_Release(&view);
            PyErr_SetString(PyExc_TypeError, "params must be a gq_params");
            throw Refused();
        }
    }
    ~Params() { PyBuffer_Release(&view); }
    Params(const Params &) = delete;
    Params &operator=(const Params &) = delete;
    const gq_params *get() const { return reinterpret_cast<const gq_params *>(view.buf); }
    int64_t agg_bytes() const { return get()->agg == GQ_AGG_I16 ? 2 : 4; }
    int64_t levels_nbytes(int64_t d) const { return get()->pack == GQ_PACK_I8 || get()->pack == GQ_PACK_U8_SIGNPLANE ? d : (d + 1) / 2; }
    bool planes() const { return get()->pack >= GQ_PACK_U8_SIGNPLANE; }
};

// A list, a tuple or another sequence (rows of a tensor among them) as a list or tuple; its items are borrowed while this lives.
// An iterator has no length and is refused: its tensors may be nobody else's.  None: no list.
struct List {
    PyObject *seq = nullptr;
    explicit List(PyObject *o)
    {
        if (o == Py_None) return;
        if (PyObject_Size(o) < 0 || !(seq = PySequence_Fast(o, "a list of tensors is wanted"))) throw Refused();
    }
    ~List() { Py_XDECREF(seq); }
    List(const List &) = delete;
    List &operator=(const List &) = delete;
    int64_t size() const { return seq ? (int64_t)PySequence_Fast_GET_SIZE(seq) : 0; }
    PyObject *operator[](int64_t i) const { return PySequence_Fast_GET_ITEM(seq, i); }
};

typedef c10::SmallVector<void *, GQ_MAX_WORKERS> Pointers;

// The addresses of a list of tensors of at least nbytes each, the list kept with them; None gives a null address.  A list that the
// call does not use (`used` false) is not looked at.
struct Addresses {
    const List list;
    Pointers p;
    Addresses(PyObject *o, int64_t nbytes, const char *what, bool used = true) : list(used ? o : Py_None)
    {
        for (int64_t i = 0; i < list.size(); i++) p.push_back(need(list[i], nbytes, what));
    }
    bool given() const { return list.seq != nullptr; }
    template <typename T> T *const *as() const { return given() ? reinterpret_cast<T *const *>(p.data()) : nullptr; }
    int K() const { return (int)p.size(); }
};

void wanted(PyObject *o)                                               // a list that may not be None
{
    if (o != Py_None) return;
    PyErr_SetString(PyExc_TypeError, "a list of tensors is wanted, not None");
    throw Refused();
}

struct Gradients {
    const List list;
    Pointers p;
    int64_t d = 0;
    void add(const at::Tensor &t, bool first)
    {
        if (first) d = t.numel();
        if (t.scalar_type() != at::kFloat || t.numel() != d) {
            PyErr_SetString(PyExc_ValueError, "gradients must be float32 tensors of equal length");
            throw Refused();
        }
        p.push_back(need(t, 4 * d, "gradient"));
    }
    explicit Gradients(const at::Tensor &x) : list(Py_None) { add(x, true); }
    explicit Gradients(PyObject *o) : list(o)
    {
        wanted(o);
        for (int64_t i = 0; i < list.size(); i++) add(tensor(list[i], "gradient"), i == 0);
    }
    const float *const *x() const { return reinterpret_cast<const float *const *>(p.data()); }
    int K() const { return (int)p.size(); }
};

// the stream's address, or the current one of the current device
void *stream_of(PyObject *o)
{
    if (o != Py_None) return reinterpret_cast<void *>((uintptr_t)integer(o));
    PyObject *dev = PyObject_CallObject(current_device, nullptr);
    if (!dev) throw Refused();
    PyObject *raw = PyObject_CallFunctionObjArgs(current_raw_stream, dev, nullptr);
    Py_DECREF(dev);
    if (!raw) throw Refused();
    void *s = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    if (!s && PyErr_Occurred()) throw Refused();
    return s;
}

template <typename F> PyObject *call(F &&f)
{
    gq_status st;
    {
        PyThreadState *save = PyEval_SaveThread();
        st = f();                                                      // C entry points: nothing is thrown
        PyEval_RestoreThread(save);
    }
    return PyLong_FromLong((long)st);
}

// Every function: exactly N positional arguments; C++ exceptions (torch's, bad_alloc) become Python ones.
template <int N, PyObject *(*F)(PyObject *const *)> PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments are wanted", N);
        return nullptr;
    }
    try {
        return F(a);
    } catch (const Refused &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// xs, kind, norm_out, status_flags, workspace, stream
PyObject *global_norm(PyObject *const *a)
{
    const Gradients g(a[0]);
    void *norm = need(a[2], 4, "norm_out"), *flags = need(a[3], 4, "status_flags");
    const at::Tensor &ws = tensor(a[4], "workspace");
    const size_t bytes = (size_t)(ws.numel() * (int64_t)ws.element_size());
    void *wsp = ws.data_ptr(), *st = stream_of(a[5]);
    const gq_norm_kind kind = (gq_norm_kind)integer(a[1]);
    return call([&] { return lib.gq_global_norm_(g.x(), g.K(), g.d, kind, (float *)norm, (uint32_t *)flags, wsp, bytes, st); });
}

// xs, kind, norm_out, status_flags, stream
PyObject *global_norm_static(PyObject *const *a)
{
    const Gradients g(a[0]);
    void *norm = need(a[2], 4, "norm_out"), *flags = need(a[3], 4, "status_flags"), *st = stream_of(a[4]);
    const gq_norm_kind kind = (gq_norm_kind)integer(a[1]);
    return call([&] { return lib.gq_global_norm_static_(g.x(), g.K(), g.d, kind, (float *)norm, (uint32_t *)flags, st); });
}

// x, norm, params, worker, index_base, levels_out, signplane_out, stream
PyObject *quantize(PyObject *const *a)
{
    const Params p(a[2]);
    const Gradients g(tensor(a[0], "gradient"));
    void *norm = need(a[1], 4, "norm"), *lv = need(a[5], p.levels_nbytes(g.d), "levels_out");
    void *sp = a[6] == Py_None ? nullptr : p.planes() ? need(a[6], 4 * ((g.d + 31) / 32), "sign plane") : tensor(a[6], "sign plane").data_ptr();
    void *st = stream_of(a[7]);
    const uint32_t worker = (uint32_t)integer(a[3]);
    const int64_t base = integer(a[4]);
    return call([&] { return lib.gq_quantize_(g.x()[0], g.d, (const float *)norm, p.get(), worker, base, lv, (uint32_t *)sp, st); });
}

// levels, signplanes, d, params, agg_out, stream
PyObject *int_aggregate(PyObject *const *a)
{
    const Params p(a[3]);
    const int64_t d = integer(a[2]);
    wanted(a[0]);
    const Addresses lv(a[0], p.levels_nbytes(d), "levels"), sp(a[1], 4 * ((d + 31) / 32), "sign plane", p.planes());
    if (sp.given() && sp.K() < lv.K()) {
        PyErr_SetString(PyExc_ValueError, "fewer sign planes than levels");
        throw Refused();
    }
    void *agg = need(a[4], p.agg_bytes() * d, "agg_out"), *st = stream_of(a[5]);
    return call([&] {
        return lib.gq_int_aggregate_(lv.as<const void>(), sp.as<const uint32_t>(), lv.K(), d, p.get(), agg, st);
    });
}

// agg, d, norm, params, K, out, stream
PyObject *dequantize(PyObject *const *a)
{
    const Params p(a[3]);
    const int64_t d = integer(a[1]);
    void *agg = need(a[0], p.agg_bytes() * d, "agg"), *out = need(a[5], 4 * d, "out"), *norm = need(a[2], 4, "norm");
    void *st = stream_of(a[6]);
    const int K = (int)integer(a[4]);
    return call([&] { return lib.gq_dequantize_(agg, d, (const float *)norm, p.get(), K, (float *)out, st); });
}

// xs, norm, params, index_base, agg_out, dequant_out, levels_out, signplanes_out, stream
PyObject *fused_quantize_aggregate(PyObject *const *a)
{
    const Params p(a[2]);
    const Gradients g(a[0]);
    void *norm = need(a[1], 4, "norm"), *agg = need(a[4], p.agg_bytes() * g.d, "agg_out"), *mean = need(a[5], 4 * g.d, "dequant_out");
    const Addresses lv(a[6], p.levels_nbytes(g.d), "levels_out");
    const Addresses sp(a[7], 4 * ((g.d + 31) / 32), "sign plane", lv.given() && p.planes());
    if ((lv.given() && lv.K() < g.K()) || (sp.given() && sp.K() < g.K())) {
        PyErr_SetString(PyExc_ValueError, "fewer level buffers or sign planes than gradients");
        throw Refused();
    }
    void *st = stream_of(a[8]);
    const int64_t base = integer(a[3]);
    return call([&] {
        return lib.gq_fused_quantize_aggregate_(g.x(), g.K(), g.d, (const float *)norm, p.get(), base, agg, (float *)mean,
                                                lv.as<void>(), sp.as<uint32_t>(), st);
    });
}

// xs, bucket, kind, params, norms_out, status_flags, agg_out, dequant_out, workspace, stream, side_stream (0: none)
PyObject *bucketed_quantize_aggregate(PyObject *const *a)
{
    const Params p(a[3]);
    const Gradients g(a[0]);
    const int64_t bucket = integer(a[1]);
    const int64_t nb = bucket > 0 ? (g.d + bucket - 1) / bucket : 0;
    void *norms = need(a[4], 4 * nb, "norms_out"), *flags = need(a[5], 4 * nb, "status_flags");
    void *agg = need(a[6], p.agg_bytes() * g.d, "agg_out"), *mean = need(a[7], 4 * g.d, "dequant_out");
    const at::Tensor &ws = tensor(a[8], "workspace");
    const size_t bytes = (size_t)(ws.numel() * (int64_t)ws.element_size());
    void *wsp = ws.data_ptr(), *st = stream_of(a[9]), *side = reinterpret_cast<void *>((uintptr_t)integer(a[10]));
    const gq_norm_kind kind = (gq_norm_kind)integer(a[2]);
    return call([&] {
        return lib.gq_bucketed_quantize_aggregate_(g.x(), g.K(), g.d, bucket, kind, p.get(), (float *)norms, (uint32_t *)flags, agg,
                                                   (float *)mean, wsp, bytes, st, side);
    });
}

// levels, d, params, index_base, norm, reduced_out, dequant_out, stream
template <bool EXP> PyObject *tree_reduce(PyObject *const *a)
{
    const Params p(a[2]);
    const int64_t d = integer(a[1]), nbytes = EXP ? d : p.levels_nbytes(d);      // Algorithm 2 takes int8 codes
    wanted(a[0]);
    const Addresses lv(a[0], nbytes, "levels");
    void *red = need(a[5], nbytes, "reduced_out"), *mean = need(a[6], 4 * d, "dequant_out"), *norm = need(a[4], 4, "norm");
    void *st = stream_of(a[7]);
    const int64_t base = integer(a[3]);
    return call([&] {
        return (EXP ? lib.gq_exp_reduce_ : lib.gq_avg_reduce_)(lv.as<const void>(), lv.K(), d, p.get(), base, (const float *)norm, red,
                                                               (float *)mean, st);
    });
}

// the buffers of a sender's list
struct ListOut {
    int64_t capacity;
    void *count, *values, *indices, *starts, *ws;
    size_t ws_bytes;
    ListOut(int64_t d, PyObject *indices_, PyObject *values_, PyObject *count_, PyObject *workspace, PyObject *starts_)
    {
        count = need(count_, 8, "count_out");
        const at::Tensor &i = tensor(indices_, "indices_out");
        capacity = i.numel();
        values = need(values_, capacity, "values_out");
        indices = need(i, 0, "indices_out");
        starts = need(starts_, 4 * lib.gq_tile_starts_len_(d), "tile_starts_out");
        const at::Tensor &w = tensor(workspace, "workspace");
        ws = w.data_ptr();
        ws_bytes = (size_t)(w.numel() * (int64_t)w.element_size());
    }
};

// levels, d, params, indices_out, values_out, count_out, workspace, tile_starts_out, stream
PyObject *compact(PyObject *const *a)
{
    const Params p(a[2]);
    const int64_t d = integer(a[1]);
    void *lv = need(a[0], d, "levels");
    const ListOut o(d, a[3], a[4], a[5], a[6], a[7]);
    void *st = stream_of(a[8]);
    return call([&] {
        return lib.gq_compact_(lv, d, p.get(), (uint32_t *)o.indices, (int8_t *)o.values, o.capacity, (uint64_t *)o.count, (uint32_t *)o.starts,
                               o.ws, o.ws_bytes, st);
    });
}

// x, norm, params, worker, index_base, indices_out, values_out, count_out, workspace, tile_starts_out, stream
PyObject *quantize_compact(PyObject *const *a)
{
    const Params p(a[2]);
    const Gradients g(tensor(a[0], "gradient"));
    void *norm = need(a[1], 4, "norm");
    const ListOut o(g.d, a[5], a[6], a[7], a[8], a[9]);
    void *st = stream_of(a[10]);
    const uint32_t worker = (uint32_t)integer(a[3]);
    const int64_t base = integer(a[4]);
    return call([&] {
        return lib.gq_quantize_compact_(g.x()[0], g.d, (const float *)norm, p.get(), worker, base, (uint32_t *)o.indices, (int8_t *)o.values,
                                        o.capacity, (uint64_t *)o.count, (uint32_t *)o.starts, o.ws, o.ws_bytes, st);
    });
}

// indices, values, counts, d, params, agg_out, tile_starts, stream
PyObject *sparse_aggregate(PyObject *const *a)
{
    const Params p(a[4]);
    const int64_t d = integer(a[3]);
    for (int i = 0; i < 3; i++) wanted(a[i]);
    const List il(a[0]), vl(a[1]), cl(a[2]);
    if (vl.size() < il.size() || cl.size() < il.size()) {
        PyErr_SetString(PyExc_ValueError, "fewer values or counts than index lists");
        throw Refused();
    }
    Pointers idx, val, cnt;
    c10::SmallVector<int64_t, GQ_MAX_WORKERS> cap;
    for (int64_t i = 0; i < il.size(); i++) {
        const at::Tensor &t = tensor(il[i], "indices");
        idx.push_back(need(t, 0, "indices"));
        cap.push_back(t.numel());
        val.push_back(need(vl[i], t.numel(), "values"));
        cnt.push_back(need(cl[i], 8, "count"));
    }
    const Addresses starts(a[6], 4 * lib.gq_tile_starts_len_(d), "tile_starts");
    if (starts.given() && starts.K() < (int)idx.size()) {
        PyErr_SetString(PyExc_ValueError, "fewer tables of tile starts than index lists");
        throw Refused();
    }
    void *agg = need(a[5], 4 * d, "agg_out"), *st = stream_of(a[7]);
    return call([&] {
        return lib.gq_sparse_aggregate_(reinterpret_cast<const uint32_t *const *>(idx.data()), reinterpret_cast<const int8_t *const *>(val.data()),
                                        reinterpret_cast<const uint64_t *const *>(cnt.data()), cap.data(),
                                        starts.as<const uint32_t>(), (int)idx.size(), d, p.get(), agg, st);
    });
}

// a dict of addresses by name, torch's functions for the current device and a device's current stream
PyObject *bind(PyObject *const *a)
{
#define GQ_BIND(name)                                                                                                    \
    {                                                                                                                    \
        PyObject *v = PyDict_GetItemString(a[0], #name);                                                                 \
        void *f = v ? PyLong_AsVoidPtr(v) : nullptr;                                                                     \
        if (!f) {                                                                                                        \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);                                               \
            throw Refused();                                                                                             \
        }                                                                                                                \
        lib.name##_ = reinterpret_cast<decltype(&name)>(f);                                                              \
    }
    GQ_ENTRY_POINTS(GQ_BIND)
#undef GQ_BIND
    Py_INCREF(a[1]);
    Py_INCREF(a[2]);
    Py_XSETREF(current_device, a[1]);
    Py_XSETREF(current_raw_stream, a[2]);
    Py_RETURN_NONE;
}

typedef PyObject *(*Fast)(PyObject *, PyObject *const *, Py_ssize_t);
#define GQ_METHOD(name, n, f) {name, (PyCFunction)(void (*)(void))(Fast)entry<n, f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    GQ_METHOD("bind", 3, bind),
    GQ_METHOD("global_norm", 6, global_norm),
    GQ_METHOD("global_norm_static", 5, global_norm_static),
    GQ_METHOD("quantize", 8, quantize),
    GQ_METHOD("int_aggregate", 6, int_aggregate),
    GQ_METHOD("dequantize", 7, dequantize),
    GQ_METHOD("fused_quantize_aggregate", 9, fused_quantize_aggregate),
    GQ_METHOD("bucketed_quantize_aggregate", 11, bucketed_quantize_aggregate),
    GQ_METHOD("exp_reduce", 8, tree_reduce<true>),
    GQ_METHOD("avg_reduce", 8, tree_reduce<false>),
    GQ_METHOD("compact", 9, compact),
    GQ_METHOD("quantize_compact", 11, quantize_compact),
    GQ_METHOD("sparse_aggregate", 8, sparse_aggregate),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    PyObject *m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "built_for", GQ_BUILT_FOR) != 0) Py_CLEAR(m);
    return m;
}
