// Python module `_native`: the per-call half of binding.py and network.py in native code.
//
// A call on a small layer takes the GPU about 4 us, so what the host spends per call is what such a layer costs.
// Through ctypes (argument conversion, a tensor check and a stream look-up in Python per call) that was 6 - 8 us, of
// which the launch itself is about 2; a network pass of 19 launches was bound by it (181 us of host work against
// 131 us on the GPU).  Here the tensors are unpacked through torch's own C++ interface and the entry point of
// include/apnn.h is called directly; a Chain holds the descriptors and tensors of a whole network and enqueues it
// with one call.  Nothing is computed here, and nothing depends on values: marshalling only.
//
// As with ctypes, the interpreter lock is released while the library runs (a launch can wait for queue space).
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <exception>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/apnn.h"

namespace {

PyObject *g_error = nullptr;                              // binding.ApnnError

void *current_stream() { return static_cast<void *>(c10::hip::getCurrentHIPStream().stream()); }

// Status of a library call -> None, or ApnnError(status, text).
PyObject *finish(int status)
{
    if (status == APNN_OK) Py_RETURN_NONE;
    PyObject *args = Py_BuildValue("(is)", status, apnn_last_error());
    PyObject *e = args && g_error ? PyObject_CallObject(g_error, args) : nullptr;
    Py_XDECREF(args);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_SetString(PyExc_RuntimeError, apnn_last_error());
    }
    return nullptr;
}

// A Python object that is held (made, moved and dropped with the interpreter lock).
class Held {
public:
    explicit Held(PyObject *o) : o_(o) { Py_INCREF(o_); }
    Held(Held &&other) noexcept : o_(std::exchange(other.o_, nullptr)) {}
    Held &operator=(Held &&) = delete;
    ~Held() { Py_XDECREF(o_); }
    PyObject *get() const { return o_; }

private:
    PyObject *o_;
};

// A tensor whose device pointer stands `offset` bytes into a recorded step.  The Python object is held, as by any other
// owner: what it stands for can be exchanged (torch.utils.swap_tensors), which a reference to its tensor would forbid.
struct Ref {
    size_t offset;
    Held tensor;
};

// What a kernel is given of a tensor: its device pointer.  False (Python error set) if it has none that can be used.
bool device_pointer(const at::Tensor &t, void *&p)
{
    if (t.is_cuda() && t.is_contiguous()) {
        p = t.data_ptr();
        return true;
    }
    PyErr_SetString(PyExc_AssertionError, "device, contiguous tensors only");
    return false;
}

// Reads positional arguments in order; after the first failure (Python error set) everything reads as zero.
class Args {
public:
    Args(PyObject *const *a, Py_ssize_t n, Py_ssize_t want) : a_(a)
    {
        if (n != want) { ok_ = false; PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n); }
    }
    bool ok() const { return ok_; }
    PyObject *object() { return ok_ ? a_[i_++] : nullptr; }
    long long integer() { return integer(object()); }
    int small() { return static_cast<int>(integer()); }
    float real() { return real(object()); }
    void *tensor() { return tensor(object()); }

    // Pointers read by `tensor_into` are also noted in `refs`, by their place in the record that starts at `base`.
    void note(const void *base, std::vector<Ref> *refs) { base_ = static_cast<const char *>(base); refs_ = refs; }
    template <class T> void tensor_into(T *&field)
    {
        PyObject *o = object();
        field = static_cast<T *>(tensor(o));
        if (refs_ && ok_ && o != Py_None) refs_->push_back({static_cast<size_t>(reinterpret_cast<const char *>(&field) - base_), Held(o)});
    }

    long long integer(PyObject *o)
    {
        if (!ok_) return 0;
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) {                // (numpy integers and the like)
            PyErr_Clear();
            PyObject *n = PyNumber_Index(o);
            const long long w = n ? PyLong_AsLongLong(n) : 0;
            Py_XDECREF(n);
            if (PyErr_Occurred()) ok_ = false;
            return w;
        }
        return v;
    }
    // what int(o) gives
    int flag()
    {
        PyObject *o = object();
        if (!ok_ || PyLong_Check(o)) return static_cast<int>(integer(o));
        PyObject *n = PyNumber_Long(o);
        if (!n) ok_ = false;
        const int v = static_cast<int>(integer(n));
        Py_XDECREF(n);
        return v;
    }
    float real(PyObject *o)
    {
        if (!ok_) return 0.0f;
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) ok_ = false;
        return static_cast<float>(v);
    }
    // device pointer of a tensor, null for None
    void *tensor(PyObject *o)
    {
        if (!ok_ || o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) {
            ok_ = false;
            PyErr_SetString(PyExc_TypeError, "a torch tensor is expected");
            return nullptr;
        }
        void *p = nullptr;
        ok_ = device_pointer(THPVariable_Unpack(o), p);
        return p;
    }
    // sizes of a tensor of `n` dimensions
    void sizes(PyObject *o, int n, int64_t *out)
    {
        for (int i = 0; i < n; ++i) out[i] = 0;
        if (!ok_) return;
        if (!THPVariable_Check(o)) {
            ok_ = false;
            PyErr_SetString(PyExc_TypeError, "a torch tensor is expected");
            return;
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.dim() != n) {
            ok_ = false;
            PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions is expected, got %lld", n, static_cast<long long>(t.dim()));
            return;
        }
        for (int i = 0; i < n; ++i) out[i] = t.size(i);
    }
    // a binding.Conv (plain attributes)
    apnn_conv_desc conv()
    {
        static const char *const names[13] = {"N", "H", "W", "Cin", "Cout", "R", "S", "stride", "pad", "p", "q", "encW", "encX"};
        static PyObject *keys[13];
        if (!keys[0])
            for (int i = 0; i < 13; ++i) keys[i] = PyUnicode_InternFromString(names[i]);
        PyObject *d = object();
        int64_t v[13] = {};
        for (int i = 0; i < 13 && ok_; ++i) {
            PyObject *o = PyObject_GetAttr(d, keys[i]);
            if (!o) { ok_ = false; break; }
            v[i] = integer(o);
            Py_DECREF(o);
        }
        apnn_conv_desc c;
        c.N = v[0]; c.H = v[1]; c.W = v[2]; c.Cin = v[3]; c.Cout = v[4];
        c.R = static_cast<int>(v[5]); c.S = static_cast<int>(v[6]);
        c.stride = static_cast<int>(v[7]); c.pad = static_cast<int>(v[8]);
        c.p = static_cast<int>(v[9]); c.q = static_cast<int>(v[10]);
        c.encW = static_cast<apnn_encoding>(v[11]); c.encX = static_cast<apnn_encoding>(v[12]);
        return c;
    }

private:
    PyObject *const *a_;
    Py_ssize_t i_ = 0;
    bool ok_ = true;
    const char *base_ = nullptr;
    std::vector<Ref> *refs_ = nullptr;
};

template <class F> PyObject *call(F &&f)
{
    void *stream = current_stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(stream);
    Py_END_ALLOW_THREADS
    return finish(rc);
}

// One layer as apnn_layer takes it: descriptor, weights, features, packed output.
struct Layer {
    apnn_layer_desc L;
    const uint32_t *W, *X;
    uint32_t *out;
};

// (d, W, X, is_gemm, q_out, scale, bias, residual, q_res, res_scale, acc_out, float_out, out, pool)
constexpr Py_ssize_t kLayerArgs = 14;
void read_layer(Args &a, Layer &y)
{
    y.L.conv = a.conv();
    a.tensor_into(y.W);
    a.tensor_into(y.X);
    y.L.is_gemm = a.flag();
    y.L.q_out = a.small();
    a.tensor_into(y.L.scale_dev);
    a.tensor_into(y.L.bias_dev);
    a.tensor_into(y.L.residual_dev);
    y.L.q_res = a.small();
    y.L.res_scale = a.real();
    a.tensor_into(y.L.acc_out_dev);
    a.tensor_into(y.L.float_out_dev);
    if (y.L.q_out > 0) a.tensor_into(y.out);
    else a.object();                                      // (there is no packed output: whatever is given is not looked at)
    y.L.pool = a.small();
}

PyObject *py_set_error(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XDECREF(g_error);
    g_error = cls;
    Py_RETURN_NONE;
}

PyObject *py_pack(PyObject *, PyObject *const *args, Py_ssize_t n)      // (src, bits, enc, out)
{
    Args a(args, n, 4);
    int64_t s[2];
    PyObject *src = a.object();
    a.sizes(src, 2, s);
    const void *p = a.tensor(src);
    const int bits = a.small(), enc = a.small();
    auto *out = static_cast<uint32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_pack(p, s[0], s[1], bits, static_cast<apnn_encoding>(enc), out, st); });
}

PyObject *py_pack_fmap(PyObject *, PyObject *const *args, Py_ssize_t n) // (src, layout, bits, enc, out)
{
    Args a(args, n, 5);
    int64_t s[4];
    PyObject *src = a.object();
    a.sizes(src, 4, s);
    const void *p = a.tensor(src);
    const int layout = a.small(), bits = a.small(), enc = a.small();
    auto *out = static_cast<uint32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    const bool nhwc = layout == APNN_LAYOUT_NHWC;
    return call([&](void *st) {
        return apnn_pack_fmap(p, static_cast<apnn_layout>(layout), s[0], nhwc ? s[1] : s[2], nhwc ? s[2] : s[3], nhwc ? s[3] : s[1],
                              bits, static_cast<apnn_encoding>(enc), out, st);
    });
}

PyObject *py_quantize(PyObject *, PyObject *const *args, Py_ssize_t n)  // (src, zero, step, bits, out)
{
    Args a(args, n, 5);
    int64_t s[2];
    PyObject *src = a.object();
    a.sizes(src, 2, s);
    const auto *p = static_cast<const float *>(a.tensor(src));
    const float zero = a.real(), step = a.real();
    const int bits = a.small();
    auto *out = static_cast<uint32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_quantize(p, s[0], s[1], zero, step, bits, out, st); });
}

PyObject *py_gemm(PyObject *, PyObject *const *args, Py_ssize_t n)      // (W, X, M, N, K, p, q, encW, encX, out)
{
    Args a(args, n, 10);
    const auto *W = static_cast<const uint32_t *>(a.tensor());
    const auto *X = static_cast<const uint32_t *>(a.tensor());
    const int64_t M = a.integer(), N = a.integer(), K = a.integer();
    const int p = a.small(), q = a.small(), encW = a.small(), encX = a.small();
    PyObject *result = a.object();                        // (one without elements is not written, wherever it is)
    const bool empty = result && THPVariable_Check(result) && THPVariable_Unpack(result).numel() == 0;
    auto *out = empty ? nullptr : static_cast<int32_t *>(a.tensor(result));
    if (!a.ok()) return nullptr;
    return call([&](void *st) {
        return apnn_gemm(W, X, out, M, N, K, p, q, static_cast<apnn_encoding>(encW), static_cast<apnn_encoding>(encX), st);
    });
}

PyObject *py_conv2d(PyObject *, PyObject *const *args, Py_ssize_t n)    // (d, W, X, out)
{
    Args a(args, n, 4);
    const apnn_conv_desc d = a.conv();
    const auto *W = static_cast<const uint32_t *>(a.tensor());
    const auto *X = static_cast<const uint32_t *>(a.tensor());
    auto *out = static_cast<int32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_conv2d(&d, W, X, out, st); });
}

PyObject *py_layer(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a(args, n, kLayerArgs);
    Layer y{};
    read_layer(a, y);
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_layer(&y.L, y.W, y.X, y.out, st); });
}

PyObject *py_layer_pair(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a(args, n, 2 * kLayerArgs);
    Layer x{}, y{};
    read_layer(a, x);
    read_layer(a, y);
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_layer_pair(&x.L, x.W, x.X, x.out, &y.L, y.W, y.X, y.out, st); });
}

PyObject *py_input_layer(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    Args a(args, n, kLayerArgs);
    Layer y{};
    read_layer(a, y);
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_input_layer(&y.L, y.W, reinterpret_cast<const uint8_t *>(y.X), y.out, st); });
}

PyObject *py_maxpool(PyObject *, PyObject *const *args, Py_ssize_t n)   // (X, N, H, W, C, bits, k, stride, pad, out)
{
    Args a(args, n, 10);
    const auto *X = static_cast<const uint32_t *>(a.tensor());
    const int64_t N = a.integer(), H = a.integer(), W = a.integer(), C = a.integer();
    const int bits = a.small(), k = a.small(), stride = a.small(), pad = a.small();
    auto *out = static_cast<uint32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_maxpool(X, N, H, W, C, bits, k, stride, pad, out, st); });
}

PyObject *py_sumpool(PyObject *, PyObject *const *args, Py_ssize_t n)   // (X, N, H, W, C, bits, out_bits, out)
{
    Args a(args, n, 8);
    const auto *X = static_cast<const uint32_t *>(a.tensor());
    const int64_t N = a.integer(), H = a.integer(), W = a.integer(), C = a.integer();
    const int bits = a.small(), out_bits = a.small();
    auto *out = static_cast<uint32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_sumpool(X, N, H, W, C, bits, out_bits, out, st); });
}

PyObject *py_sumpool_fc(PyObject *, PyObject *const *args, Py_ssize_t n)    // (X, N, H, W, C, bits, Wt, Cout, p, encW, out)
{
    Args a(args, n, 11);
    const auto *X = static_cast<const uint32_t *>(a.tensor());
    const int64_t N = a.integer(), H = a.integer(), W = a.integer(), C = a.integer();
    const int bits = a.small();
    const auto *Wt = static_cast<const uint32_t *>(a.tensor());
    const int64_t Cout = a.integer();
    const int p = a.small(), encW = a.small();
    auto *out = static_cast<int32_t *>(a.tensor());
    if (!a.ok()) return nullptr;
    return call([&](void *st) { return apnn_sumpool_fc(X, N, H, W, C, bits, Wt, Cout, p, static_cast<apnn_encoding>(encW), out, st); });
}

// ---- Chain: the library calls of a network in order, recorded once (descriptors and the tensors they were given) and
// enqueued by one call.  The tensors are held, and their device pointers are checked and taken anew by every pass, so that
// one whose storage is exchanged is read where it is now, and refused if it now lies on the host or is strided.
struct Step {
    enum Kind { INPUT, LAYER, PAIR, MAXPOOL, SUMPOOL, SUMPOOL_FC } kind;
    Layer a, b;                                           // INPUT, LAYER: a; PAIR: a and b
    // pooling
    const uint32_t *X, *Wt;
    int64_t N, H, W, C, Cout;
    int bits, k, stride, pad, out_bits, p, encW;
    void *out;
};
static_assert(std::is_trivially_copyable<Step>::value, "pointers are written into copies by offset");

struct Record {
    Step step{};
    std::vector<Ref> refs;

    // The step with the pointers of now; false (Python error set) if a tensor has none that can be used.
    bool resolve(Step &s) const
    {
        s = step;
        for (const Ref &r : refs) {
            void *p = nullptr;
            if (!device_pointer(THPVariable_Unpack(r.tensor.get()), p)) return false;
            std::memcpy(reinterpret_cast<char *>(&s) + r.offset, &p, sizeof p);
        }
        return true;
    }
};

struct ChainObject {
    PyObject_HEAD
    std::vector<Record> *records;
};

PyObject *chain_new(PyTypeObject *type, PyObject *, PyObject *)
{
    auto *self = reinterpret_cast<ChainObject *>(type->tp_alloc(type, 0));
    if (self && !(self->records = new (std::nothrow) std::vector<Record>())) {
        Py_DECREF(self);
        return PyErr_NoMemory();
    }
    return reinterpret_cast<PyObject *>(self);
}

void chain_dealloc(PyObject *self)
{
    delete reinterpret_cast<ChainObject *>(self)->records;
    PyTypeObject *type = Py_TYPE(self);
    type->tp_free(self);
    Py_DECREF(type);
}

// Reads one call's arguments with `read` into a new record.
template <class F> PyObject *append(PyObject *self, Args a, Step::Kind kind, F &&read)
{
    Record r;
    r.step.kind = kind;
    a.note(&r.step, &r.refs);
    read(a, r.step);
    if (!a.ok()) return nullptr;
    reinterpret_cast<ChainObject *>(self)->records->push_back(std::move(r));
    Py_RETURN_NONE;
}

PyObject *chain_input_layer(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, kLayerArgs), Step::INPUT, [](Args &a, Step &s) { read_layer(a, s.a); });
}

PyObject *chain_layer(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, kLayerArgs), Step::LAYER, [](Args &a, Step &s) { read_layer(a, s.a); });
}

PyObject *chain_layer_pair(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, 2 * kLayerArgs), Step::PAIR, [](Args &a, Step &s) {
        read_layer(a, s.a);
        read_layer(a, s.b);
    });
}

void read_frame(Args &a, Step &s)
{
    a.tensor_into(s.X);
    s.N = a.integer(); s.H = a.integer(); s.W = a.integer(); s.C = a.integer();
    s.bits = a.small();
}

PyObject *chain_maxpool(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, 10), Step::MAXPOOL, [](Args &a, Step &s) {
        read_frame(a, s);
        s.k = a.small(); s.stride = a.small(); s.pad = a.small();
        a.tensor_into(s.out);
    });
}

PyObject *chain_sumpool(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, 8), Step::SUMPOOL, [](Args &a, Step &s) {
        read_frame(a, s);
        s.out_bits = a.small();
        a.tensor_into(s.out);
    });
}

PyObject *chain_sumpool_fc(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    return append(self, Args(args, n, 11), Step::SUMPOOL_FC, [](Args &a, Step &s) {
        read_frame(a, s);
        a.tensor_into(s.Wt);
        s.Cout = a.integer(); s.p = a.small(); s.encW = a.small();
        a.tensor_into(s.out);
    });
}

int run_step(const Step &s, const void *image, void *stream)
{
    switch (s.kind) {
        case Step::INPUT: return apnn_input_layer(&s.a.L, s.a.W, static_cast<const uint8_t *>(image), s.a.out, stream);
        case Step::LAYER: return apnn_layer(&s.a.L, s.a.W, s.a.X, s.a.out, stream);
        case Step::PAIR: return apnn_layer_pair(&s.a.L, s.a.W, s.a.X, s.a.out, &s.b.L, s.b.W, s.b.X, s.b.out, stream);
        case Step::MAXPOOL:
            return apnn_maxpool(s.X, s.N, s.H, s.W, s.C, s.bits, s.k, s.stride, s.pad, static_cast<uint32_t *>(s.out), stream);
        case Step::SUMPOOL: return apnn_sumpool(s.X, s.N, s.H, s.W, s.C, s.bits, s.out_bits, static_cast<uint32_t *>(s.out), stream);
        case Step::SUMPOOL_FC:
            return apnn_sumpool_fc(s.X, s.N, s.H, s.W, s.C, s.bits, s.Wt, s.Cout, s.p, static_cast<apnn_encoding>(s.encW),
                                   static_cast<int32_t *>(s.out), stream);
    }
    return APNN_ERR_INVALID_ARG;
}

PyObject *chain_run(PyObject *self, PyObject *const *args, Py_ssize_t n)    // (image)
{
    Args a(args, n, 1);
    const void *image = a.tensor();
    if (!a.ok()) return nullptr;
    const auto &records = *reinterpret_cast<ChainObject *>(self)->records;
    std::vector<Step> steps(records.size());              // this pass's own, made while the interpreter lock is held
    for (size_t i = 0; i < records.size(); ++i)
        if (!records[i].resolve(steps[i])) return nullptr;
    return call([&](void *st) {
        for (const Step &s : steps)
            if (const int rc = run_step(s, image, st)) return rc;
        return static_cast<int>(APNN_OK);
    });
}

// What a network is made of, as bytes that stay equal for as long as no entry of any of it is set, exchanged or removed:
// (class of its layers, list of layers, dict of layers, dicts ...).  The interpreter gives a dict a number that no dict has
// had before whenever it is made or modified; a layer counts by the dict of its attributes.  None if it cannot be told:
// containers or layers of another class (what they answer can come from methods), or an interpreter that counts otherwise.
#if PY_VERSION_HEX < 0x030B0000
bool add_version(std::vector<uint64_t> &out, PyObject *dict)
{
    if (!dict || !PyDict_CheckExact(dict)) return false;
    out.push_back(reinterpret_cast<PyDictObject *>(dict)->ma_version_tag);
    return true;
}

bool add_layer_version(std::vector<uint64_t> &out, PyObject *layer, PyObject *cls)
{
    if (reinterpret_cast<PyObject *>(Py_TYPE(layer)) != cls) return false;
    PyObject **dict = _PyObject_GetDictPtr(layer);
    return dict && add_version(out, *dict);
}
#endif

PyObject *py_versions(PyObject *, PyObject *const *args, Py_ssize_t n)
{
#if PY_VERSION_HEX < 0x030B0000
    if (n < 3) { PyErr_SetString(PyExc_TypeError, "a class, a list and at least one dict are expected"); return nullptr; }
    std::vector<uint64_t> tags;
    if (!PyList_CheckExact(args[1]) && !PyTuple_CheckExact(args[1])) Py_RETURN_NONE;
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(args[1]); ++i)
        if (!add_layer_version(tags, PySequence_Fast_GET_ITEM(args[1], i), args[0])) Py_RETURN_NONE;
    for (Py_ssize_t i = 2; i < n; ++i)
        if (!add_version(tags, args[i])) Py_RETURN_NONE;
    PyObject *key, *layer;
    for (Py_ssize_t at = 0; PyDict_Next(args[2], &at, &key, &layer);)
        if (!add_layer_version(tags, layer, args[0])) Py_RETURN_NONE;
    return PyBytes_FromStringAndSize(reinterpret_cast<const char *>(tags.data()), static_cast<Py_ssize_t>(tags.size() * sizeof(uint64_t)));
#else
    Py_RETURN_NONE;
#endif
}

Py_ssize_t chain_length(PyObject *self) { return static_cast<Py_ssize_t>(reinterpret_cast<ChainObject *>(self)->records->size()); }

// What torch or the standard library throws (a tensor without storage or sizes, no device, no memory) becomes a Python
// error: no exception leaves a function that the interpreter calls.
using Function = PyObject *(PyObject *, PyObject *const *, Py_ssize_t);
template <Function F> PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    try {
        return F(self, args, n);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<f>)), METH_FASTCALL, nullptr}

PyMethodDef chain_methods[] = {
    FAST("input_layer", chain_input_layer), FAST("layer", chain_layer), FAST("layer_pair", chain_layer_pair),
    FAST("maxpool", chain_maxpool), FAST("sumpool", chain_sumpool), FAST("sumpool_fc", chain_sumpool_fc),
    FAST("run", chain_run), {nullptr, nullptr, 0, nullptr}};

PyType_Slot chain_slots[] = {{Py_tp_new, reinterpret_cast<void *>(chain_new)}, {Py_tp_dealloc, reinterpret_cast<void *>(chain_dealloc)},
                             {Py_tp_methods, chain_methods}, {Py_sq_length, reinterpret_cast<void *>(chain_length)}, {0, nullptr}};
PyType_Spec chain_spec = {"paper_2106_12169_amd._native.Chain", sizeof(ChainObject), 0, Py_TPFLAGS_DEFAULT, chain_slots};

PyMethodDef methods[] = {
    {"set_error_class", py_set_error, METH_O, nullptr},
    FAST("pack", py_pack), FAST("pack_fmap", py_pack_fmap), FAST("quantize", py_quantize), FAST("gemm", py_gemm),
    FAST("conv2d", py_conv2d), FAST("layer", py_layer), FAST("layer_pair", py_layer_pair), FAST("input_layer", py_input_layer),
    FAST("maxpool", py_maxpool), FAST("sumpool", py_sumpool), FAST("sumpool_fc", py_sumpool_fc), FAST("versions", py_versions),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    PyObject *chain = PyType_FromSpec(&chain_spec);
    if (!chain || PyModule_AddObject(m, "Chain", chain) < 0) {
        Py_XDECREF(chain);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
