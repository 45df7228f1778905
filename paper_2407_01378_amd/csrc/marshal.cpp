// Argument marshalling of the Python binding in native code: every function takes the arguments
// of the binding's function of the same name, turns tensors into pointers and sizes and calls
// the library's entry point.  Returns the status code, or None when an argument is not of the
// plain form expected here (a tensor, a list or tuple of tensors, an int, None): the binding
// then goes through its own checks, which raise the error that describes it.
//
// What bounds a small call is the host: the same marshalling in Python took 11 us of the 22 us
// of an encode + decode pair over eight workers (a method call per tensor and attribute).
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <vector>

#include "thc.h"

namespace {

constexpr Py_ssize_t kMaxList = 64;   // longer lists take the binding's own path

enum Entry {
    kRhtForward, kRhtInverse, kChunkAbsmax, kScaleReduce, kEncode, kAggregate, kDecode, kEncodeAll, kEncodeAllCleared,
    kSatEncodeAll, kSatEncodeAllCleared, kEncodeAllStatic, kWorkspaceClear, kAggregateDecode, kSatAggregateDecode,
    kEncodeAllMinmax, kAggregateDecodeMinmax, kEncodeAllBatch, kAggregateDecodeBatch, kForwardFullDeferred,
    kFullEncodeDeferred, kFullDecodeInverse, kTopkcNorms, kTopkcSumNorms, kTopkcSelect, kTopkcGather, kTopkcScatter,
    kEntries
};
const char* const kNames[kEntries] = {
    "rht_forward", "rht_inverse", "thc_chunk_absmax", "thc_scale_reduce", "thc_encode", "thc_aggregate", "thc_decode",
    "thc_encode_all", "thc_encode_all_cleared", "thc_sat_encode_all", "thc_sat_encode_all_cleared",
    "thc_encode_all_static", "thc_workspace_clear", "thc_aggregate_decode", "thc_sat_aggregate_decode",
    "thc_encode_all_minmax", "thc_aggregate_decode_minmax", "thc_encode_all_batch", "thc_aggregate_decode_batch",
    "rht_forward_full_deferred", "thc_full_encode_deferred", "thc_full_decode_inverse", "topkc_chunk_norms",
    "topkc_sum_norms", "topkc_select", "topkc_gather_sum", "topkc_scatter_mean"};
void* g_entry[kEntries];   // addresses in the loaded library, set once by bind()

template <typename F>
F* entry(Entry e) {
    return reinterpret_cast<F*>(g_entry[e]);
}

// The arguments of one call; `ok` turns false at the first one that is not of the plain form.
struct Args {
    PyObject* const* a;
    bool ok;

    Args(PyObject* const* args, Py_ssize_t given, Py_ssize_t wanted) : a(args), ok(given == wanted) {}

    const at::Tensor* as_tensor(PyObject* o) {
        if (!ok || !THPVariable_Check(o)) {
            ok = false;
            return nullptr;
        }
        return &THPVariable_Unpack(o);
    }
    const at::Tensor* tensor(int i) { return ok ? as_tensor(a[i]) : nullptr; }
    // a contiguous one-dimensional tensor
    const at::Tensor* flat(int i) {
        const at::Tensor* t = tensor(i);
        if (t && (t->dim() != 1 || !t->is_contiguous())) ok = false;
        return t;
    }
    const at::Tensor* flat(int i, at::ScalarType type) {
        const at::Tensor* t = flat(i);
        if (t && t->scalar_type() != type) ok = false;
        return t;
    }
    template <typename T>
    T* ptr(const at::Tensor* t) {
        return ok && t ? static_cast<T*>(t->data_ptr()) : nullptr;
    }
    template <typename T>
    T* ptr(int i) {   // None: a null pointer
        if (!ok || a[i] == Py_None) return nullptr;
        return ptr<T>(tensor(i));
    }
    uint64_t bytes(const at::Tensor* t) { return ok && t ? (uint64_t)t->numel() * t->element_size() : 0u; }
    uint64_t numel(const at::Tensor* t) { return ok && t ? (uint64_t)t->numel() : 0u; }
    int dtype(const at::Tensor* t) {
        if (!ok || !t) return THC_F32;
        if (t->scalar_type() == at::kBFloat16) return THC_BF16;
        if (t->scalar_type() != at::kFloat) ok = false;
        return THC_F32;
    }
    uint64_t as_u64(PyObject* o) {
        if (!ok || !PyLong_CheckExact(o)) {
            ok = false;
            return 0u;
        }
        return PyLong_AsUnsignedLongLongMask(o);
    }
    uint64_t u64(int i) { return ok ? as_u64(a[i]) : 0u; }
    uint32_t u32(int i) { return (uint32_t)u64(i); }
    bool truth(int i) {
        const int t = ok ? PyObject_IsTrue(a[i]) : 0;
        if (t < 0) {   // (it has none, an array of several elements for instance)
            PyErr_Clear();
            ok = false;
        }
        return t == 1;
    }
    void* stream(int i) {
        if (!ok) return nullptr;
        if (a[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* h = PyObject_GetAttrString(a[i], "cuda_stream");
        if (!h) {
            PyErr_Clear();
            ok = false;
            return nullptr;
        }
        void* s = reinterpret_cast<void*>(as_u64(h));
        Py_DECREF(h);
        return s;
    }
};

// A list or tuple of tensors as an array of pointers.
struct List {
    const void* p[kMaxList];
    uint32_t count = 0;
    const at::Tensor* first = nullptr;

    // gradients: flat, of one size and type
    List(Args& c, PyObject* o, bool gradients) {
        const bool list = PyList_CheckExact(o);
        if (!c.ok || (!list && !PyTuple_CheckExact(o))) {
            c.ok = false;
            return;
        }
        const Py_ssize_t n = list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o);
        if (n < 1 || n > kMaxList) {
            c.ok = false;
            return;
        }
        for (Py_ssize_t i = 0; i < n; ++i) {
            const at::Tensor* t = c.as_tensor(list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i));
            if (!t) return;
            if (i == 0) first = t;
            if (gradients && (t->dim() != 1 || !t->is_contiguous() || t->numel() != first->numel() ||
                              t->scalar_type() != first->scalar_type())) {
                c.ok = false;
                return;
            }
            p[i] = t->data_ptr();
        }
        count = (uint32_t)n;
    }
    uint8_t* const* bytes() const { return const_cast<uint8_t* const*>(reinterpret_cast<const uint8_t* const*>(p)); }
};

// Runs the call without the interpreter lock, as ctypes does, and returns its status.
template <typename F>
PyObject* finish(const Args& c, F&& call) {
    if (!c.ok) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = call();
    Py_END_ALLOW_THREADS return PyLong_FromLong(rc);
}

#define THC_FN(NAME) PyObject* NAME(PyObject*, PyObject* const* args, Py_ssize_t n)

// Tensors may throw (a tensor without storage, say, or a subclass that answers in Python, whose error
// may still be pending): the binding's own path then reports it.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    try {
        return F(self, args, n);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

THC_FN(rht_forward_) {   // x, chunk_log2, seed, y, stream
    Args c(args, n, 5);
    const at::Tensor* x = c.flat(0);
    float* y = c.ptr<float>(c.flat(3, at::kFloat));
    const void* px = c.ptr<void>(x);
    const int dt = c.dtype(x);
    const uint64_t count = c.numel(x), seed = c.u64(2);
    const uint32_t l = c.u32(1);
    void* s = c.stream(4);
    return finish(c, [&] { return entry<decltype(rht_forward)>(kRhtForward)(px, dt, count, l, seed, y, s); });
}
THC_FN(rht_inverse_) {   // y, n, chunk_log2, seed, x, stream
    Args c(args, n, 6);
    const float* y = c.ptr<float>(c.flat(0, at::kFloat));
    float* x = c.ptr<float>(c.flat(4, at::kFloat));
    const uint64_t count = c.u64(1), seed = c.u64(3);
    const uint32_t l = c.u32(2);
    void* s = c.stream(5);
    return finish(c, [&] { return entry<decltype(rht_inverse)>(kRhtInverse)(y, count, l, seed, x, s); });
}
THC_FN(chunk_absmax_) {   // grad, chunk_log2, seed, absmax, stream
    Args c(args, n, 5);
    const at::Tensor* g = c.flat(0);
    float* m = c.ptr<float>(c.flat(3, at::kFloat));
    const void* pg = c.ptr<void>(g);
    const int dt = c.dtype(g);
    const uint64_t count = c.numel(g), seed = c.u64(2);
    const uint32_t l = c.u32(1);
    void* s = c.stream(4);
    return finish(c, [&] { return entry<decltype(thc_chunk_absmax)>(kChunkAbsmax)(pg, dt, count, l, seed, m, s); });
}
THC_FN(scale_reduce_) {   // absmax_all, W, chunks, scale, stream
    Args c(args, n, 5);
    const float* m = c.ptr<float>(0);
    const uint32_t W = c.u32(1);
    const uint64_t chunks = c.u64(2);
    float* scale = c.ptr<float>(3);
    void* s = c.stream(4);
    return finish(c, [&] { return entry<decltype(thc_scale_reduce)>(kScaleReduce)(m, W, chunks, scale, s); });
}
THC_FN(encode_) {   // grad, chunk_log2, seed, worker, bits, shared_scale, payload, scale_out, stream
    Args c(args, n, 9);
    const at::Tensor* g = c.flat(0);
    uint8_t* p = c.ptr<uint8_t>(c.flat(6, at::kByte));
    const void* pg = c.ptr<void>(g);
    const int dt = c.dtype(g);
    const uint64_t count = c.numel(g), seed = c.u64(2);
    const uint32_t l = c.u32(1), worker = c.u32(3), bits = c.u32(4);
    const float* scale = c.ptr<float>(5);
    float* scale_out = c.ptr<float>(7);
    void* s = c.stream(8);
    return finish(c, [&] {
        return entry<decltype(thc_encode)>(kEncode)(pg, dt, count, l, seed, worker, bits, scale, p, scale_out, s);
    });
}
THC_FN(aggregate_) {   // payloads, n, chunk_log2, bits, sums, stream
    Args c(args, n, 6);
    if (!c.ok) Py_RETURN_NONE;
    const List p(c, args[0], false);
    const uint64_t count = c.u64(1);
    const uint32_t l = c.u32(2), bits = c.u32(3);
    void* sums = c.ptr<void>(4);
    void* s = c.stream(5);
    return finish(c, [&] { return entry<decltype(thc_aggregate)>(kAggregate)(p.bytes(), p.count, count, l, bits, sums, s); });
}
THC_FN(decode_) {   // sums, scale, W, n, chunk_log2, seed, bits, out, stream
    Args c(args, n, 9);
    float* out = c.ptr<float>(c.flat(7, at::kFloat));
    const void* sums = c.ptr<void>(0);
    const float* scale = c.ptr<float>(1);
    const uint32_t W = c.u32(2), l = c.u32(4), bits = c.u32(6);
    const uint64_t count = c.u64(3), seed = c.u64(5);
    void* s = c.stream(8);
    return finish(c, [&] { return entry<decltype(thc_decode)>(kDecode)(sums, scale, W, count, l, seed, bits, out, s); });
}
template <Entry E>
THC_FN(encode_all_) {   // grads, chunk_log2, seed, bits, payloads, scale, workspace, stream
    Args c(args, n, 8);
    if (!c.ok) Py_RETURN_NONE;
    const List g(c, args[0], true), p(c, args[4], false);
    const int dt = c.dtype(g.first);
    const uint64_t count = c.numel(g.first), seed = c.u64(2);
    const uint32_t l = c.u32(1), bits = c.u32(3);
    float* scale = c.ptr<float>(5);
    const at::Tensor* ws = c.tensor(6);
    void* pw = c.ptr<void>(ws);
    const uint64_t wb = c.bytes(ws);
    void* s = c.stream(7);
    if (g.count != p.count) c.ok = false;
    return finish(c, [&] {
        return entry<decltype(thc_encode_all)>(E)(g.p, dt, g.count, count, l, seed, bits, p.bytes(), scale, pw, wb, s);
    });
}
THC_FN(encode_all_static_) {   // grads, chunk_log2, seed, bits, payloads, scale, timed_out, stream
    Args c(args, n, 8);
    if (!c.ok) Py_RETURN_NONE;
    const List g(c, args[0], true), p(c, args[4], false);
    const int dt = c.dtype(g.first);
    const uint64_t count = c.numel(g.first), seed = c.u64(2);
    const uint32_t l = c.u32(1), bits = c.u32(3);
    float* scale = c.ptr<float>(5);
    uint32_t* timed_out = c.ptr<uint32_t>(6);
    void* s = c.stream(7);
    if (g.count != p.count) c.ok = false;
    return finish(c, [&] {
        return entry<decltype(thc_encode_all_static)>(kEncodeAllStatic)(g.p, dt, g.count, count, l, seed, bits,
                                                                        p.bytes(), scale, timed_out, s);
    });
}
THC_FN(workspace_clear_) {   // workspace, stream
    Args c(args, n, 2);
    const at::Tensor* ws = c.flat(0);
    void* p = c.ptr<void>(ws);
    const uint64_t bytes = c.bytes(ws);
    void* s = c.stream(1);
    return finish(c, [&] { return entry<decltype(thc_workspace_clear)>(kWorkspaceClear)(p, bytes, s); });
}
THC_FN(aggregate_decode_) {   // payloads, scale, n, chunk_log2, seed, bits, sums, out, stream
    Args c(args, n, 9);
    if (!c.ok) Py_RETURN_NONE;
    const List p(c, args[0], false);
    const float* scale = c.ptr<float>(1);
    const uint64_t count = c.u64(2), seed = c.u64(4);
    const uint32_t l = c.u32(3), bits = c.u32(5);
    void* sums = c.ptr<void>(6);
    float* out = c.ptr<float>(c.flat(7, at::kFloat));
    void* s = c.stream(8);
    return finish(c, [&] {
        return entry<decltype(thc_aggregate_decode)>(kAggregateDecode)(p.bytes(), p.count, scale, count, l, seed, bits,
                                                                       sums, out, s);
    });
}
THC_FN(sat_aggregate_decode_) {   // payloads, scale, n, chunk_log2, seed, bits, aggregate, overflow_count, out, stream
    Args c(args, n, 10);
    if (!c.ok) Py_RETURN_NONE;
    const List p(c, args[0], false);
    const float* scale = c.ptr<float>(1);
    const uint64_t count = c.u64(2), seed = c.u64(4);
    const uint32_t l = c.u32(3), bits = c.u32(5);
    uint8_t* aggregate = c.ptr<uint8_t>(6);
    unsigned long long* overflow = c.ptr<unsigned long long>(7);
    float* out = c.ptr<float>(c.flat(8, at::kFloat));
    void* s = c.stream(9);
    return finish(c, [&] {
        return entry<decltype(thc_sat_aggregate_decode)>(kSatAggregateDecode)(p.bytes(), p.count, scale, count, l, seed,
                                                                              bits, aggregate, overflow, out, s);
    });
}
THC_FN(encode_all_minmax_) {   // grads, chunk_log2, seed, bits, rotate, payloads, range, workspace, stream
    Args c(args, n, 9);
    if (!c.ok) Py_RETURN_NONE;
    const List g(c, args[0], true), p(c, args[5], false);
    const int dt = c.dtype(g.first), rotate = c.truth(4);
    const uint64_t count = c.numel(g.first), seed = c.u64(2);
    const uint32_t l = c.u32(1), bits = c.u32(3);
    float* range = c.ptr<float>(6);
    const at::Tensor* ws = c.tensor(7);
    void* pw = c.ptr<void>(ws);
    const uint64_t wb = c.bytes(ws);
    void* s = c.stream(8);
    if (g.count != p.count) c.ok = false;
    return finish(c, [&] {
        return entry<decltype(thc_encode_all_minmax)>(kEncodeAllMinmax)(g.p, dt, g.count, count, l, seed, bits, rotate,
                                                                        p.bytes(), range, pw, wb, s);
    });
}
THC_FN(aggregate_decode_minmax_) {   // payloads, range, n, chunk_log2, seed, bits, rotate, out, stream
    Args c(args, n, 9);
    if (!c.ok) Py_RETURN_NONE;
    const List p(c, args[0], false);
    const float* range = c.ptr<float>(1);
    const uint64_t count = c.u64(2), seed = c.u64(4);
    const uint32_t l = c.u32(3), bits = c.u32(5);
    const int rotate = c.truth(6);
    float* out = c.ptr<float>(c.flat(7, at::kFloat));
    void* s = c.stream(8);
    return finish(c, [&] {
        return entry<decltype(thc_aggregate_decode_minmax)>(kAggregateDecodeMinmax)(p.bytes(), p.count, range, count, l,
                                                                                    seed, bits, rotate, out, s);
    });
}

// ---- batched forms: a list of dicts with keys n, seed, grads, payloads, scale, out
struct Buckets {
    std::vector<thc_bucket> records;
    std::vector<const void*> pointers;   // of all buckets, in order
    uint32_t W = 1;
    int dt = THC_F32;

    enum Key { kN, kSeed, kGrads, kPayloads, kScale, kOut, kKeys };
    static PyObject* value(PyObject* dict, Key k) {   // borrowed; null if absent
        static PyObject* const keys[kKeys] = {
            PyUnicode_InternFromString("n"),        PyUnicode_InternFromString("seed"),
            PyUnicode_InternFromString("grads"),    PyUnicode_InternFromString("payloads"),
            PyUnicode_InternFromString("scale"),    PyUnicode_InternFromString("out")};
        return PyDict_GetItem(dict, keys[k]);
    }
    static PyObject* item(PyObject* dict, Key k) {   // the same, and null if None
        PyObject* o = value(dict, k);
        return o == Py_None ? nullptr : o;
    }
    Buckets(Args& c, PyObject* list, bool encode) {
        if (!c.ok || !PyList_CheckExact(list) || PyList_GET_SIZE(list) == 0) {
            c.ok = false;
            return;
        }
        const Py_ssize_t count = PyList_GET_SIZE(list);
        records.resize((size_t)count);
        pointers.reserve((size_t)count * 2u * 8u);
        std::vector<size_t> at((size_t)count * 2u, (size_t)-1);
        for (Py_ssize_t i = 0; i < count && c.ok; ++i) {
            PyObject* d = PyList_GET_ITEM(list, i);
            if (!PyDict_CheckExact(d)) {
                c.ok = false;
                return;
            }
            thc_bucket& b = records[(size_t)i];
            for (int side = 0; side < 2; ++side) {
                PyObject* o = item(d, side == 0 ? kGrads : kPayloads);
                if (!encode && side == 0) {   // (the decoder reads no gradients, but a list of anything else is an error)
                    if (o) List(c, o, false);
                    if (!c.ok) return;
                    continue;
                }
                if (!o) {   // (what a bucket needs is the library's to check; the first one has to name the workers)
                    if (i == 0 && side == (encode ? 0 : 1)) c.ok = false;
                    continue;
                }
                const List t(c, o, false);
                if (!c.ok) return;
                if (i == 0 && side == (encode ? 0 : 1)) {
                    W = t.count;
                    if (encode) dt = c.dtype(t.first);
                } else if (t.count != W) {   // (the library reads W pointers of each list)
                    c.ok = false;
                }
                at[2u * (size_t)i + side] = pointers.size();
                pointers.insert(pointers.end(), t.p, t.p + t.count);
            }
            PyObject* o = item(d, kScale);
            const at::Tensor* t = o ? c.as_tensor(o) : nullptr;
            b.scale = c.ptr<float>(t);
            o = item(d, kOut);
            t = o ? c.as_tensor(o) : nullptr;
            b.out = c.ptr<float>(t);
            PyObject* count_o = value(d, kN);
            PyObject* seed_o = value(d, kSeed);   // (0 where there is none; None is not a number)
            if (!count_o) c.ok = false;
            b.n = count_o ? c.as_u64(count_o) : 0u;
            b.seed = seed_o ? c.as_u64(seed_o) : 0u;
        }
        for (Py_ssize_t i = 0; i < count; ++i) {
            const size_t g = at[2u * (size_t)i], p = at[2u * (size_t)i + 1u];
            records[(size_t)i].grads = g == (size_t)-1 ? nullptr : pointers.data() + g;
            records[(size_t)i].payloads =
                p == (size_t)-1 ? nullptr
                                : const_cast<uint8_t* const*>(reinterpret_cast<const uint8_t* const*>(pointers.data() + p));
        }
    }
};
THC_FN(encode_all_batch_) {   // buckets, chunk_log2, bits, workspace, stream
    Args c(args, n, 5);
    if (!c.ok) Py_RETURN_NONE;
    const Buckets b(c, args[0], true);
    const uint32_t l = c.u32(1), bits = c.u32(2);
    const at::Tensor* ws = c.tensor(3);
    void* pw = c.ptr<void>(ws);
    const uint64_t wb = c.bytes(ws);
    void* s = c.stream(4);
    return finish(c, [&] {
        return entry<decltype(thc_encode_all_batch)>(kEncodeAllBatch)(b.records.data(), (uint32_t)b.records.size(), b.dt,
                                                                      b.W, l, bits, pw, wb, s);
    });
}
THC_FN(aggregate_decode_batch_) {   // buckets, chunk_log2, bits, workspace, stream
    Args c(args, n, 5);
    if (!c.ok) Py_RETURN_NONE;
    const Buckets b(c, args[0], false);
    const uint32_t l = c.u32(1), bits = c.u32(2);
    const at::Tensor* ws = c.tensor(3);
    void* pw = c.ptr<void>(ws);
    const uint64_t wb = c.bytes(ws);
    void* s = c.stream(4);
    return finish(c, [&] {
        return entry<decltype(thc_aggregate_decode_batch)>(kAggregateDecodeBatch)(
            b.records.data(), (uint32_t)b.records.size(), b.W, l, bits, pw, wb, s);
    });
}

// ---- full rotation
THC_FN(forward_full_deferred_) {   // x, log2_size, seed, y, absmax, stream
    Args c(args, n, 6);
    const at::Tensor* x = c.flat(0);
    float* y = c.ptr<float>(c.flat(3, at::kFloat));
    float* m = c.ptr<float>(c.flat(4, at::kFloat));
    const void* px = c.ptr<void>(x);
    const int dt = c.dtype(x);
    const uint64_t count = c.numel(x), seed = c.u64(2);
    const uint32_t l = c.u32(1);
    void* s = c.stream(5);
    return finish(c, [&] {
        return entry<decltype(rht_forward_full_deferred)>(kForwardFullDeferred)(px, dt, count, l, seed, y, m, s);
    });
}
THC_FN(full_encode_deferred_) {   // y, n, log2_size, seed, worker, bits, scale, payload, stream
    Args c(args, n, 9);
    const float* y = c.ptr<float>(0);
    const uint64_t count = c.u64(1), seed = c.u64(3);
    const uint32_t l = c.u32(2), worker = c.u32(4), bits = c.u32(5);
    const float* scale = c.ptr<float>(6);
    uint8_t* p = c.ptr<uint8_t>(7);
    void* s = c.stream(8);
    return finish(c, [&] {
        return entry<decltype(thc_full_encode_deferred)>(kFullEncodeDeferred)(y, count, l, seed, worker, bits, scale, p, s);
    });
}
THC_FN(full_decode_inverse_) {   // sums, scale, W, n, log2_size, seed, bits, work, x, stream
    Args c(args, n, 10);
    const void* sums = c.ptr<void>(0);
    const float* scale = c.ptr<float>(1);
    const uint32_t W = c.u32(2), l = c.u32(4), bits = c.u32(6);
    const uint64_t count = c.u64(3), seed = c.u64(5);
    float* work = c.ptr<float>(7);
    float* x = c.ptr<float>(8);
    void* s = c.stream(9);
    return finish(c, [&] {
        return entry<decltype(thc_full_decode_inverse)>(kFullDecodeInverse)(sums, scale, W, count, l, seed, bits, work, x, s);
    });
}

// ---- TopKC
THC_FN(topkc_norms_) {   // grad, C, norms, stream
    Args c(args, n, 4);
    const at::Tensor* g = c.flat(0);
    uint16_t* norms = c.ptr<uint16_t>(c.flat(2, at::kHalf));
    const void* pg = c.ptr<void>(g);
    const int dt = c.dtype(g);
    const uint64_t count = c.numel(g);
    const uint32_t C = c.u32(1);
    void* s = c.stream(3);
    return finish(c, [&] { return entry<decltype(topkc_chunk_norms)>(kTopkcNorms)(pg, dt, count, C, norms, s); });
}
THC_FN(topkc_sum_norms_) {   // norms_all, W, P, s, stream
    Args c(args, n, 5);
    const uint16_t* all = c.ptr<uint16_t>(0);
    const uint32_t W = c.u32(1);
    const uint64_t P = c.u64(2);
    uint16_t* sum = c.ptr<uint16_t>(3);
    void* s = c.stream(4);
    return finish(c, [&] { return entry<decltype(topkc_sum_norms)>(kTopkcSumNorms)(all, W, P, sum, s); });
}
THC_FN(topkc_select_) {   // s, J, indices, workspace, stream
    Args c(args, n, 5);
    const at::Tensor* keys = c.flat(0, at::kHalf);
    const uint16_t* pk = c.ptr<uint16_t>(keys);
    const uint64_t P = c.numel(keys);
    uint32_t* idx = c.ptr<uint32_t>(c.flat(2, at::kInt));
    const uint32_t J = c.u32(1);
    const at::Tensor* ws = c.tensor(3);
    void* pw = c.ptr<void>(ws);
    const uint64_t wb = c.bytes(ws);
    void* s = c.stream(4);
    return finish(c, [&] { return entry<decltype(topkc_select)>(kTopkcSelect)(pk, P, J, idx, pw, wb, s); });
}
THC_FN(topkc_gather_sum_) {   // grads, C, indices, J, values, stream
    Args c(args, n, 6);
    if (!c.ok) Py_RETURN_NONE;
    const List g(c, args[0], false);
    const int dt = c.dtype(g.first);
    const uint64_t count = c.numel(g.first);
    const uint32_t C = c.u32(1), J = c.u32(3);
    const uint32_t* idx = c.ptr<uint32_t>(2);
    uint16_t* values = c.ptr<uint16_t>(c.flat(4, at::kHalf));
    void* s = c.stream(5);
    return finish(c, [&] {
        return entry<decltype(topkc_gather_sum)>(kTopkcGather)(g.p, dt, g.count, count, C, idx, J, values, s);
    });
}
THC_FN(topkc_scatter_mean_) {   // values, indices, J, C, W, out, stream
    Args c(args, n, 7);
    const uint16_t* values = c.ptr<uint16_t>(0);
    const uint32_t* idx = c.ptr<uint32_t>(1);
    const uint32_t J = c.u32(2), C = c.u32(3), W = c.u32(4);
    const at::Tensor* o = c.flat(5, at::kFloat);
    float* out = c.ptr<float>(o);
    const uint64_t count = c.numel(o);
    void* s = c.stream(6);
    return finish(c, [&] { return entry<decltype(topkc_scatter_mean)>(kTopkcScatter)(values, idx, J, C, W, count, out, s); });
}

// bind(name, address): where the loaded library's entry point is.
PyObject* bind(PyObject*, PyObject* args) {
    const char* name;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
    for (int e = 0; e < kEntries; ++e)
        if (!strcmp(name, kNames[e])) g_entry[e] = reinterpret_cast<void*>(address);
    Py_RETURN_NONE;
}
PyObject* names(PyObject*, PyObject*) {
    PyObject* t = PyTuple_New(kEntries);
    for (int e = 0; t && e < kEntries; ++e) PyTuple_SET_ITEM(t, e, PyUnicode_FromString(kNames[e]));
    return t;
}

#define THC_METHOD(NAME, FN) \
    { NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<FN>)), METH_FASTCALL, nullptr }
PyMethodDef kMethods[] = {
    THC_METHOD("rht_forward", rht_forward_),
    THC_METHOD("rht_inverse", rht_inverse_),
    THC_METHOD("thc_chunk_absmax", chunk_absmax_),
    THC_METHOD("thc_scale_reduce", scale_reduce_),
    THC_METHOD("thc_encode", encode_),
    THC_METHOD("thc_aggregate", aggregate_),
    THC_METHOD("thc_decode", decode_),
    THC_METHOD("thc_encode_all", encode_all_<kEncodeAll>),
    THC_METHOD("thc_encode_all_cleared", encode_all_<kEncodeAllCleared>),
    THC_METHOD("thc_sat_encode_all", encode_all_<kSatEncodeAll>),
    THC_METHOD("thc_sat_encode_all_cleared", encode_all_<kSatEncodeAllCleared>),
    THC_METHOD("thc_encode_all_static", encode_all_static_),
    THC_METHOD("thc_workspace_clear", workspace_clear_),
    THC_METHOD("thc_aggregate_decode", aggregate_decode_),
    THC_METHOD("thc_sat_aggregate_decode", sat_aggregate_decode_),
    THC_METHOD("thc_encode_all_minmax", encode_all_minmax_),
    THC_METHOD("thc_aggregate_decode_minmax", aggregate_decode_minmax_),
    THC_METHOD("thc_encode_all_batch", encode_all_batch_),
    THC_METHOD("thc_aggregate_decode_batch", aggregate_decode_batch_),
    THC_METHOD("rht_forward_full_deferred", forward_full_deferred_),
    THC_METHOD("thc_full_encode_deferred", full_encode_deferred_),
    THC_METHOD("thc_full_decode_inverse", full_decode_inverse_),
    THC_METHOD("topkc_chunk_norms", topkc_norms_),
    THC_METHOD("topkc_sum_norms", topkc_sum_norms_),
    THC_METHOD("topkc_select", topkc_select_),
    THC_METHOD("topkc_gather_sum", topkc_gather_sum_),
    THC_METHOD("topkc_scatter_mean", topkc_scatter_mean_),
    {"bind", bind, METH_VARARGS, nullptr},
    {"names", names, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&kModule); }
