// _tq_marshal: the per-tensor part of the Python binding.  A batched call takes up to four lists of tensors, of each of
// which the binding wants to know that it is a contiguous device tensor of the right size, and its address; in Python
// that is five attribute calls a tensor and, for small tensors, as long as the launches themselves.
//
// All functions look at plain tensors (torch.Tensor, nn.Parameter), lists and tuples of them and plain numbers, and at nothing
// else: anything they do not know, or that raises, is left to the caller's own Python code, which raises the error.
//
// `pointers` and `sized` look lists over; the functions further down take a whole call -- checks, addresses, stream and the C
// entry point -- because for small tensors the binding's Python code and ctypes took longer than the launch.
#include <cstdint>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tq.h"

namespace {

// Not their subclasses: what one of those hands out may differ from what it stores.
bool plain_sequence(PyObject* seq) { return PyList_CheckExact(seq) || PyTuple_CheckExact(seq); }

// What is asked of the tensors of a list: how many there are (any number where count < 0), their elements and type.
struct Wanted {
    long long count = -1, low = 0, high = INT64_MAX;
    PyObject* dtype = Py_None;
};

// Fills `w` from (count, low, high, dtype); false with an exception set.
bool wanted(PyObject* const* args, Wanted& w)
{
    w.count = PyLong_AsLongLong(args[0]);
    w.low = PyLong_AsLongLong(args[1]);
    w.high = PyLong_AsLongLong(args[2]);
    w.dtype = args[3];
    return !PyErr_Occurred();
}

// Whether `seq` is a list or tuple of as many tensors as are wanted, each of which is as wanted and `use` takes it.
template <typename Use>
bool all_as_wanted(PyObject* seq, const Wanted& w, Use use)
{
    if (!plain_sequence(seq)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    if ((w.count >= 0 && n != w.count) || (w.dtype != Py_None && !THPDtype_Check(w.dtype))) return false;
    try {
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
            if (!THPVariable_CheckExact(o)) return false;
            const at::Tensor& t = THPVariable_Unpack(o);
            const long long elems = t.numel();
            if (elems < w.low || elems > w.high) return false;
            if (w.dtype != Py_None && t.scalar_type() != reinterpret_cast<THPDtype*>(w.dtype)->scalar_type) return false;
            if (!use(i, t)) return false;
        }
    } catch (...) {
        return false;
    }
    return true;
}

// pointers(tensors[, count, low, high, dtype or None]) -> bytes: the addresses, 8 bytes each; None unless all are
// contiguous device tensors and, where that is asked, as `sized` wants them.
PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    Wanted w;
    if (nargs != 1 && nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "pointers takes one argument or five");
        return nullptr;
    }
    if (nargs == 5 && !wanted(args + 1, w)) return nullptr;
    if (!plain_sequence(args[0])) Py_RETURN_NONE;
    PyObject* out = PyBytes_FromStringAndSize(nullptr, PySequence_Fast_GET_SIZE(args[0]) * (Py_ssize_t)sizeof(void*));
    if (!out) return nullptr;
    void** p = reinterpret_cast<void**>(PyBytes_AS_STRING(out));
    const bool usable = all_as_wanted(args[0], w, [&](Py_ssize_t i, const at::Tensor& t) {
        if (!t.is_cuda() || !t.is_contiguous()) return false;
        p[i] = t.data_ptr();
        return true;
    });
    if (usable) return out;
    Py_DECREF(out);
    Py_RETURN_NONE;
}

// sized(tensors, count, low, high, dtype or None) -> bool: whether there are `count` tensors, each of low .. high elements
// and of that dtype.
PyObject* sized(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    Wanted w;
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "sized takes five arguments");
        return nullptr;
    }
    if (!wanted(args + 1, w)) return nullptr;
    if (w.count < 0) Py_RETURN_FALSE;
    return PyBool_FromLong(all_as_wanted(args[0], w, [](Py_ssize_t, const at::Tensor&) { return true; }));
}

// ---- whole calls ------------------------------------------------------------------------------
//
// name(address of the C entry point, the binding's arguments in order) -> its return code, or None for whatever is not as
// plain as can be: the binding's Python code then takes the call from the start.  61,706 elements, host time of a call, us,
// through ctypes / this way: a batch of four
// statistics 5.5 / 4.1, parameters 4.7 / 4.1, compress 5.8 / 4.4, average 5.9 / 4.3 (3.4 of each the launch); one step 30.4 / 24.9.

// The arguments of one call.  `ok` falls once something is not as the fast way wants it; what is read after that is not used.
struct Args {
    PyObject* const* a;
    Py_ssize_t n;
    bool ok;

    Args(PyObject* const* args, Py_ssize_t nargs, Py_ssize_t wanted) : a(args), n(nargs), ok(nargs == wanted) {}

    unsigned long long u64(Py_ssize_t i, unsigned long long most = UINT64_MAX)
    {
        if (!ok || !PyLong_CheckExact(a[i])) return fail();
        const unsigned long long v = PyLong_AsUnsignedLongLong(a[i]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return fail();
        }
        return v <= most ? v : fail();
    }
    int i32(Py_ssize_t i) { return (int)u64(i, INT32_MAX); }       // every int the interface knows is small and not negative
    uint32_t u32(Py_ssize_t i) { return (uint32_t)u64(i, UINT32_MAX); }
    float f32(Py_ssize_t i)
    {
        if (ok && PyFloat_CheckExact(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
        if (!ok || !PyLong_CheckExact(a[i])) return (float)fail();
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(a[i], &overflow);
        return overflow || v > (1 << 24) || v < -(1 << 24) ? (float)fail() : (float)v;   // a whole number that fp32 holds
    }
    int flag(Py_ssize_t i)
    {
        if (!ok || !PyBool_Check(a[i])) return (int)fail();
        return a[i] == Py_True;
    }
    template <typename F> F entry()
    {
        const unsigned long long address = u64(0);
        if (address == 0) ok = false;
        return reinterpret_cast<F>((uintptr_t)address);
    }
    // A contiguous device tensor of low .. high elements; nullptr if it is not one.
    const at::Tensor* tensor(Py_ssize_t i, long long low = 0, long long high = INT64_MAX)
    {
        if (!ok || !THPVariable_CheckExact(a[i])) return fail(), nullptr;
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        const long long elems = t.numel();
        if (elems < low || elems > high || !t.is_cuda() || !t.is_contiguous()) return fail(), nullptr;
        return &t;
    }
    void* address(Py_ssize_t i, long long low, long long high = INT64_MAX)
    {
        const at::Tensor* t = tensor(i, low, high);
        return t ? t->data_ptr() : nullptr;
    }
    void* floats(Py_ssize_t i, long long low = 0, long long high = INT64_MAX)
    {
        const at::Tensor* t = tensor(i, low, high);
        if (t && t->scalar_type() != at::kFloat) ok = false;
        return t ? t->data_ptr() : nullptr;
    }
    unsigned long long fail() { return ok = false, 0; }
};

// A gradient: address, elements, type of the interface.
struct Gradient {
    const void* p = nullptr;
    uint64_t d = 0;
    int dtype = -1;
};

Gradient gradient(Args& in, Py_ssize_t i)
{
    Gradient g;
    const at::Tensor* t = in.tensor(i);
    if (!t) return g;
    g.p = t->data_ptr();
    g.d = (uint64_t)t->numel();
    g.dtype = t->scalar_type() == at::kFloat ? TQ_F32 : (t->scalar_type() == at::kBFloat16 ? TQ_BF16 : -1);
    if (g.dtype < 0) in.ok = false;
    return g;
}

// A batch: `count` addresses (any number if `count` < 0) of contiguous device tensors of low .. high elements, of `type` if there is one.
struct Batch {
    const void* p[TQ_MAX_WORKERS];
    int count = 0;

    Batch(Args& in, Py_ssize_t i, long long count_wanted, long long low, long long high = INT64_MAX, const at::ScalarType* type = nullptr)
    {
        if (!in.ok) return;
        const Py_ssize_t n = plain_sequence(in.a[i]) ? PySequence_Fast_GET_SIZE(in.a[i]) : 0;
        Wanted w;
        w.low = low;
        w.high = high;
        if (n < 1 || n > TQ_MAX_WORKERS || (count_wanted >= 0 && n != count_wanted)) { in.ok = false; return; }
        count = (int)n;
        in.ok = all_as_wanted(in.a[i], w, [&](Py_ssize_t k, const at::Tensor& t) {
            if (!t.is_cuda() || !t.is_contiguous() || (type && t.scalar_type() != *type)) return false;
            p[k] = t.data_ptr();
            return true;
        });
    }
    template <typename T> T* const* as() const { return (T* const*)p; }
};

// The first tensor of a batch, which says what all are.
Gradient first_gradient(Args& in, Py_ssize_t i, at::ScalarType& type)
{
    if (!in.ok || !plain_sequence(in.a[i]) || PySequence_Fast_GET_SIZE(in.a[i]) < 1) return in.ok = false, Gradient();
    PyObject* first = PySequence_Fast_GET_ITEM(in.a[i], 0);
    Args one(&first, 1, 1);
    const Gradient g = gradient(one, 0);
    in.ok = one.ok;
    type = g.dtype == TQ_BF16 ? at::kBFloat16 : at::kFloat;
    return g;
}

long long records(Args& in, uint64_t d, uint64_t bucket_elems)
{
    if (d == 0 || d > (1ull << 40) || bucket_elems > (1ull << 62)) return (long long)in.fail();
    return (long long)(bucket_elems ? (d + bucket_elems - 1) / bucket_elems : 1);
}

long long payload_size(Args& in, uint64_t d, int bits)
{
    if (d > (1ull << 40) || bits < 2 || bits > 4) return (long long)in.fail();
    return (long long)(((d * (uint64_t)bits + 7) / 8 + 15) / 16 * 16);
}

constexpr long long kStats = sizeof(tq_stats_t), kParams = sizeof(tq_params_t);

// The entry point on the current stream, without the interpreter's lock, as ctypes calls it.
template <typename F, typename... A>
PyObject* finish(const Args& in, F f, A... args)
{
    if (!in.ok) Py_RETURN_NONE;
    void* stream = c10::hip::getCurrentHIPStream().stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(args..., stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// g, stats, workspace, bucket_elems, g_min
PyObject* call_stats(Args in)
{
    const auto f = in.entry<decltype(&tq_stats)>();
    const Gradient g = gradient(in, 1);
    const uint64_t be = in.u64(4);
    auto* stats = (tq_stats_t*)in.address(2, records(in, g.d, be) * kStats);
    const at::Tensor* ws = in.tensor(3);
    const float g_min = in.f32(5);
    return finish(in, f, g.p, g.dtype, g.d, be, g_min, stats, ws ? ws->data_ptr() : nullptr, ws ? (uint64_t)ws->numel() : 0);
}

// gs, stats, workspace, bucket_elems, g_min
PyObject* call_stats_multi(Args in)
{
    const auto f = in.entry<decltype(&tq_stats_multi)>();
    at::ScalarType type = at::kFloat;
    const Gradient g = first_gradient(in, 1, type);
    const Batch gs(in, 1, -1, (long long)g.d, INT64_MAX, &type);
    const uint64_t be = in.u64(4);
    const Batch stats(in, 2, gs.count, records(in, g.d, be) * kStats);
    const at::Tensor* ws = in.tensor(3);
    const float g_min = in.f32(5);
    return finish(in, f, gs.as<const void>(), gs.count, g.dtype, g.d, be, g_min, stats.as<tq_stats_t>(), ws ? ws->data_ptr() : nullptr,
                  ws ? (uint64_t)ws->numel() : 0);
}

// stats, params, bits, grid, alpha_override
PyObject* call_params(Args in)
{
    const auto f = in.entry<decltype(&tq_params)>();
    const at::Tensor* stats = in.tensor(1);
    const long long nb = stats ? stats->numel() / kStats : 0;
    auto* params = (tq_params_t*)in.address(2, nb * kParams, nb * kParams);
    const int bits = in.i32(3), grid = in.i32(4);
    const float alpha = in.f32(5);
    return finish(in, f, stats ? (const tq_stats_t*)stats->data_ptr() : nullptr, (uint64_t)nb, bits, grid, alpha, params);
}

// stats, params, bits, grid, alpha_override
PyObject* call_params_multi(Args in)
{
    const auto f = in.entry<decltype(&tq_params_multi)>();
    long long nb = 0;
    if (in.ok && plain_sequence(in.a[1]) && PySequence_Fast_GET_SIZE(in.a[1]) > 0) {
        PyObject* first = PySequence_Fast_GET_ITEM(in.a[1], 0);
        Args one(&first, 1, 1);
        const at::Tensor* t = one.tensor(0);
        in.ok = one.ok;
        nb = t ? t->numel() / kStats : 0;
    }
    const Batch stats(in, 1, -1, nb * kStats), params(in, 2, stats.count, nb * kParams);
    const int bits = in.i32(3), grid = in.i32(4);
    const float alpha = in.f32(5);
    return finish(in, f, stats.as<const tq_stats_t>(), stats.count, (uint64_t)nb, bits, grid, alpha, params.as<tq_params_t>());
}

// g, params, payload, bits, seed, worker, step, bucket_elems, grid
PyObject* call_compress(Args in)
{
    const auto f = in.entry<decltype(&tq_compress)>();
    const Gradient g = gradient(in, 1);
    const int bits = in.i32(4), grid = in.i32(9);
    const uint64_t seed = in.u64(5), be = in.u64(8);
    const uint32_t worker = in.u32(6), step = in.u32(7);
    const long long qbytes = records(in, g.d, be) * kParams;
    const auto* params = (const tq_params_t*)in.address(2, qbytes, qbytes);
    void* payload = in.address(3, payload_size(in, g.d, bits));
    return finish(in, f, g.p, g.dtype, g.d, be, params, bits, grid, seed, worker, step, payload);
}

// gs, params, payloads, bits, seed, first_worker, step, bucket_elems, grid
PyObject* call_compress_multi(Args in)
{
    const auto f = in.entry<decltype(&tq_compress_multi)>();
    at::ScalarType type = at::kFloat;
    const Gradient g = first_gradient(in, 1, type);
    const int bits = in.i32(4), grid = in.i32(9);
    const uint64_t seed = in.u64(5), be = in.u64(8);
    const uint32_t worker = in.u32(6), step = in.u32(7);
    const long long qbytes = records(in, g.d, be) * kParams;
    const Batch gs(in, 1, -1, (long long)g.d, (long long)g.d, &type), params(in, 2, gs.count, qbytes, qbytes),
        payloads(in, 3, gs.count, payload_size(in, g.d, bits));
    return finish(in, f, gs.as<const void>(), gs.count, g.dtype, g.d, be, params.as<const tq_params_t>(), bits, grid, seed, worker, step,
                  payloads.as<void>());
}

// Weights: None, or as many plain floats as there are workers.
struct Weights {
    float w[TQ_MAX_WORKERS];
    const float* p = nullptr;

    Weights(Args& in, Py_ssize_t i, int count)
    {
        if (!in.ok || in.a[i] == Py_None) return;
        if (!plain_sequence(in.a[i]) || PySequence_Fast_GET_SIZE(in.a[i]) != count) { in.ok = false; return; }
        Args each(PySequence_Fast_ITEMS(in.a[i]), count, count);
        for (int k = 0; k < count && each.ok; ++k) w[k] = each.f32(k);
        in.ok = each.ok;
        p = w;
    }
};

// payloads, params, out, bits, bucket_elems, weights, accumulate
PyObject* call_aggregate(Args in)
{
    const auto f = in.entry<decltype(&tq_decompress_aggregate)>();
    const at::Tensor* t = in.tensor(3);
    const uint64_t d = t ? (uint64_t)t->numel() : 0;
    auto* out = (float*)in.floats(3);
    const int bits = in.i32(4);
    const uint64_t be = in.u64(5);
    const long long qbytes = records(in, d, be) * kParams;
    const Batch payloads(in, 1, -1, payload_size(in, d, bits)), params(in, 2, payloads.count, qbytes, qbytes);
    const Weights weights(in, 6, payloads.count);
    const int accumulate = in.flag(7);
    return finish(in, f, payloads.as<const void>(), params.as<const tq_params_t>(), weights.p, payloads.count, d, be, bits, accumulate, out);
}

// payloads, params, theta, bits, eta, momentum, weight_decay, velocity, bucket_elems, weights
PyObject* call_update(Args in)
{
    const auto f = in.entry<decltype(&tq_decompress_aggregate_update)>();
    const at::Tensor* t = in.tensor(3);
    const long long n = t ? t->numel() : 0;
    const uint64_t d = (uint64_t)n;
    auto* theta = (float*)in.floats(3);
    const int bits = in.i32(4);
    const float eta = in.f32(5), momentum = in.f32(6), decay = in.f32(7);
    float* velocity = !in.ok || in.a[8] == Py_None ? nullptr : (float*)in.floats(8, n, n);
    const uint64_t be = in.u64(9);
    const long long qbytes = records(in, d, be) * kParams;
    const Batch payloads(in, 1, -1, payload_size(in, d, bits)), params(in, 2, payloads.count, qbytes, qbytes);
    const Weights weights(in, 10, payloads.count);
    return finish(in, f, payloads.as<const void>(), params.as<const tq_params_t>(), weights.p, payloads.count, d, be, bits, eta, momentum,
                  decay, theta, velocity);
}

// g, params, out, bits, seed, worker, step, bucket_elems, accumulate
PyObject* call_simulate(Args in)
{
    const auto f = in.entry<decltype(&tq_quantize_dequantize)>();
    const Gradient g = gradient(in, 1);
    const int bits = in.i32(4), accumulate = in.flag(9);
    const uint64_t seed = in.u64(5), be = in.u64(8);
    const uint32_t worker = in.u32(6), step = in.u32(7);
    const long long qbytes = records(in, g.d, be) * kParams;
    const auto* params = (const tq_params_t*)in.address(2, qbytes, qbytes);
    auto* out = (float*)in.floats(3, (long long)g.d, (long long)g.d);
    return finish(in, f, g.p, g.dtype, g.d, be, params, bits, seed, worker, step, accumulate, out);
}

// Segments: the table's device address, host address and number of segments, as the binding's Segments gives them.
struct Table {
    const uint64_t *dev, *host;
    uint64_t n;

    Table(Args& in, Py_ssize_t i)
        : dev((const uint64_t*)(uintptr_t)in.u64(i)), host((const uint64_t*)(uintptr_t)in.u64(i + 1)), n(in.u64(i + 2, UINT32_MAX)) {}
};

// g, stats, workspace, g_min, table
PyObject* call_stats_segments(Args in)
{
    const auto f = in.entry<decltype(&tq_stats_segments)>();
    const Gradient g = gradient(in, 1);
    const float g_min = in.f32(4);
    const Table seg(in, 5);
    auto* stats = (tq_stats_t*)in.address(2, (long long)seg.n * kStats);
    const at::Tensor* ws = in.tensor(3);
    return finish(in, f, g.p, g.dtype, g.d, seg.dev, seg.host, seg.n, g_min, stats, ws ? ws->data_ptr() : nullptr,
                  ws ? (uint64_t)ws->numel() : 0);
}

// gs, stats, workspace, g_min, table
PyObject* call_stats_segments_multi(Args in)
{
    const auto f = in.entry<decltype(&tq_stats_segments_multi)>();
    at::ScalarType type = at::kFloat;
    const Gradient g = first_gradient(in, 1, type);
    const float g_min = in.f32(4);
    const Table seg(in, 5);
    const Batch gs(in, 1, -1, (long long)g.d, INT64_MAX, &type), stats(in, 2, gs.count, (long long)seg.n * kStats);
    const at::Tensor* ws = in.tensor(3);
    return finish(in, f, gs.as<const void>(), gs.count, g.dtype, g.d, seg.dev, seg.host, seg.n, g_min, stats.as<tq_stats_t>(),
                  ws ? ws->data_ptr() : nullptr, ws ? (uint64_t)ws->numel() : 0);
}

// g, params, payload, bits, seed, worker, step, table
PyObject* call_compress_segments(Args in)
{
    const auto f = in.entry<decltype(&tq_compress_segments)>();
    const Gradient g = gradient(in, 1);
    const int bits = in.i32(4);
    const uint64_t seed = in.u64(5);
    const uint32_t worker = in.u32(6), step = in.u32(7);
    const Table seg(in, 8);
    const auto* params = (const tq_params_t*)in.address(2, (long long)seg.n * kParams, (long long)seg.n * kParams);
    void* payload = in.address(3, payload_size(in, g.d, bits));
    return finish(in, f, g.p, g.dtype, g.d, seg.dev, seg.host, seg.n, params, bits, seed, worker, step, payload);
}

// gs, params, payloads, bits, seed, first_worker, step, table
PyObject* call_compress_segments_multi(Args in)
{
    const auto f = in.entry<decltype(&tq_compress_segments_multi)>();
    at::ScalarType type = at::kFloat;
    const Gradient g = first_gradient(in, 1, type);
    const int bits = in.i32(4);
    const uint64_t seed = in.u64(5);
    const uint32_t worker = in.u32(6), step = in.u32(7);
    const Table seg(in, 8);
    const long long qbytes = (long long)seg.n * kParams;
    const Batch gs(in, 1, -1, (long long)g.d, (long long)g.d, &type), params(in, 2, gs.count, qbytes, qbytes),
        payloads(in, 3, gs.count, payload_size(in, g.d, bits));
    return finish(in, f, gs.as<const void>(), gs.count, g.dtype, g.d, seg.dev, seg.host, seg.n, params.as<const tq_params_t>(), bits, seed,
                  worker, step, payloads.as<void>());
}

// payloads, params, out, bits, weights, accumulate, table
PyObject* call_aggregate_segments(Args in)
{
    const auto f = in.entry<decltype(&tq_decompress_aggregate_segments)>();
    const at::Tensor* t = in.tensor(3);
    const uint64_t d = t ? (uint64_t)t->numel() : 0;
    auto* out = (float*)in.floats(3);
    const int bits = in.i32(4);
    const Table seg(in, 7);
    const long long qbytes = (long long)seg.n * kParams;
    const Batch payloads(in, 1, -1, payload_size(in, d, bits)), params(in, 2, payloads.count, qbytes, qbytes);
    const Weights weights(in, 5, payloads.count);
    const int accumulate = in.flag(6);
    return finish(in, f, payloads.as<const void>(), params.as<const tq_params_t>(), weights.p, payloads.count, d, seg.dev, seg.host, seg.n,
                  bits, accumulate, out);
}

template <PyObject* (*CALL)(Args), int ARGS>
PyObject* take(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    try {
        return CALL(Args(args, nargs, ARGS));
    } catch (...) {
        Py_RETURN_NONE;
    }
}

template <PyObject* (*CALL)(Args), int ARGS>
PyMethodDef method(const char* name)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&take<CALL, ARGS>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointers)), METH_FASTCALL, nullptr},
    {"sized", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(sized)), METH_FASTCALL, nullptr},
    method<call_stats, 6>("stats"),
    method<call_stats_multi, 6>("stats_multi"),
    method<call_params, 6>("params"),
    method<call_params_multi, 6>("params_multi"),
    method<call_compress, 10>("compress"),
    method<call_compress_multi, 10>("compress_multi"),
    method<call_aggregate, 8>("aggregate"),
    method<call_update, 11>("update"),
    method<call_simulate, 10>("simulate"),
    method<call_stats_segments, 8>("stats_segments"),
    method<call_stats_segments_multi, 8>("stats_segments_multi"),
    method<call_compress_segments, 11>("compress_segments"),
    method<call_compress_segments_multi, 11>("compress_segments_multi"),
    method<call_aggregate_segments, 10>("aggregate_segments"),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tq_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// `interface`: what binding.py asks for before it uses the module; it goes up with every change to the functions or their arguments.
PyMODINIT_FUNC PyInit__tq_marshal()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddIntConstant(m, "interface", 1) != 0) Py_CLEAR(m);
    return m;
}
