"""Thin ctypes layer over ``libtq.so``: same names as the C ABI, argument marshalling only.

Tensors are torch CUDA (ROCm) tensors used purely as device memory; every call passes
``data_ptr()`` values and the current HIP stream to the library.  There is no fallback:
if the library is missing or a call fails, an exception is raised.
"""
import ctypes as C
import os
import warnings

import numpy as np
import torch

HERE = os.path.dirname(os.path.abspath(__file__))
try:
    from . import _tq_marshal
    if getattr(_tq_marshal, "interface", 0) != 1:
        raise ImportError("built from other sources than this file's")
except ImportError as e:                # the loops below do the same, slower
    _tq_marshal = None
    if os.path.exists(os.path.join(HERE, "_tq_marshal.so")):
        warnings.warn("_tq_marshal.so does not load, batched calls take longer (build it again: "
                      "`python -m paper_2402_01798_amd.build`): %s" % e, RuntimeWarning)

# TQ_LIBRARY_PATH selects another build of the same library (the tests' grid-fold build)
LIB_PATH = os.environ.get("TQ_LIBRARY_PATH") or os.path.join(HERE, "libtq.so")

OK, EINVAL, EALIGN, EUNSUPPORTED, EHIP = 0, 1, 2, 3, 4
F32, BF16 = 0, 1
GRID_UNIFORM, GRID_NONUNIFORM, GRID_BISCALED = 0, 1, 2
NBINS = 898
MAX_WORKERS = 64
STATS_BYTES = 3632
PARAMS_BYTES = 160

# numpy views of the interface structs (layout fixed by include/tq.h)
STATS_DTYPE = np.dtype([
    ("hist", np.uint32, (NBINS,)), ("n_nonfinite", np.uint32), ("absmax", np.float32),
    ("n", np.uint64), ("g_min", np.float32), ("reserved", np.uint32),
    ("n_tail", np.uint64), ("sum_log_tail", np.float64)], align=True)
PARAMS_DTYPE = np.dtype([
    ("alpha", np.float32), ("bits", np.uint32), ("s", np.uint32), ("grid", np.uint32),
    ("level", np.float32, (16,)), ("inv_w", np.float32, (16,)),
    ("gamma_hat", np.float32), ("rho_hat", np.float32), ("g_min", np.float32),
    ("flags", np.uint32)], align=True)
assert STATS_DTYPE.itemsize == STATS_BYTES and PARAMS_DTYPE.itemsize == PARAMS_BYTES


class TqError(RuntimeError):
    def __init__(self, code, what):
        self.code = code
        super().__init__("%s: %s (code %d)" % (what, strerror(code), code))


_lib = None


def lib():
    """The loaded library; raises if it has not been built (no fallback exists)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(
                "%s not found: build it with `python -m paper_2402_01798_amd.build`" % LIB_PATH)
        L = C.CDLL(LIB_PATH)
        u64, u32, i32, f32, vp = C.c_uint64, C.c_uint32, C.c_int, C.c_float, C.c_void_p
        L.tq_num_buckets.argtypes = [u64, u64]
        L.tq_num_buckets.restype = u64
        L.tq_payload_bytes.argtypes = [u64, i32]
        L.tq_payload_bytes.restype = u64
        L.tq_stats_workspace_bytes.argtypes = [u64, u64]
        L.tq_stats_workspace_bytes.restype = u64
        L.tq_stats.argtypes = [vp, i32, u64, u64, f32, vp, vp, u64, vp]
        L.tq_stats_static.argtypes = [vp, i32, u64, u64, f32, vp, vp]
        L.tq_params.argtypes = [vp, u64, i32, i32, f32, vp, vp]
        L.tq_compress.argtypes = [vp, i32, u64, u64, vp, i32, i32, u64, u32, u32, vp, vp]
        L.tq_decompress_aggregate.argtypes = [vp, vp, vp, i32, u64, u64, i32, i32, vp, vp]
        L.tq_decompress_aggregate_update.argtypes = [vp, vp, vp, i32, u64, u64, i32, f32, f32, f32, vp, vp, vp]
        L.tq_quantize_dequantize.argtypes = [vp, i32, u64, u64, vp, i32, u64, u32, u32, i32, vp, vp]
        L.tq_quantize_dequantize.restype = i32
        L.tq_strerror.argtypes = [i32]
        L.tq_strerror.restype = C.c_char_p
        L.tq_stats_multi.argtypes = [vp, i32, i32, u64, u64, f32, vp, vp, u64, vp]
        L.tq_params_multi.argtypes = [vp, i32, u64, i32, i32, f32, vp, vp]
        L.tq_compress_multi.argtypes = [vp, i32, i32, u64, u64, vp, i32, i32, u64, u32, u32, vp, vp]
        L.tq_stats_segments_workspace_bytes.argtypes = [u64, u64]
        L.tq_stats_segments_workspace_bytes.restype = u64
        L.tq_stats_segments.argtypes = [vp, i32, u64, vp, vp, u64, f32, vp, vp, u64, vp]
        L.tq_compress_segments.argtypes = [vp, i32, u64, vp, vp, u64, vp, i32, u64, u32, u32, vp, vp]
        L.tq_decompress_aggregate_segments.argtypes = [vp, vp, vp, i32, u64, vp, vp, u64, i32, i32, vp, vp]
        L.tq_stats_segments_multi.argtypes = [vp, i32, i32, u64, vp, vp, u64, f32, vp, vp, u64, vp]
        L.tq_compress_segments_multi.argtypes = [vp, i32, i32, u64, vp, vp, u64, vp, i32, u64, u32, u32, vp, vp]
        for f in (L.tq_stats_segments, L.tq_compress_segments, L.tq_decompress_aggregate_segments,
                  L.tq_stats_segments_multi, L.tq_compress_segments_multi):
            f.restype = i32
        for f in (L.tq_stats, L.tq_stats_static, L.tq_params, L.tq_compress, L.tq_decompress_aggregate,
                  L.tq_decompress_aggregate_update, L.tq_stats_multi, L.tq_params_multi, L.tq_compress_multi):
            f.restype = i32
        for name in _NATIVE:
            f = getattr(L, name)
            f.address = C.cast(f, C.c_void_p).value
        _lib = L
    return _lib


# Calls whose arguments are plain tensors, lists of them and plain numbers are taken whole by the host module, which looks at
# them as the code below does; it answers None for everything else, errors among it, and the code below takes the call.
_NATIVE = {"tq_stats": "stats", "tq_stats_multi": "stats_multi", "tq_params": "params", "tq_params_multi": "params_multi",
           "tq_compress": "compress", "tq_compress_multi": "compress_multi", "tq_decompress_aggregate": "aggregate",
           "tq_decompress_aggregate_update": "update", "tq_quantize_dequantize": "simulate",
           "tq_stats_segments": "stats_segments", "tq_stats_segments_multi": "stats_segments_multi",
           "tq_compress_segments": "compress_segments", "tq_compress_segments_multi": "compress_segments_multi",
           "tq_decompress_aggregate_segments": "aggregate_segments"}


def _native(name, *args):
    """Whether the host module has made the call; a code other than OK raises."""
    if _tq_marshal is None:
        return False
    rc = getattr(_tq_marshal, _NATIVE[name])(getattr(getattr(lib(), name), "address", 0), *args)
    if rc:
        raise TqError(rc, name)
    return rc is not None


def strerror(code):
    return lib().tq_strerror(code).decode()


def _check(rc, what):
    if rc != OK:
        raise TqError(rc, what)


# Host time per call is what bounds small tensors, so addresses are passed as plain integers (ctypes
# converts them by the declared argument types), sizes that all tensors of a batch share are computed
# once, and the stream handle is read without building a torch Stream object (3 us of an 8 us call).
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream():
    if _raw_stream is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(torch.cuda.current_device())


def _dtype_code(g):
    if g.dtype == torch.float32:
        return F32
    if g.dtype == torch.bfloat16:
        return BF16
    raise TypeError("gradient must be float32 or bfloat16, got %s" % g.dtype)


def _dev(t, what):
    if not (t.is_cuda and t.is_contiguous()):
        raise ValueError("%s must be a contiguous device tensor" % what)
    return t.data_ptr()


def num_buckets(d, bucket_elems=0):
    return int(lib().tq_num_buckets(d, bucket_elems))


def payload_bytes(d, bits):
    return int(lib().tq_payload_bytes(d, bits))


def alloc_stats(d, bucket_elems=0, device="cuda"):
    return torch.empty(num_buckets(d, bucket_elems) * STATS_BYTES, dtype=torch.uint8, device=device)


def stats_workspace_bytes(d, bucket_elems=0):
    return int(lib().tq_stats_workspace_bytes(d, bucket_elems))


def alloc_stats_workspace(d, bucket_elems=0, device="cuda"):
    return torch.empty(stats_workspace_bytes(d, bucket_elems), dtype=torch.uint8, device=device)


def alloc_params(d, bucket_elems=0, device="cuda"):
    return torch.empty(num_buckets(d, bucket_elems) * PARAMS_BYTES, dtype=torch.uint8, device=device)


def alloc_payload(d, bits, device="cuda"):
    return torch.empty(payload_bytes(d, bits), dtype=torch.uint8, device=device)


def _records(d, bucket_elems):
    """num_buckets; a call into the library (0.4 us) only for what it refuses later."""
    if bucket_elems == 0 and d:
        return 1
    return -(-d // bucket_elems) if bucket_elems > 0 else num_buckets(d, bucket_elems)


def _stats_bytes(d, bucket_elems):
    """Bytes of the records tq_stats writes, without a call into the library."""
    return -(-d // bucket_elems) * STATS_BYTES if bucket_elems > 0 else STATS_BYTES if d else 0


def _holds(buf, nbytes, what):
    if buf.numel() < nbytes and buf.nbytes < nbytes:
        raise ValueError("%s buffer too small: %d bytes of %d" % (what, buf.nbytes, nbytes))


def tq_stats(g, stats, workspace, bucket_elems=0, g_min=0.0):
    if _native("tq_stats", g, stats, workspace, bucket_elems, g_min):
        return stats
    d = g.numel()
    if stats.numel() < (_stats_bytes(d, bucket_elems) if bucket_elems else STATS_BYTES):
        _holds(stats, _stats_bytes(d, bucket_elems), "stats")
    _check(lib().tq_stats(_dev(g, "g"), _dtype_code(g), d, bucket_elems, g_min,
                          _dev(stats, "stats"), _dev(workspace, "workspace"), workspace.numel(),
                          _stream()), "tq_stats")
    return stats


def tq_stats_static(g, stats, bucket_elems=0, g_min=0.0):
    d = g.numel()
    if stats.numel() < (_stats_bytes(d, bucket_elems) if bucket_elems else STATS_BYTES):
        _holds(stats, _stats_bytes(d, bucket_elems), "stats")
    _check(lib().tq_stats_static(_dev(g, "g"), _dtype_code(g), d, bucket_elems, g_min,
                                 _dev(stats, "stats"), _stream()), "tq_stats_static")
    return stats


def tq_params(stats, params, bits, grid, alpha_override=0.0):
    if _native("tq_params", stats, params, bits, grid, alpha_override):
        return params
    nb = stats.numel() // STATS_BYTES
    if params.numel() != nb * PARAMS_BYTES:
        raise ValueError("params buffer does not match the number of buckets")
    _check(lib().tq_params(_dev(stats, "stats"), nb, bits, grid, alpha_override,
                           _dev(params, "params"), _stream()), "tq_params")
    return params


def tq_compress(g, params, payload, bits, seed, worker, step, bucket_elems=0, grid=GRID_UNIFORM):
    """``grid``: the family ``params`` was designed with; it only shapes the launch (see tq.h)."""
    if _native("tq_compress", g, params, payload, bits, seed, worker, step, bucket_elems, grid):
        return payload
    d = g.numel()
    if params.numel() != _records(d, bucket_elems) * PARAMS_BYTES:
        raise ValueError("params buffer does not match the number of buckets")
    if payload.numel() < payload_bytes(d, bits):
        raise ValueError("payload buffer too small")
    _check(lib().tq_compress(_dev(g, "g"), _dtype_code(g), d, bucket_elems, _dev(params, "params"),
                             bits, grid, seed, worker, step, _dev(payload, "payload"), _stream()),
           "tq_compress")
    return payload


def tq_quantize_dequantize(g, params, out, bits, seed, worker, step, bucket_elems=0, accumulate=False):
    if _native("tq_quantize_dequantize", g, params, out, bits, seed, worker, step, bucket_elems, accumulate):
        return out
    d = g.numel()
    if params.numel() != _records(d, bucket_elems) * PARAMS_BYTES:
        raise ValueError("params buffer does not match the number of buckets")
    if out.dtype != torch.float32 or out.numel() != d:
        raise ValueError("out must be float32 of the gradient's size")
    _check(lib().tq_quantize_dequantize(_dev(g, "g"), _dtype_code(g), d, bucket_elems, _dev(params, "params"),
                                        bits, seed, worker, step, int(bool(accumulate)), _dev(out, "out"),
                                        _stream()), "tq_quantize_dequantize")
    return out


# Batches of plain tensors are looked over by the host module: 61,706 elements x 4 workers, host time of the four calls of
# a step 11.2 + 7.6 + 11.4 + 9.9 -> 5.8 + 5.1 + 6.4 + 6.4 us (one statistics launch instead of two among it).  What it does not
# take, and every error, is left to the Python code.
_ANY_SIZE = (1 << 63) - 1


def _sized(tensors, count, low, high, dtype=None):
    return _tq_marshal is not None and _tq_marshal.sized(tensors, count, low, high, dtype)


def _one_each(count, buffers, what):
    """The library reads `count` addresses, however many the list holds: one that is too short is refused here."""
    if len(buffers) < count:
        raise ValueError("%d %s buffers for a batch of %d tensors" % (len(buffers), what, count))


def _each_holds(count, buffers, nbytes, what):
    for _, buf in zip(range(count), buffers):
        _holds(buf, nbytes, what)


def _ptr_array(tensors, what):
    ptrs = None if _tq_marshal is None else _tq_marshal.pointers(tensors)
    if ptrs is not None:
        return ptrs
    return (C.c_void_p * len(tensors))(*[_dev(t, what) for t in tensors])


def _stats_batch(gs, stats, d, dtype, nbytes):
    """The two address arrays.  The first tensor's elements are read of every tensor (longer ones have them), `nbytes`
    written to every buffer."""
    m, n = _tq_marshal, len(gs)
    if m is not None:
        gp, sp = m.pointers(gs, n, d, _ANY_SIZE, dtype), m.pointers(stats, n, nbytes, _ANY_SIZE, None)
        if gp is not None and sp is not None:
            return gp, sp
    _one_each(n, stats, "stats")
    if any(g.numel() < d or g.dtype != dtype for g in gs):
        raise ValueError("batched tensors must share shape and dtype")
    _each_holds(n, stats, nbytes, "stats")
    return _ptr_array(gs, "g"), _ptr_array(stats, "stats")


def _params_batch(stats, params, nb):
    m, n, sbytes, qbytes = _tq_marshal, len(stats), nb * STATS_BYTES, nb * PARAMS_BYTES
    if m is not None:
        sp, qp = m.pointers(stats, n, sbytes, _ANY_SIZE, None), m.pointers(params, n, qbytes, _ANY_SIZE, None)
        if sp is not None and qp is not None:
            return sp, qp
    _one_each(n, params, "params")
    _each_holds(n, stats, sbytes, "stats")
    _each_holds(n, params, qbytes, "params")
    return _ptr_array(stats, "stats"), _ptr_array(params, "params")


def _compress_batch(gs, params, payloads, d, dtype, qbytes, pbytes, of):
    m, n = _tq_marshal, len(gs)
    if m is not None:
        gp, qp = m.pointers(gs, n, d, d, dtype), m.pointers(params, n, qbytes, qbytes, None)
        pp = m.pointers(payloads, n, pbytes, _ANY_SIZE, None)
        if gp is not None and qp is not None and pp is not None:
            return gp, qp, pp
    _one_each(n, params, "params")
    _one_each(n, payloads, "payload")
    for g, q, p in zip(gs, params, payloads):
        if g.numel() != d or g.dtype != dtype:
            raise ValueError("batched tensors must share shape and dtype")
        if q.numel() != qbytes or p.numel() < pbytes:
            raise ValueError("params / payload buffer size does not match " + of)
    return _ptr_array(gs, "g"), _ptr_array(params, "params"), _ptr_array(payloads, "payload")


def tq_stats_multi(gs, stats, workspace, bucket_elems=0, g_min=0.0):
    """Batched tq_stats: lists of same-shaped gradients and their stats buffers."""
    if _native("tq_stats_multi", gs, stats, workspace, bucket_elems, g_min):
        return stats
    g = gs[0]
    d = g.numel()
    gp, sp = _stats_batch(gs, stats, d, g.dtype, _stats_bytes(d, bucket_elems))
    _check(lib().tq_stats_multi(gp, len(gs), _dtype_code(g), d, bucket_elems, g_min, sp,
                                _dev(workspace, "workspace"), workspace.numel(), _stream()),
           "tq_stats_multi")
    return stats


def tq_params_multi(stats, params, bits, grid, alpha_override=0.0):
    if _native("tq_params_multi", stats, params, bits, grid, alpha_override):
        return params
    nb = stats[0].numel() // STATS_BYTES
    sp, qp = _params_batch(stats, params, nb)
    _check(lib().tq_params_multi(sp, len(stats), nb, bits, grid, alpha_override, qp, _stream()), "tq_params_multi")
    return params


def tq_compress_multi(gs, params, payloads, bits, seed, first_worker, step, bucket_elems=0, grid=GRID_UNIFORM):
    if _native("tq_compress_multi", gs, params, payloads, bits, seed, first_worker, step, bucket_elems, grid):
        return payloads
    d, dtype = gs[0].numel(), gs[0].dtype
    gp, qp, pp = _compress_batch(gs, params, payloads, d, dtype, _records(d, bucket_elems) * PARAMS_BYTES, payload_bytes(d, bits), "d")
    _check(lib().tq_compress_multi(gp, len(gs), _dtype_code(gs[0]), d, bucket_elems, qp, bits, grid, seed, first_worker, step,
                                   pp, _stream()), "tq_compress_multi")
    return payloads


def _decode_args(payloads, params, d, bits, bucket_elems, weights):
    N = len(payloads)
    if len(params) != N:
        raise ValueError("one params buffer per payload")
    psize, qsize = payload_bytes(d, bits), _records(d, bucket_elems) * PARAMS_BYTES
    if not (_sized(payloads, N, psize, _ANY_SIZE) and _sized(params, N, qsize, qsize)):
        for p, q in zip(payloads, params):
            if p.numel() < psize or q.numel() != qsize:
                raise ValueError("payload / params buffer size does not match d")
    pp, qq = _ptr_array(payloads, "payload"), _ptr_array(params, "params")
    ww = None
    if weights is not None:
        if len(weights) != N:
            raise ValueError("one weight per worker")
        ww = (C.c_float * N)(*[float(w) for w in weights])
    return pp, qq, ww, N


def tq_decompress_aggregate(payloads, params, out, bits, bucket_elems=0, weights=None,
                            accumulate=False):
    if _native("tq_decompress_aggregate", payloads, params, out, bits, bucket_elems, weights, accumulate):
        return out
    d = out.numel()
    if out.dtype != torch.float32:
        raise TypeError("out must be float32")
    pp, qq, ww, N = _decode_args(payloads, params, d, bits, bucket_elems, weights)
    _check(lib().tq_decompress_aggregate(pp, qq, ww, N, d, bucket_elems, bits, int(bool(accumulate)),
                                         _dev(out, "out"), _stream()), "tq_decompress_aggregate")
    return out


def tq_decompress_aggregate_update(payloads, params, theta, bits, eta, momentum=0.0, weight_decay=0.0,
                                   velocity=None, bucket_elems=0, weights=None):
    if _native("tq_decompress_aggregate_update", payloads, params, theta, bits, eta, momentum, weight_decay, velocity, bucket_elems,
               weights):
        return theta
    d = theta.numel()
    if theta.dtype != torch.float32 or (velocity is not None and velocity.dtype != torch.float32):
        raise TypeError("theta and velocity must be float32")
    if velocity is not None and velocity.numel() != d:
        raise ValueError("velocity must have theta's size")
    pp, qq, ww, N = _decode_args(payloads, params, d, bits, bucket_elems, weights)
    _check(lib().tq_decompress_aggregate_update(
        pp, qq, ww, N, d, bucket_elems, bits, float(eta), float(momentum), float(weight_decay),
        _dev(theta, "theta"), None if velocity is None else _dev(velocity, "velocity"), _stream()),
        "tq_decompress_aggregate_update")
    return theta


class Segments:
    """A segment table in both memories: ``offsets`` (host, numpy uint64, nseg + 1 entries) and
    its device copy.  Pure marshalling: the library checks the host copy."""

    def __init__(self, offsets, device="cuda"):
        self.host = np.ascontiguousarray(offsets, dtype=np.uint64)
        self.dev = torch.from_numpy(self.host.view(np.int64).copy()).to(device)
        self.nseg = self.host.size - 1
        self.d = int(self.host[-1])

    def args(self):
        return self.dev.data_ptr(), self.host.ctypes.data, self.nseg


def stats_segments_workspace_bytes(d, nseg):
    return int(lib().tq_stats_segments_workspace_bytes(d, nseg))


def tq_stats_segments(g, seg, stats, workspace, g_min=0.0):
    if _native("tq_stats_segments", g, stats, workspace, g_min, *seg.args()):
        return stats
    _holds(stats, seg.nseg * STATS_BYTES, "stats")
    dev, host, nseg = seg.args()
    _check(lib().tq_stats_segments(_dev(g, "g"), _dtype_code(g), g.numel(), dev, host, nseg, g_min,
                                   _dev(stats, "stats"), _dev(workspace, "workspace"), workspace.numel(),
                                   _stream()), "tq_stats_segments")
    return stats


def tq_compress_segments(g, seg, params, payload, bits, seed, worker, step):
    if _native("tq_compress_segments", g, params, payload, bits, seed, worker, step, *seg.args()):
        return payload
    d = g.numel()
    if params.numel() != seg.nseg * PARAMS_BYTES or payload.numel() < payload_bytes(d, bits):
        raise ValueError("params / payload buffer size does not match the segments")
    dev, host, nseg = seg.args()
    _check(lib().tq_compress_segments(_dev(g, "g"), _dtype_code(g), d, dev, host, nseg, _dev(params, "params"),
                                      bits, seed, worker, step, _dev(payload, "payload"), _stream()),
           "tq_compress_segments")
    return payload


def tq_stats_segments_multi(gs, seg, stats, workspace, g_min=0.0):
    """Batched tq_stats_segments: same-shaped gradients that share the segment table."""
    if _native("tq_stats_segments_multi", gs, stats, workspace, g_min, *seg.args()):
        return stats
    g = gs[0]
    gp, sp = _stats_batch(gs, stats, g.numel(), g.dtype, seg.nseg * STATS_BYTES)
    dev, host, nseg = seg.args()
    _check(lib().tq_stats_segments_multi(gp, len(gs), _dtype_code(g), g.numel(), dev, host,
                                         nseg, g_min, sp, _dev(workspace, "workspace"),
                                         workspace.numel(), _stream()), "tq_stats_segments_multi")
    return stats


def tq_compress_segments_multi(gs, seg, params, payloads, bits, seed, first_worker, step):
    if _native("tq_compress_segments_multi", gs, params, payloads, bits, seed, first_worker, step, *seg.args()):
        return payloads
    d, dtype = gs[0].numel(), gs[0].dtype
    gp, qp, pp = _compress_batch(gs, params, payloads, d, dtype, seg.nseg * PARAMS_BYTES, payload_bytes(d, bits), "the segments")
    dev, host, nseg = seg.args()
    _check(lib().tq_compress_segments_multi(gp, len(gs), _dtype_code(gs[0]), d, dev, host, nseg, qp, bits, seed, first_worker,
                                            step, pp, _stream()), "tq_compress_segments_multi")
    return payloads


def tq_decompress_aggregate_segments(payloads, params, seg, out, bits, weights=None, accumulate=False):
    if _native("tq_decompress_aggregate_segments", payloads, params, out, bits, weights, accumulate, *seg.args()):
        return out
    d = out.numel()
    if out.dtype != torch.float32:
        raise TypeError("out must be float32")
    N = len(payloads)
    psize, qsize = payload_bytes(d, bits), seg.nseg * PARAMS_BYTES
    if not (_sized(payloads, N, psize, _ANY_SIZE) and _sized(params, N, qsize, qsize)):
        _one_each(N, params, "params")
        for p, q in zip(payloads, params):
            if p.numel() < psize or q.numel() != qsize:
                raise ValueError("payload / params buffer size does not match the segments")
    pp, qq = _ptr_array(payloads, "payload"), _ptr_array(params, "params")
    ww = None if weights is None else (C.c_float * N)(*[float(w) for w in weights])
    dev, host, nseg = seg.args()
    _check(lib().tq_decompress_aggregate_segments(pp, qq, ww, N, d, dev, host, nseg, bits, int(bool(accumulate)),
                                                  _dev(out, "out"), _stream()), "tq_decompress_aggregate_segments")
    return out


def stats_to_numpy(stats):
    """Host copy of a stats buffer as a structured array (synchronises)."""
    return stats.cpu().numpy().view(STATS_DTYPE)


def params_to_numpy(params):
    """Host copy of a params buffer as a structured array (synchronises)."""
    return params.cpu().numpy().view(PARAMS_DTYPE)


def params_from_numpy(arr, device="cuda"):
    """Device buffer holding the given PARAMS_DTYPE-compatible records (same byte layout)."""
    raw = np.ascontiguousarray(arr).view(np.uint8).reshape(-1)
    return torch.from_numpy(raw.copy()).to(device)
