"""Calls that the host module takes whole do what the binding's Python code and ctypes do, on the same stream."""
import pytest
import torch

from paper_2402_01798_amd import binding as B

pytestmark = pytest.mark.gpu
D, N, BITS, BUCKET = 50_001, 3, 3, 16_384


class State:
    """One step's buffers; every call below writes its own part of them."""

    def __init__(self):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(5)
        self.gs = [torch.randn(D, generator=gen, device="cuda") * 1e-3 for _ in range(N)]
        nb = B.num_buckets(D, BUCKET)
        self.seg = B.Segments([0, 1024, 20_480, D])
        new = lambda size: [torch.zeros(size, dtype=torch.uint8, device="cuda") for _ in range(N)]
        self.stats, self.params, self.payload = new(nb * B.STATS_BYTES), new(nb * B.PARAMS_BYTES), new(B.payload_bytes(D, BITS))
        self.sstats, self.sparams = new(3 * B.STATS_BYTES), new(3 * B.PARAMS_BYTES)
        ws = N * max(B.stats_workspace_bytes(D, BUCKET), B.stats_segments_workspace_bytes(D, 3))
        self.ws = torch.empty(ws, dtype=torch.uint8, device="cuda")
        self.out, self.theta, self.v = (torch.zeros(D, device="cuda") for _ in range(3))

    def steps(self):
        w = [0.5, 0.25, 0.25]
        B.tq_stats(self.gs[0], self.stats[0], self.ws, BUCKET, 1e-4)
        B.tq_stats_multi(self.gs, self.stats, self.ws, BUCKET)
        B.tq_params(self.stats[0], self.params[0], BITS, B.GRID_NONUNIFORM)
        B.tq_params_multi(self.stats, self.params, BITS, B.GRID_UNIFORM, -1)
        B.tq_compress(self.gs[0], self.params[0], self.payload[0], BITS, 7, 0, 1, BUCKET)
        B.tq_compress_multi(self.gs, self.params, self.payload, BITS, 7, 0, 1, BUCKET)
        B.tq_decompress_aggregate(self.payload, self.params, self.out, BITS, BUCKET)
        B.tq_decompress_aggregate(self.payload, self.params, self.out, BITS, BUCKET, w, True)
        B.tq_decompress_aggregate_update(self.payload, self.params, self.theta, BITS, 0.1, 0.9, 1e-3, self.v, BUCKET, w)
        B.tq_quantize_dequantize(self.gs[1], self.params[1], self.out, BITS, 7, 1, 1, BUCKET, True)
        B.tq_stats_segments(self.gs[0], self.seg, self.sstats[0], self.ws)
        B.tq_stats_segments_multi(self.gs, self.seg, self.sstats, self.ws)
        B.tq_params_multi(self.sstats, self.sparams, BITS, B.GRID_BISCALED)
        B.tq_compress_segments(self.gs[0], self.seg, self.sparams[0], self.payload[0], BITS, 7, 0, 2)
        B.tq_compress_segments_multi(self.gs, self.seg, self.sparams, self.payload, BITS, 7, 0, 2)
        B.tq_decompress_aggregate_segments(self.payload, self.sparams, self.seg, self.out, BITS, None, True)

    def all(self):
        torch.cuda.synchronize()
        return [t.clone() for t in self.stats + self.params + self.payload + self.sstats + self.sparams + [self.out, self.theta, self.v]]


def same(a, b):
    return all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(a, b))


def test_same_bytes_as_through_ctypes(monkeypatch):
    taken = []
    real = B._native
    monkeypatch.setattr(B, "_native", lambda name, *a: taken.append(real(name, *a)) or taken[-1])
    native, plain = State(), State()
    native.steps()
    assert len(taken) == 16 and all(taken)                   # every one of them by the module
    monkeypatch.setattr(B, "_tq_marshal", None)
    plain.steps()
    assert len(taken) == 32 and not any(taken[16:])
    assert same(native.all(), plain.all())


def test_the_current_stream_is_the_one_that_is_captured():
    want, got = State(), State()
    want.steps()
    want.steps()
    got.steps()
    for t in (got.out, got.theta, got.v):
        t.zero_()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got.steps()
    torch.cuda.synchronize()
    assert not got.theta.any()                               # recorded, not run
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
    assert same(got.all(), want.all())


def test_refused_by_the_library_as_before():
    s = State()
    for call in (lambda: B.tq_stats(s.gs[0], s.stats[0], s.ws, 16_385),
                 lambda: B.tq_params(s.stats[0], s.params[0], 5, B.GRID_UNIFORM),
                 lambda: B.tq_compress_multi(s.gs, s.params, s.payload, BITS, 7, 0, 1, BUCKET, 9),
                 lambda: B.tq_stats_multi(s.gs, s.stats, s.ws[:16], BUCKET),
                 lambda: B.tq_stats(s.gs[0][1:], s.stats[0], s.ws, BUCKET)):
        with pytest.raises(B.TqError):
            call()
