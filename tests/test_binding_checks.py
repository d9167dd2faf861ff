"""What the binding refuses because the device would read or write past a buffer: lists shorter than the batch (the library
reads one address per tensor of it), tensors of a batch that differ, buffers too small for their records."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2402_01798_amd import binding as B

D = 1024
G = [torch.zeros(D) for _ in range(3)]
STATS = [torch.zeros(B.STATS_BYTES, dtype=torch.uint8) for _ in range(3)]
PARAMS = [torch.zeros(B.PARAMS_BYTES, dtype=torch.uint8) for _ in range(3)]
PAYLOADS = [torch.zeros(B.payload_bytes(D, 3), dtype=torch.uint8) for _ in range(3)]
WORKSPACE = torch.zeros(1 << 20, dtype=torch.uint8)
SEG = B.Segments([0, 128, D], device="cpu")
SEG_STATS = [torch.zeros(2 * B.STATS_BYTES, dtype=torch.uint8) for _ in range(3)]
SEG_PARAMS = [torch.zeros(2 * B.PARAMS_BYTES, dtype=torch.uint8) for _ in range(3)]

CALLS = {
    "stats": lambda n: B.tq_stats_multi(G, STATS[:n], WORKSPACE),
    "params": lambda n: B.tq_params_multi(STATS, PARAMS[:n], 3, B.GRID_UNIFORM),
    "compress-params": lambda n: B.tq_compress_multi(G, PARAMS[:n], PAYLOADS, 3, 1, 0, 0),
    "compress-payload": lambda n: B.tq_compress_multi(G, PARAMS, PAYLOADS[:n], 3, 1, 0, 0),
    "segments-stats": lambda n: B.tq_stats_segments_multi(G, SEG, SEG_STATS[:n], WORKSPACE),
    "segments-compress-params": lambda n: B.tq_compress_segments_multi(G, SEG, SEG_PARAMS[:n], PAYLOADS, 3, 1, 0, 0),
    "segments-compress-payload": lambda n: B.tq_compress_segments_multi(G, SEG, SEG_PARAMS, PAYLOADS[:n], 3, 1, 0, 0),
    "segments-decode": lambda n: B.tq_decompress_aggregate_segments(PAYLOADS, SEG_PARAMS[:n], SEG, torch.zeros(D), 3),
}


@pytest.fixture
def reached(monkeypatch):
    """The library's functions replaced: what a call would have handed to the device."""
    counts = []

    class Calls:
        def __getattr__(self, name):
            return lambda *args: counts.append(name) or B.OK

    real = B.lib()
    sizes = {n: getattr(real, n) for n in ("tq_num_buckets", "tq_payload_bytes")}
    stub = Calls()
    for name, f in sizes.items():
        setattr(stub, name, f)
    monkeypatch.setattr(B, "lib", lambda: stub)
    monkeypatch.setattr(B, "_ptr_array", lambda tensors, what: tensors)
    monkeypatch.setattr(B, "_dev", lambda t, what: t.data_ptr())
    monkeypatch.setattr(B, "_stream", lambda: 0)
    return counts


@pytest.mark.parametrize("n", [0, 1, 2])
@pytest.mark.parametrize("call", CALLS)
def test_short_lists_are_refused(call, n, reached):
    with pytest.raises(ValueError, match="%d [a-z]+ buffers for a batch of 3 tensors" % n):
        CALLS[call](n)
    assert not reached


@pytest.mark.parametrize("call", CALLS)
def test_a_buffer_for_each_tensor_is_enough(call, reached):
    CALLS[call](3)
    assert len(reached) == 1


SHORT = torch.zeros(B.STATS_BYTES - 1, dtype=torch.uint8)
SMALL = {
    "stats": lambda: B.tq_stats(G[0], SHORT, WORKSPACE),
    "stats-buckets": lambda: B.tq_stats(G[0], SEG_STATS[0], WORKSPACE, 384),                 # three records
    "stats-static": lambda: B.tq_stats_static(G[0], SEG_STATS[0], 384),
    "stats-multi": lambda: B.tq_stats_multi(G, STATS[:2] + [SHORT], WORKSPACE),
    "stats-multi-buckets": lambda: B.tq_stats_multi(G, SEG_STATS, WORKSPACE, 384),
    "params-multi-stats": lambda: B.tq_params_multi(SEG_STATS[:2] + STATS[:1], SEG_PARAMS, 3, B.GRID_UNIFORM),
    "params-multi": lambda: B.tq_params_multi(SEG_STATS, SEG_PARAMS[:2] + PARAMS[:1], 3, B.GRID_UNIFORM),
    "segments-stats": lambda: B.tq_stats_segments(G[0], SEG, STATS[0], WORKSPACE),
    "segments-stats-multi": lambda: B.tq_stats_segments_multi(G, SEG, SEG_STATS[:2] + STATS[:1], WORKSPACE),
}


@pytest.mark.parametrize("call", SMALL)
def test_small_buffers_are_refused(call, reached):
    with pytest.raises(ValueError, match="buffer too small"):
        SMALL[call]()
    assert not reached


@pytest.mark.parametrize("odd", [torch.zeros(D - 1), torch.zeros(D, dtype=torch.bfloat16)])
@pytest.mark.parametrize("call", [lambda gs: B.tq_stats_multi(gs, STATS, WORKSPACE),
                                  lambda gs: B.tq_stats_segments_multi(gs, SEG, SEG_STATS, WORKSPACE)])
def test_batches_of_different_tensors_are_refused(call, odd, reached):
    with pytest.raises(ValueError, match="share shape and dtype"):
        call(G[:2] + [odd])
    assert not reached


@pytest.mark.parametrize("module", [True, False])
def test_roomy_buffers_and_longer_lists_are_taken(module, reached, monkeypatch):
    if not module:
        monkeypatch.setattr(B, "_tq_marshal", None)
    B.tq_stats(G[0], SEG_STATS[0], WORKSPACE)
    B.tq_stats(G[0], torch.zeros(3 * B.STATS_BYTES, dtype=torch.uint8), WORKSPACE, 384)
    B.tq_stats_multi(G[:2], SEG_STATS[:2] + [SHORT], WORKSPACE, 512)
    B.tq_stats_multi(G, [t.view(torch.float64) for t in STATS], WORKSPACE)                    # bytes count, not elements
    B.tq_params_multi(STATS, SEG_PARAMS, 3, B.GRID_UNIFORM)
    B.tq_stats_segments_multi(G, SEG, SEG_STATS, WORKSPACE)
    longer = G[:2] + [torch.zeros(D + 1)]
    B.tq_stats_multi(longer, STATS, WORKSPACE)
    B.tq_stats_segments_multi(longer, SEG, SEG_STATS, WORKSPACE)
    assert len(reached) == 8


def test_bucket_sizes_that_cannot_be_added_to_are_refused():
    """In a process of its own: a division by zero is a signal, not an exception."""
    code = """
import ctypes as C
from paper_2402_01798_amd import binding as B
L, p = B.lib(), C.c_void_p(0x1000)
for be in (2**64 - 128, 2**64 - 896):
    assert B.stats_workspace_bytes(1000, be) == 0
    assert L.tq_stats(p, 0, 1000, be, 0.0, p, p, 1 << 30, None) == B.EUNSUPPORTED
    assert L.tq_stats_static(p, 0, 1000, be, 0.0, p, None) == B.EUNSUPPORTED
    assert L.tq_compress(p, 0, 1000, be, p, 3, 0, 0, 0, 0, p, None) == B.EUNSUPPORTED
assert B.stats_workspace_bytes(1000, 2**64 - 1024) > 0
"""
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert run.returncode == 0, (run.returncode, run.stderr)


def test_records_are_the_librarys_buckets():
    for d in (0, 1, 127, 128, 129, 61_706, (1 << 40) - 1, 1 << 40):
        for bucket in (0, 1, 128, 16_384, 61_706, 1 << 20, 1 << 40, -1, -128):
            assert B._records(d, bucket) == B.num_buckets(d, bucket), (d, bucket)


@pytest.mark.parametrize("d,bucket,rows", [
    (1, 0, 1), (16_385, 0, 2), (32_767, 0, 2), (32_768, 0, 1025), (61_706, 0, 1025), (128 * 4096, 128, 4096), (20_000, 1 << 20, 64),
    (100_000, 16_384, 7), (100_000, 32_640, 8), (11_200_000, 16_512, 679), (124_000_000, 1 << 20, 1024 + 119)])
def test_workspace_sizes(d, bucket, rows):
    """Rows of 898 counts and 32 bytes of sums, in multiples of 256 bytes: sizes that callers rely on."""
    assert B.stats_workspace_bytes(d, bucket) == -(-rows * (B.NBINS * 4 + 32) // 256) * 256
