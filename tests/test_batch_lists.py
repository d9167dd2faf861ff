"""The batched calls refuse lists that are shorter than the batch: the library reads one address per tensor of it."""
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
SEG_PARAMS = [torch.zeros(2 * B.PARAMS_BYTES, dtype=torch.uint8) for _ in range(3)]

CALLS = {
    "stats": lambda n: B.tq_stats_multi(G, STATS[:n], WORKSPACE),
    "params": lambda n: B.tq_params_multi(STATS, PARAMS[:n], 3, B.GRID_UNIFORM),
    "compress-params": lambda n: B.tq_compress_multi(G, PARAMS[:n], PAYLOADS, 3, 1, 0, 0),
    "compress-payload": lambda n: B.tq_compress_multi(G, PARAMS, PAYLOADS[:n], 3, 1, 0, 0),
    "segments-stats": lambda n: B.tq_stats_segments_multi(G, SEG, STATS[:n], WORKSPACE),
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
