"""Averages laid out through LDS and in registers: the bucketed call takes one or the other by bits, workers and size, the
segment call always the second, and one segment is one bucket: the same bytes on both sides of every line."""
import numpy as np
import pytest
import torch

from paper_2402_01798_amd import binding as B

pytestmark = pytest.mark.gpu

MIB = (1 << 20) // 4                                           # elements


@pytest.mark.parametrize("N,bits,d", [
    (16, 2, 4_099), (13, 2, 1_000_003), (16, 2, 64 * MIB + 4_096), (9, 2, 161 * MIB + 13),
    (8, 2, 64 * MIB), (8, 2, 64 * MIB + 1), (5, 2, 100 * MIB + 4_095), (7, 2, 160 * MIB + 1),
    (8, 4, 160 * MIB), (5, 4, 160 * MIB + 4_097),
    (1, 4, 1536 * MIB + 3), (2, 4, 1536 * MIB + 2_049), (4, 4, 1536 * MIB + 128),
    (1, 3, 2560 * MIB + 9), (2, 2, 2560 * MIB + 1),
    (1, 2, 4352 * MIB + 1), (1, 3, 2816 * MIB + 9), (1, 4, 2048 * MIB + 3), (2, 4, 1024 * MIB + 2_049), (2, 2, 2048 * MIB + 1)])
@pytest.mark.parametrize("weighted", [False, True])
def test_same_bytes(N, bits, d, weighted):
    gen = torch.Generator(device="cuda").manual_seed(d)
    rng = np.random.default_rng(N * 8 + bits)
    payloads = [torch.randint(0, 256, (B.payload_bytes(d, bits),), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(N)]
    params = []
    for _ in range(N):
        rec = np.zeros(1, dtype=B.PARAMS_DTYPE)
        rec["bits"], rec["s"], rec["grid"] = bits, (1 << bits) - 1, B.GRID_NONUNIFORM
        rec["level"][0, :1 << bits] = np.sort(rng.standard_normal(1 << bits).astype(np.float32))
        params.append(B.params_from_numpy(rec))
    weights = (rng.random(N) + 0.5).tolist() if weighted else None
    buckets = torch.full((d + 64,), 7.0, device="cuda")
    B.tq_decompress_aggregate(payloads, params, buckets[:d], bits, 0, weights)
    segments = torch.full((d + 64,), 7.0, device="cuda")
    B.tq_decompress_aggregate_segments(payloads, params, B.Segments([0, d]), segments[:d], bits, weights)
    assert torch.equal(buckets, segments)                      # and nothing past the end on either side
    assert torch.unique(buckets[:4096]).numel() >= 1 << bits     # one worker's average takes its 2^b levels, several workers' more
