"""Batches beyond the memory-side cache take loads and stores of their own: the same bytes as tensor by tensor.

The tensors of a batch may be the same one: 64 times a tensor of 8 MiB is a batch of 512 MiB."""
import pytest
import torch

from paper_2402_01798_amd import binding as B

pytestmark = pytest.mark.gpu

N, SEED, STEP = 64, 77, 5


def gradient(d, dtype):
    gen = torch.Generator().manual_seed(d)
    x = (1.0 - torch.rand(d, generator=gen)).pow_(-1.0 / 1.5).mul_(1e-5)
    x *= torch.randint(0, 2, (d,), generator=gen) * 2 - 1
    x[::100_003] = float("inf")
    x[5::70_001] = float("nan")
    x[9::65_537] = 1e9
    return x.to(dtype).cuda()


@pytest.mark.parametrize("bits,grid,bucket,g_min", [
    (2, B.GRID_UNIFORM, 0, 0.0), (3, B.GRID_NONUNIFORM, 65_536, 1e-5), (4, B.GRID_NONUNIFORM, 1 << 18, 0.0),
    (2, B.GRID_NONUNIFORM, 0, 3e-5), (3, B.GRID_UNIFORM, 33_024, 2e-5), (3, B.GRID_BISCALED, 16_384, 0.0)])
@pytest.mark.parametrize("d,dtype", [(2_100_003, torch.float32), (4_200_005, torch.bfloat16)])
def test_bucketed(d, dtype, bits, grid, bucket, g_min):
    g = gradient(d, dtype)
    stats, params = B.alloc_stats(d, bucket), B.alloc_params(d, bucket)
    B.tq_stats(g, stats, B.alloc_stats_workspace(d, bucket), bucket, g_min)
    B.tq_params(stats, params, bits, grid)
    ws = torch.empty(N * B.stats_workspace_bytes(d, bucket), dtype=torch.uint8, device="cuda")
    many = [B.alloc_stats(d, bucket).fill_(0x11) for _ in range(N)]
    payloads = [B.alloc_payload(d, bits).fill_(0x33) for _ in range(N)]
    B.tq_stats_multi([g] * N, many, ws, bucket, g_min)
    B.tq_compress_multi([g] * N, [params] * N, payloads, bits, SEED, 0, STEP, bucket, grid)
    one = B.alloc_payload(d, bits)
    for i in range(N):
        assert torch.equal(many[i], stats), i
        B.tq_compress(g, params, one.fill_(0x44), bits, SEED, i, STEP, bucket, grid)
        assert torch.equal(payloads[i], one), i


@pytest.mark.parametrize("bits,bucket", [(4, 0), (4, 1 << 20), (4, 2_048), (3, 0)])
def test_bf16_beyond_two_gib(bits, bucket):
    """64 times 34 MB: the uniform codebook at b = 4 reads through the caches again."""
    d = 17_000_003
    g = gradient(d, torch.bfloat16)
    stats, params = B.alloc_stats(d, bucket), B.alloc_params(d, bucket)
    B.tq_stats(g, stats, B.alloc_stats_workspace(d, bucket), bucket)
    B.tq_params(stats, params, bits, B.GRID_UNIFORM)
    payloads = [B.alloc_payload(d, bits).fill_(0x33) for _ in range(N)]
    B.tq_compress_multi([g] * N, [params] * N, payloads, bits, SEED, 0, STEP, bucket)
    one = B.alloc_payload(d, bits)
    for i in range(N):
        B.tq_compress(g, params, one.fill_(0x44), bits, SEED, i, STEP, bucket)
        assert torch.equal(payloads[i], one), i


@pytest.mark.parametrize("bits,grid,g_min", [(2, B.GRID_NONUNIFORM, 0.0), (3, B.GRID_NONUNIFORM, 1e-5), (4, B.GRID_UNIFORM, 0.0)])
@pytest.mark.parametrize("d,dtype", [(2_100_003, torch.float32), (4_200_005, torch.bfloat16)])
def test_segments(d, dtype, bits, grid, g_min):
    seg = B.Segments([0, 128, 1_152, 40_960, 300_032, 1_700_096, d])
    g = gradient(d, dtype)
    stats = torch.empty(seg.nseg * B.STATS_BYTES, dtype=torch.uint8, device="cuda")
    params = torch.empty(seg.nseg * B.PARAMS_BYTES, dtype=torch.uint8, device="cuda")
    ws = torch.empty(N * B.stats_segments_workspace_bytes(d, seg.nseg), dtype=torch.uint8, device="cuda")
    B.tq_stats_segments(g, seg, stats, ws, g_min)
    B.tq_params(stats, params, bits, grid)
    many = [torch.empty_like(stats).fill_(0x11) for _ in range(N)]
    payloads = [B.alloc_payload(d, bits).fill_(0x33) for _ in range(N)]
    B.tq_stats_segments_multi([g] * N, seg, many, ws, g_min)
    B.tq_compress_segments_multi([g] * N, seg, [params] * N, payloads, bits, SEED, 0, STEP)
    one = B.alloc_payload(d, bits)
    for i in range(N):
        assert torch.equal(many[i], stats), i
        B.tq_compress_segments(g, seg, params, one.fill_(0x44), bits, SEED, i, STEP)
        assert torch.equal(payloads[i], one), i
