"""Updates, sums and simulated gradients large enough to go past the caches, whole wavefronts reading and writing 16-byte
pieces of the lanes' groups, against the plain aggregate (which the oracle checks elsewhere) and the same roundings in torch."""
import numpy as np
import pytest
import torch

from paper_2402_01798_amd import binding as B

pytestmark = pytest.mark.gpu
MIB = 1 << 20


def book(bits, nb, rng):
    s = (1 << bits) - 1
    rec = np.zeros(nb, dtype=B.PARAMS_DTYPE)
    level = np.sort(rng.uniform(-1, 1, (nb, s + 1)), axis=1).astype(np.float32)
    rec["alpha"], rec["bits"], rec["s"], rec["grid"] = 1.0, bits, s, B.GRID_NONUNIFORM
    rec["level"][:, :s + 1] = level
    rec["level"][:, 0], rec["level"][:, s] = -1.0, 1.0
    rec["inv_w"][:, :s] = 1.0 / np.maximum(np.diff(rec["level"][:, :s + 1].astype(np.float64), axis=1), 1e-6)
    return rec


def server(d, N, bits, bucket):
    """N payloads of random codes (any bytes are codes at every width) and their records."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d % 1000 + N)
    rng = np.random.default_rng(N)
    params = [B.params_from_numpy(book(bits, B.num_buckets(d, bucket), rng)) for _ in range(N)]
    payload = [torch.randint(0, 256, (B.payload_bytes(d, bits),), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(N)]
    g_bar = torch.empty(d, device="cuda")
    B.tq_decompress_aggregate(payload, params, g_bar, bits, bucket)
    theta, vel = (torch.randn(d, generator=gen, device="cuda") for _ in range(2))
    return payload, params, g_bar, theta, vel


SINGLE, DOUBLE = 96 * MIB // 4, 32 * MIB // 4                 # elements above which they go past the caches


@pytest.mark.parametrize("N,bits", [(1, 4), (3, 2), (8, 3), (16, 2), (12, 4), (20, 3), (33, 4)])
@pytest.mark.parametrize("extra,bucket", [(1, 0), (4_097, 1 << 20), (777, 9 * 4096 + 128), (2_048, 32_768)])
def test_updates(N, bits, extra, bucket):
    d, eta, mu, wd = DOUBLE + extra, 0.1, 0.9, 1e-3
    payload, params, g_bar, theta, vel = server(d, N, bits, bucket)
    f = lambda x: torch.tensor(x, dtype=torch.float32, device="cuda")
    v = f(mu) * vel + (g_bar + f(wd) * theta)
    want = theta - f(eta) * v
    B.tq_decompress_aggregate_update(payload, params, theta, bits, eta, mu, wd, vel, bucket)
    torch.cuda.synchronize()
    assert torch.equal(vel.view(torch.int32), v.view(torch.int32)) and torch.equal(theta.view(torch.int32), want.view(torch.int32))


# from 48 MiB of parameters on whatever the payloads are; at 32 MiB it is the payloads of 8 and more workers that decide
@pytest.mark.parametrize("N,bits", [(1, 4), (3, 2), (8, 3), (16, 2), (12, 4), (20, 3), (33, 4)])
@pytest.mark.parametrize("extra,bucket", [(1, 0), (4_097, 1 << 20), (777, 9 * 4096 + 128), (2_048, 32_768)])
def test_updates_of_few_payloads(N, bits, extra, bucket):
    test_updates(N, bits, 16 * MIB // 4 + extra, bucket)


@pytest.mark.parametrize("N,bits", [(2, 4), (8, 2), (17, 3)])
@pytest.mark.parametrize("extra,bucket", [(5, 0), (4_095, 65_536 + 128)])
def test_sums_and_plain_sgd(N, bits, extra, bucket):
    d, eta = SINGLE + extra, 0.25
    payload, params, g_bar, theta, _ = server(d, N, bits, bucket)
    total, want = theta + g_bar, theta - torch.tensor(eta, device="cuda") * g_bar
    out = theta.clone()
    B.tq_decompress_aggregate(payload, params, out, bits, bucket, None, True)
    B.tq_decompress_aggregate_update(payload, params, theta, bits, eta, 0.0, 0.0, None, bucket)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), total.view(torch.int32)) and torch.equal(theta.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("dtype,bits", [(torch.float32, 2), (torch.bfloat16, 3), (torch.float32, 4), (torch.bfloat16, 2)])
@pytest.mark.parametrize("extra,bucket", [(3, 0), (2_047, 5 * 2048 + 128), (513, 1 << 20)])
def test_simulated_gradients(dtype, bits, extra, bucket):
    """Q[T(g)] is what the server decodes from this worker alone; a sum adds it to what was there."""
    d = SINGLE + extra
    gen = torch.Generator(device="cuda")
    gen.manual_seed(bits)
    g = (torch.randn(d, generator=gen, device="cuda") * 0.5).to(dtype)
    g[:3] = torch.tensor([float("nan"), float("inf"), -float("inf")])
    params = B.params_from_numpy(book(bits, B.num_buckets(d, bucket), np.random.default_rng(bits)))
    payload = torch.empty(B.payload_bytes(d, bits), dtype=torch.uint8, device="cuda")
    B.tq_compress(g, params, payload, bits, 5, 1, 2, bucket, B.GRID_UNIFORM)
    want, out, old = torch.empty(d, device="cuda"), torch.full((d + 8,), 7.0, device="cuda"), torch.randn(d, generator=gen, device="cuda")
    B.tq_decompress_aggregate([payload], [params], want, bits, bucket)
    B.tq_quantize_dequantize(g, params, out[:d], bits, 5, 1, 2, bucket)
    total = old + want
    B.tq_quantize_dequantize(g, params, old, bits, 5, 1, 2, bucket, True)
    torch.cuda.synchronize()
    assert torch.equal(out[:d].view(torch.int32), want.view(torch.int32)) and (out[d:] == 7.0).all()
    assert torch.equal(old.view(torch.int32), total.view(torch.int32))


# payloads of up to 16 MiB, of 18 to 112 and above, one and two tiles a workgroup, whole and broken batches of eight workers
@pytest.mark.parametrize("N,d", [(9, 61_707), (33, 1_000_003), (20, 2_000_003), (64, 4_000_001), (12, 4_500_001), (16, 5_000_003),
                                 (16, 15_000_001), (25, 10_000_001), (17, 15_000_003), (40, 6_000_002)])
@pytest.mark.parametrize("bucket", [0, 300 * 2048 + 128])
def test_many_workers_at_four_bits(N, d, bucket):
    """The levels added in worker order and scaled, the same roundings in torch."""
    bits, nb = 4, B.num_buckets(d, bucket)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d % 1000 + N)
    recs = [book(bits, nb, np.random.default_rng(1000 * N + i)) for i in range(N)]
    payload = [torch.randint(0, 256, (B.payload_bytes(d, bits),), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(N)]
    out = torch.full((d + 8,), 7.0, device="cuda")
    B.tq_decompress_aggregate(payload, [B.params_from_numpy(r) for r in recs], out[:d], bits, bucket)
    first = torch.arange(d, device="cuda") // (bucket or d) * 16
    want = torch.zeros(d, device="cuda")
    for r, p in zip(recs, payload):
        codes = torch.stack([p & 15, p >> 4], 1).view(-1)[:d]
        want += torch.from_numpy(r["level"].reshape(-1).copy()).cuda()[first + codes]
    want *= torch.tensor(1.0 / N, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    assert torch.equal(out[:d].view(torch.int32), want.view(torch.int32)) and (out[d:] == 7.0).all()
