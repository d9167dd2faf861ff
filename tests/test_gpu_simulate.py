"""tq_quantize_dequantize against the oracle (client step of Alg. 1, then the server's look-up
of the level) and against the library's own compress -> decode round trip: bit for bit."""
import numpy as np
import pytest
import torch

from oracle import binding as O
from paper_2402_01798_amd import binding as B
from gpu_common import oracle_params, small_gradient

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("grid", [B.GRID_UNIFORM, B.GRID_NONUNIFORM, B.GRID_BISCALED])
@pytest.mark.parametrize("d,bucket", [(1, 0), (13, 0), (2048, 0), (61_706, 0), (3 * 2048 + 5, 2048 + 128), (40_001, 4096)])
def test_values_match_oracle_and_round_trip(bits, grid, d, bucket):
    g_dev, g_np = small_gradient("cfg1", 2, d)
    P = oracle_params(g_np, bits, grid, bucket_elems=bucket)
    params_dev = B.params_from_numpy(P)
    out = torch.full((d,), 7.0, dtype=torch.float32, device="cuda")
    B.tq_quantize_dequantize(g_dev, params_dev, out, bits, 0xABCDEF0123, 5, 9, bucket)
    want = O.quantize_dequantize(g_np, P, 0xABCDEF0123, 5, 9, bucket_elems=bucket)
    assert (out.cpu().numpy() == want).all()
    # the library's own round trip gives the same values
    pay = B.alloc_payload(d, bits)
    B.tq_compress(g_dev, params_dev, pay, bits, 0xABCDEF0123, 5, 9, bucket)
    rt = torch.empty(d, dtype=torch.float32, device="cuda")
    B.tq_decompress_aggregate([pay], [params_dev], rt, bits, bucket)
    assert torch.equal(rt, out)
    # accumulate adds a second worker's values in binary32
    B.tq_quantize_dequantize(g_dev, params_dev, out, bits, 0xABCDEF0123, 6, 9, bucket, accumulate=True)
    want2 = want + O.quantize_dequantize(g_np, P, 0xABCDEF0123, 6, 9, bucket_elems=bucket)
    assert (out.cpu().numpy() == want2).all()


def test_bf16_and_special_values():
    d = 5000
    g = torch.randn(d).mul_(1e-3).to(torch.bfloat16)
    g[[0, 7, 4999]] = torch.tensor([float("nan"), float("inf"), float("-inf")], dtype=torch.bfloat16)
    g_np = g.view(torch.uint16).numpy()
    P = oracle_params(g_np, 3, B.GRID_NONUNIFORM)
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    B.tq_quantize_dequantize(g.cuda(), B.params_from_numpy(P), out, 3, 1, 0, 0)
    want = O.quantize_dequantize(g_np, P, 1, 0, 0)
    got = out.cpu().numpy()
    assert (got == want).all()
    a = float(P["alpha"][0])
    assert got[7] == np.float32(a) and got[4999] == np.float32(-a)          # +-Inf -> +-alpha


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,bucket", [(2047, 0), (2048, 0), (4096, 0), (4097, 0), (8192 + 2048 + 9, 0), (5 * 4096, 4096),
                                      (33_554_432 + 4096 + 11, 1 << 20), (41_943_040 + 4096 + 11, 1 << 20),
                                      (41_943_040 + 4096 + 11, 4096)])
def test_ranges_of_whole_and_cut_tiles_and_large_outputs(dtype, d, bucket):
    """Workgroup ranges that are whole, cut inside a tile or between two tiles, and outputs just above
    128 and 160 MiB (the latter stored past the caches): the values of the compress -> decode round trip, nothing behind them."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    g = torch.randn(d, generator=gen, device="cuda").to(dtype)
    stats, params = B.alloc_stats(d, bucket), B.alloc_params(d, bucket)
    B.tq_stats(g, stats, B.alloc_stats_workspace(d, bucket), bucket)
    for grid in (B.GRID_UNIFORM, B.GRID_NONUNIFORM):
        B.tq_params(stats, params, 3, grid)
        out = torch.full((d + 64,), 7.0, device="cuda")
        B.tq_quantize_dequantize(g, params, out[:d], 3, 21, 4, 2, bucket)
        pay, rt = B.alloc_payload(d, 3), torch.empty(d, device="cuda")
        B.tq_compress(g, params, pay, 3, 21, 4, 2, bucket, grid)
        B.tq_decompress_aggregate([pay], [params], rt, 3, bucket)
        assert torch.equal(out[:d], rt) and bool((out[d:] == 7.0).all())
        B.tq_quantize_dequantize(g, params, out[:d], 3, 21, 4, 2, bucket, accumulate=True)
        assert torch.equal(out[:d], rt + rt) and bool((out[d:] == 7.0).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("kind", ["uniform", "mirrored", "lopsided", "empty ends"])
@pytest.mark.parametrize("d,bucket", [(3 * 2048 + 517, 0), (9 * 1024 + 5, 1024), (12 * 2048 + 300, 2048), (4 * 3072 + 9, 3072),
                                      (2 * 8192 + 2048 + 7, 8192)])
def test_any_codebook_in_short_buckets(d, bucket, kind, bits, dtype):
    """Codebooks that mirror, do not mirror and have empty outer cells, buckets shorter than a workgroup's range and
    wavefronts that are whole, cut and empty, with and without accumulation: the oracle's values, nothing behind them."""
    s, nb = (1 << bits) - 1, B.num_buckets(d, bucket)
    t = 2.0 * np.arange(s + 1) / s - 1.0
    P = np.zeros(nb, dtype=O.PARAMS_DTYPE)
    for k in range(nb):
        alpha = np.float32(0.5 + 0.25 * k)
        lv = (alpha * (t if kind == "uniform" else np.sign(t) * np.abs(t) ** 1.7)).astype(np.float32)
        if kind == "lopsided":
            lv[1:s] += np.float32(0.07) * alpha / s
        if kind == "empty ends":
            lv[1], lv[s - 1] = -alpha, alpha
        lv[0], lv[s] = -alpha, alpha
        width = np.diff(lv.astype(np.float64))
        P["level"][k, : s + 1] = lv
        P["inv_w"][k, :s] = np.where(width > 0, 1.0 / np.where(width > 0, width, 1.0), 0.0)
        P["alpha"][k], P["bits"][k], P["s"][k] = alpha, bits, s
        P["grid"][k] = O.GRID_UNIFORM if kind == "uniform" else O.GRID_NONUNIFORM
        if kind == "uniform":
            P["inv_w"][k] = np.float32(s / (2.0 * float(alpha)))
    g = (torch.randn(d, generator=torch.Generator().manual_seed(bits)) * 1.5).to(dtype)
    g_np = g.view(torch.int16).numpy().view("uint16") if dtype == torch.bfloat16 else g.numpy()
    out = torch.full((d + 64,), 7.0, device="cuda")
    params = B.params_from_numpy(P)
    B.tq_quantize_dequantize(g.cuda(), params, out[:d], bits, 21, 4, 2, bucket)
    want = O.quantize_dequantize(g_np, P, 21, 4, 2, bucket_elems=bucket)
    assert (out[:d].cpu().numpy() == want).all()
    B.tq_quantize_dequantize(g.cuda(), params, out[:d], bits, 21, 5, 2, bucket, accumulate=True)
    want = want + O.quantize_dequantize(g_np, P, 21, 5, 2, bucket_elems=bucket)
    assert (out[:d].cpu().numpy() == want).all() and bool((out[d:] == 7.0).all())
