"""Records that one workgroup reads whole: sizes around the ends of the rule (65536 elements a tensor, buckets of 32768)."""
import numpy as np
import pytest
import torch

from gpu_common import small_gradient
from oracle import binding as O
from paper_2402_01798_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,bucket,count,g_min", [
    (1, 0, 1, 0.0), (16_385, 0, 2, 1e-5), (32_767, 0, 3, 0.0), (32_768, 0, 3, 1e-5), (65_535, 0, 2, 1e-5), (65_536, 0, 64, 0.0),
    (65_537, 0, 2, 1e-5), (65_536, 65_536, 2, 1e-5), (65_000, 32_768, 3, 1e-5), (100_001, 32_640, 2, 1e-5), (70_001, 16_512, 5, 0.0)])
def test_statistics(d, bucket, count, g_min, dtype):
    gs, hosts = zip(*[small_gradient("cfg2", i % 5, d, dtype) for i in range(count)])
    nb = B.num_buckets(d, bucket)
    stats = [B.alloc_stats(d, bucket).fill_(0xA5) for _ in range(count)]
    ws = torch.empty(count * B.stats_workspace_bytes(d, bucket), dtype=torch.uint8, device="cuda")
    B.tq_stats_multi(list(gs), stats, ws, bucket, g_min)
    for i in range(count):
        got = B.stats_to_numpy(stats[i]).view(O.STATS_DTYPE)
        want = O.stats(hosts[i], bucket_elems=bucket, g_min=g_min)
        assert got.size == nb
        for f in ("hist", "n_nonfinite", "absmax", "n", "n_tail"):
            assert (got[f] == want[f]).all(), (i, f)
        # one fp32 logarithm per 8 elements and 2^-28 fixed point: 1e-6 of the sum, as everywhere
        np.testing.assert_allclose(got["sum_log_tail"], want["sum_log_tail"], rtol=1e-6, atol=4e-7)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("g_min", [0.0, 1e-5])
@pytest.mark.parametrize("d,bucket", [(100_003, 128), (100_003, 4_096), (50_001, 4_224), (8_192 * 3, 8_192), (50_005, 8_320),
                                      (16_384 * 3 - 1, 16_384), (70_000, 16_512), (100_000, 24_576), (8_192, 0), (8_193, 0), (16_384, 0)])
def test_small_buckets(d, bucket, g_min, dtype):
    """Both sides of the bucket sizes where the trips' length changes (bucket_trip), whole and ragged."""
    test_statistics(d, bucket, 2, g_min, dtype)
