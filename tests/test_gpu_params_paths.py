"""tq_params where its ways of finding the threshold part: fixed points that the fp32 approach and the
Newton steps may take, those it must leave to the plain iteration, and thresholds at the ends of their range."""
import numpy as np
import pytest
import torch

from oracle import binding as O
from oracle import params as OP
from paper_2402_01798_amd import binding as B
from test_gpu_stats_params import assert_params_close

pytestmark = pytest.mark.gpu


def edge(i):
    return 2.0 ** ((i - 1) // 16 - 40) * (1 + ((i - 1) % 16) / 16)


def record(hist, absmax):
    r = np.zeros(1, dtype=B.STATS_DTYPE)
    r["hist"][0, :len(hist)] = hist
    r["absmax"] = absmax
    r["n"] = int(np.sum(hist))
    return r


def power_law(gamma, lo, width, n=2_000_000):
    x = np.arange(width)
    h = np.zeros(898, dtype=np.int64)
    h[lo:lo + width] = np.round(n * 2.0 ** (-(gamma - 1) * x / 16))
    return record(h, edge(lo + int(np.nonzero(h[lo:])[0].max())) * 1.01)


def records():
    out = []
    for gamma in (2.05, 2.5, 3.0, 4.0, 6.0, 9.0):            # slopes from nearly 0 to beyond what is certified
        for lo in (1, 300, 640):
            out.append(power_law(gamma, lo, 250))
    one = np.zeros(898, dtype=np.int64)
    one[500] = 1
    out.append(record(one, edge(500)))                        # one element
    two = np.zeros(898, dtype=np.int64)
    two[[1, 896]] = [1_000_000, 70_000]                       # first and last regular bin
    out.append(record(two, 65535.0))
    top = np.zeros(898, dtype=np.int64)
    top[880:898] = 1000                                       # into the last bin: the plain iteration
    out.append(record(top, 3.0e5))
    full = np.zeros(898, dtype=np.int64)
    full[300:400] = 40_000_000                                # counts whose sum is near 2^32
    full[400:440] = 5_000_000
    out.append(record(full, edge(440)))
    return np.concatenate(out)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("grid", [B.GRID_UNIFORM, B.GRID_NONUNIFORM, B.GRID_BISCALED])
def test_designed_histograms(bits, grid):
    st = records()
    dev = torch.from_numpy(st.view(np.uint8).reshape(-1).copy()).cuda()
    pr = torch.full((st.size * B.PARAMS_BYTES,), 0x77, dtype=torch.uint8, device="cuda")
    B.tq_params(dev, pr, bits, grid)
    torch.cuda.synchronize()
    got = B.params_to_numpy(pr)
    want = OP.tq_params(st.view(O.STATS_DTYPE), bits, grid)
    # An iteration that does not converge has no limit to compare, and whether one that ends up jumping
    # between two equally good splits (BiScaled, steep tails) does is decided by the last bits of Q_B: records
    # the oracle gives up on are left out (none of the uniform ones, at most 8 of 22 of the others).
    steady = (want["flags"] & 4) == 0
    assert steady.sum() >= (st.size if grid == B.GRID_UNIFORM else st.size - 8)
    assert (got["flags"][steady] == want["flags"][steady]).all()
    assert_params_close(got[steady], want[steady])


def design(st, bits, grid, override=0.0):
    dev = torch.from_numpy(st.view(np.uint8).reshape(-1).copy()).cuda()
    pr = torch.full((st.size * B.PARAMS_BYTES,), 0x77, dtype=torch.uint8, device="cuda")
    B.tq_params(dev, pr, bits, grid, override)
    torch.cuda.synchronize()
    return B.params_to_numpy(pr), OP.tq_params(st.view(O.STATS_DTYPE), bits, grid, override)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("grid", [B.GRID_UNIFORM, B.GRID_NONUNIFORM, B.GRID_BISCALED])
def test_thresholds_whose_reciprocal_is_subnormal(bits, grid):
    """From 2^126 on 1 / alpha is subnormal in binary32: ordinary values and one huge one, alpha = max|g| or
    given, on both sides of that line and at the top of the range."""
    values = np.abs(np.random.default_rng(3).standard_normal(1_000_000))
    h = np.bincount(np.clip((values.astype(np.float32).view(np.uint32) >> 19).astype(np.int64) - 1391, 0, 897), minlength=898)
    h[897] += 1
    tops = np.float32([2e37, 2.0 ** 126, 8.6e37, 1e38, 3.4028234663852886e38])
    got, want = design(np.concatenate([record(h, t) for t in tops]), bits, grid, -1.0)
    assert_params_close(got, want)
    for alpha in tops:
        got, want = design(record(h, 1e38), bits, grid, float(min(alpha, np.float32(3e38))))   # 3e38: the largest accepted
        assert_params_close(got, want)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("grid", [B.GRID_UNIFORM, B.GRID_NONUNIFORM, B.GRID_BISCALED])
def test_counts_that_add_up_beyond_32_bits(bits, grid):
    """A record summed over many tensors: every bin fits 32 bits, their sum does not."""
    h = np.zeros(898, dtype=np.int64)
    h[300:700] = np.round(4e9 * 2.0 ** (-2.0 * np.arange(400) / 16))
    assert h.sum() > 2 ** 35 and h.max() < 2 ** 32
    big = h.copy()
    big[300:320] = 4_000_000_000
    got, want = design(np.concatenate([record(h, edge(690)), record(big, edge(690))]), bits, grid)
    assert_params_close(got, want)
