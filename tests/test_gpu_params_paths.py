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


def two_modes(rng):
    """Counts of a histogram with two separated modes, and the edge above them."""
    w, gap = int(rng.integers(10, 60)), int(rng.integers(10, 80))
    h = np.zeros(898, dtype=np.int64)
    h[560:560 + w] = rng.uniform(0.5, 1.0, w) * 10 ** rng.uniform(3, 6)
    h[560 + w + gap:600 + w + gap] = rng.uniform(0.5, 1.0, 40) * 10 ** rng.uniform(2, 6)
    return h, edge(600 + w + gap)


def splits_change_beside_the_fixed_point(count):
    """BiScaled records (b = 3) whose fixed point lies within 1e-6 of a threshold at which the best edge changes
    and the slope of ln Q_B with it, the slopes of the iterated map on both sides within +-0.7."""
    rng, out, targets = np.random.default_rng(8), [], []
    while len(out) < count:
        h, top = two_modes(rng)
        dens = OP.Density(h, top)
        below = np.concatenate([[0.0], np.cumsum(dens.hist)]) / dens.n

        def v(a):
            lo = dens.lo[dens.lo < a]
            k, inside = lo / a, below[:lo.size]
            mass = below[lo.size - 1] + dens.hist[lo.size - 1] / dens.n * (a - lo[-1]) / dens.w[lo.size - 1]
            return np.cbrt((mass - inside) * (1 - k) ** 2) + np.cbrt(inside * k * k)

        def slope(j, a):
            return 3e6 * np.log(v(a * (1 + 5e-7))[j] / v(a * (1 - 5e-7))[j])

        grid = np.exp(np.linspace(np.log(edge(575)), np.log(top * 0.99), 400))
        best = [int(np.argmin(v(a))) for a in grid]
        for i in np.nonzero(np.diff(best))[0]:
            l, r = grid[i], grid[i + 1]
            for _ in range(50):
                m = 0.5 * (l + r)
                l, r = (m, r) if int(np.argmin(v(m))) == best[i] else (l, m)
            on_edge = np.abs(dens.lo / l - 1).min() < 1e-4
            e0, e1 = slope(best[i], l * (1 - 1e-6)), slope(int(np.argmin(v(r))), r * (1 + 1e-6))
            if on_edge or abs(e0 - e1) < 0.5 or max(abs(e0), abs(e1)) > 20:
                continue
            ex = min(0.7 / max(abs(e0), abs(e1)), 0.9)
            target = l * (1 + rng.uniform(-1e-6, 1e-6))
            # ln(target / g) = ex (ln C - ln Q), C = 2 rho s^2 / (gamma - 2): by g, then by the log-sum through gamma
            gamma, n_tail = 1 + 1 / ex, dens.n // 10
            ln_q = 3 * np.log(v(target).min())
            rho = n_tail / (2 * dens.n)
            g = np.float32(target * np.exp(-ex * (np.log(2 * rho * 49 / (gamma - 2)) - ln_q)))
            if not 2.0 ** -40 <= g < 0.8 * target:
                continue
            f = lambda gm: np.log(target / float(g)) * (gm - 1) - (np.log(2 * rho * 49 / (gm - 2)) - ln_q)
            lo_g, hi_g = max(2.03, gamma * 0.99), gamma * 1.01
            if f(lo_g) * f(hi_g) > 0:
                continue
            for _ in range(80):
                m = 0.5 * (lo_g + hi_g)
                lo_g, hi_g = (m, hi_g) if f(m) * f(lo_g) > 0 else (lo_g, m)
            st = record(h, top)
            st["g_min"], st["n_tail"], st["sum_log_tail"] = g, int(n_tail), int(n_tail) / (lo_g - 1)
            a, log_c = float(g) * 1.01, np.log(2 * rho * 49 / (lo_g - 2))
            for _ in range(100):                              # the definition's iteration
                before = a
                a = float(np.clip(float(g) * np.exp((log_c - 3 * np.log(max(v(a).min(), 1e-99))) / (lo_g - 1)), g * (1 + 2.0 ** -10), top))
            if abs(a / target - 1) > 1e-10 or abs(a / before - 1) > 1e-12:
                continue                                      # it goes elsewhere, or stays undecided
            out.append(st)
            targets.append(target)
            break
    return np.concatenate(out), np.float32(targets)


def test_the_best_split_changes_beside_the_fixed_point():
    """Where the best edge of the BiScaled search changes, ln Q_B has a kink, and a step taken with the slope of
    one side does not land on the other.  The threshold is fp64's, rounded: the fixed
    point's binary32, or its neighbour where fp64 rounds the other way."""
    st, alpha = splits_change_beside_the_fixed_point(48)
    dev = torch.from_numpy(st.view(np.uint8).reshape(-1).copy()).cuda()
    pr = torch.full((st.size * B.PARAMS_BYTES,), 0x77, dtype=torch.uint8, device="cuda")
    B.tq_params(dev, pr, 3, B.GRID_BISCALED)
    torch.cuda.synchronize()
    got = B.params_to_numpy(pr)
    assert (got["flags"] == 0).all()
    off = np.abs(got["alpha"].astype(np.float64) - alpha) / np.spacing(alpha)
    assert off.max() <= 1.0, off


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("low", [1, 200, 561, 640, 700])
def test_best_splits_in_every_window_below_the_threshold(low, bits):
    """The search looks at 64 edges at a time from the threshold's bin downwards: most of the mass 40, 104, 179, 540 and 739
    bins below it, thresholds at a bin's lower edge, inside it, and where rounding to binary32 moves them across an edge."""
    h = np.zeros(898, dtype=np.int64)
    h[low:low + 20] = 3_000_000
    h[700:760] = 400
    h[0] = 5
    st = np.concatenate([record(h, edge(760))] * 5)
    for alpha in (edge(759), edge(741) * 1.01, float(np.nextafter(np.float32(edge(750)), np.float32(0)))):
        got, want = design(st, bits, B.GRID_BISCALED, alpha)
        assert_params_close(got, want)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("grid", [B.GRID_NONUNIFORM, B.GRID_BISCALED])
def test_records_whose_iteration_does_not_settle(bits, grid):
    """The records left out above: the tail estimates are the oracle's, alpha lies in its range and is a fixed point
    unless the flag says that none was reached, and the codebook is the one the oracle designs for that alpha."""
    st = records()
    got, want = design(st, bits, grid)
    s = (1 << bits) - 1
    for i in np.nonzero(want["flags"] & 4)[0]:
        g, w = got[i], want[i]
        for f in ("gamma_hat", "rho_hat", "g_min"):
            assert np.isclose(g[f], w[f], rtol=1e-6, atol=0), (i, f)
        alpha, g_min, top = float(g["alpha"]), float(w["g_min"]), float(st["absmax"][i])
        assert g_min < alpha <= top and (g["flags"] & ~np.uint32(4 | 1 | 32)) == (w["flags"] & ~np.uint32(4 | 1 | 32))
        dens = OP.Density(st["hist"][i], top)
        if not g["flags"] & 4:
            gamma = max(float(w["gamma_hat"]), OP.GAMMA_FLOOR)
            q = dens.Q_N(alpha) if grid == B.GRID_NONUNIFORM else dens.best_k(alpha)[1]
            f_alpha = g_min * (2 * float(w["rho_hat"]) * s * s / (gamma - 2) / q) ** (1 / (gamma - 1))
            # alpha, gamma and rho are rounded to binary32, which moves the map by less than 1e-5 here
            assert abs(min(max(f_alpha, g_min * (1 + 2.0 ** -10)), top) / alpha - 1) < 1e-5, i
        own = OP.tq_params(st[i:i + 1].view(O.STATS_DTYPE), bits, grid, alpha)[0]
        assert np.allclose(g["level"], own["level"], rtol=1e-6, atol=0), i
        assert np.allclose(g["inv_w"], own["inv_w"], rtol=2e-6, atol=0), i


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("grid", [B.GRID_UNIFORM, B.GRID_NONUNIFORM, B.GRID_BISCALED])
def test_groups_of_empty_bins(bits, grid):
    """Groups of 64 bins that count nothing are left out: one group alone, its first or its last bin alone, every other group,
    all but one group, the tail's bin at a group's edges."""
    rng = np.random.default_rng(bits)
    out = []
    for group in range(14):
        alone = np.zeros(898, dtype=np.int64)
        alone[64 * group + (group == 0):64 * group + 64] = rng.integers(1, 1000, 64 - (group == 0))
        first, last, without = np.zeros(898, dtype=np.int64), np.zeros(898, dtype=np.int64), np.zeros(898, dtype=np.int64)
        first[max(64 * group, 1)] = 90
        first[max(64 * group, 1) + 20] = 10                # 90 of 100: the tail starts at the group's first bin
        last[64 * group + 63] = 95
        last[min(64 * group + 70, 896)] += 5
        without[1:897] = np.round(1e6 * 2.0 ** (-np.arange(896) / 16))
        without[64 * group:64 * group + 64] = 0
        out += [alone, first, last, without]
    for odd in (0, 1):
        every_other = np.zeros(898, dtype=np.int64)
        for group in range(odd, 14, 2):
            every_other[64 * group + 1:64 * group + 64] = 5000 >> group // 2
        out.append(every_other)
    st = np.concatenate([record(h, edge(int(np.nonzero(h)[0].max())) * 1.01) for h in out])
    got, want = design(st, bits, grid)
    steady = (want["flags"] & 4) == 0
    assert steady.sum() >= st.size // 2 and (got["flags"][steady] == want["flags"][steady]).all()
    assert_params_close(got[steady], want[steady])


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_the_same_iteration_inside_and_outside_the_regular_bins(bits):
    """Thresholds that stay below 65536 take their bin from their bits, others the general form.  Scaled by 4096 -- twelve octaves, where
    w^(2/3) scales by 256 -- the plain iteration does the same arithmetic, so its result scales to the bit."""
    low, high = [], []
    # (2.2, 400), (2.5, 400) and (2.9, 300) do not settle in 100 steps at b = 2, 3 and 4
    for gamma, width in [(g, w) for g in (2.05, 2.2, 2.5, 3.0, 4.0, 6.0, 9.0) for w in (60, 150, 400)] + [(2.9, 300)]:
        h = np.zeros(898, dtype=np.int64)
        h[897 - width:897] = np.round(2_000_000 * 2.0 ** (-(gamma - 1) * np.arange(width) / 16)) + 1
        high.append(record(h, 65536.0))
        low.append(record(np.concatenate([h[192:897], np.zeros(193, dtype=np.int64)]), 16.0))
    got, _ = design(np.concatenate(low), bits, B.GRID_NONUNIFORM)
    up, _ = design(np.concatenate(high), bits, B.GRID_NONUNIFORM)
    slow = (got["flags"] & 4) != 0                            # never handed to the Newton steps
    assert slow.any() and (got["flags"] == up["flags"]).all()
    assert (got["alpha"][slow] * np.float32(4096) == up["alpha"][slow]).all() and (got["level"][slow] * np.float32(4096) == up["level"][slow]).all()
    assert np.allclose(got["alpha"] * np.float32(4096), up["alpha"], rtol=1e-6, atol=0)


def levels_at_gaps(s, count):
    """Records of two blocks of equal bins with empty bins between them, the largest magnitude at the lower edge of its bin:
    j / s of the integral of density^(1/3) is the first block's, with j odd as the levels have it, so a level lies at the gap."""
    rng, out = np.random.default_rng(s), []
    while len(out) < count:
        j, octave, higher = 2 * int(rng.integers(1, (s + 1) // 2)) - 1, int(rng.integers(0, 40)), int(rng.integers(1, 4))
        n1, n2 = int(rng.integers(1, 16)), int(rng.integers(1, 17))
        lo1 = 1 + 16 * octave + int(rng.integers(0, 17 - n1))
        lo2 = 1 + 16 * (octave + 3 * higher) + int(rng.integers(0, 17 - n2))
        # three octaves up a bin is 8 times as wide, its share 4 times: c1^(1/3) n1 (s - j) = j 4^higher c2^(1/3) n2
        a, b = j * 4 ** higher * n2, n1 * (s - j)
        a, b = a // np.gcd(a, b), b // np.gcd(a, b)
        if max(a, b) > 1500:
            continue
        h = np.zeros(898, dtype=np.int64)
        h[lo1:lo1 + n1], h[lo2:lo2 + n2], h[lo2 + n2] = a ** 3, b ** 3, 1
        out.append(record(h, edge(lo2 + n2)))
    h = np.zeros(898, dtype=np.int64)
    h[321:331], h[380:385], h[385] = 4, 4, 1
    return np.concatenate(out + [record(h, edge(385))])


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_levels_where_the_integral_stands_still(bits):
    """The sums over the bins differ by an ulp from one empty bin to the next, so a level at a gap can be found at
    any point of it.  Wherever it is, the integral there is j / s of the whole.  A level's rounding
    to binary32 moves it by at most 2^-24 of its magnitude, 32 bin widths: by 2^-19 of one bin's share."""
    s = (1 << bits) - 1
    st = levels_at_gaps(s, 1500)
    dev = torch.from_numpy(st.view(np.uint8).reshape(-1).copy()).cuda()
    pr = torch.full((st.size * B.PARAMS_BYTES,), 0x77, dtype=torch.uint8, device="cuda")
    B.tq_params(dev, pr, bits, B.GRID_NONUNIFORM, -1.0)       # alpha = max|g|
    torch.cuda.synchronize()
    got = B.params_to_numpy(pr)
    want = np.arange(1, s + 1, 2) / s
    off = []
    for r, q in zip(st, got):
        dens = OP.Density(r["hist"], r["absmax"])
        assert (q["level"][:s + 1] == -q["level"][s::-1]).all()
        up = [dens.half_int_p13(float(x)) if np.isfinite(x) else np.inf for x in q["level"][(s + 1) // 2:s + 1]]
        off.append(np.abs(np.array(up) / dens.half_int_p13(float(q["alpha"])) - want).max())
    off = np.array(off)
    assert (off <= 2.0 ** -19).all(), (np.nonzero(off > 2.0 ** -19)[0], off.max())
