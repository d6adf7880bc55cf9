"""The DP's lower bound on the candidates (Alg. 3, App. D), checked on the CPU against the
oracle's full scan.

The library's DP looks, for row r of level j, only at the candidates l from the smallest l
that came within a rounding slack of the row's minimum one level below (the quadrangle
inequality of the interval costs keeps every smaller l worse from then on). A level's last
row hands its bound to the rows that later levels add, so its slack is that of the total
count. This test restates that rule in numpy, float64 operations in the oracle's order, and
checks codebook, cost and interval starts bit for bit, on histograms with many exact ties,
plateaus beside spikes of 1e9, empty stretches, and a few counts a bin below bins of 2e10 to
1e11 (where a slack of the handing row's own count drops candidates that win)."""
import numpy as np
import pytest

import oracle


def pruned_dp(hist, k):
    nbins = hist.size
    at = np.nonzero(hist)[0]
    c = hist[at].astype(np.float64)
    m = -1.0 + (at + 0.5) * (2.0 / nbins)
    b = at.size
    z0, z1, z2 = (np.concatenate([[0.0], np.cumsum(v)]) for v in (c, c * m, c * m * m))
    assert b >= k and z0[-1] * nbins < 2.0 ** 50
    d = np.full(b + 1, np.inf)
    d[1:] = 0.0 + (z2[1:] - 2.0 * -1.0 * z1[1:] + z0[1:])
    split = np.zeros((k + 1, b + 1), dtype=np.int64)
    split[1] = 1
    low = np.full(b + 1, 2)
    seen = 0
    for j in range(2, k + 1):
        rmax = b - k + j
        new, nlow = np.full(b + 1, np.inf), np.zeros(b + 1, dtype=np.int64)
        for r in range(b if j == k else j, rmax + 1):
            lo = j if j in (2, k) else max(j, low[r] if r < rmax else low[r - 1])
            l = np.arange(lo, r + 1)
            s0, s1, s2 = z0[r] - z0[l - 1], z1[r] - z1[l - 1], z2[r] - z2[l - 1]
            w = s2 - 2.0 * s1 + s0 if j == k else s2 - s1 * s1 / s0
            cand = d[l - 1] + w
            i = int(np.argmin(cand))
            new[r], split[j, r] = cand[i], lo + i
            slack = 2.0 ** -53 * (256.0 * (z0[b] if r == rmax else z0[r]) + 32.0 * k * cand[i])
            nlow[r] = lo + int(np.argmax(cand <= cand[i] + slack))
            seen += l.size
        d, low = new, nlow
    bounds, cb, r = np.zeros(k, dtype=np.int64), np.ones(k), b
    for j in range(k, 0, -1):
        l = int(split[j, r])
        bounds[j - 1] = l
        if j == 1:
            cb[0] = -1.0
        elif j < k:
            cb[j - 1] = (z1[r] - z1[l - 1]) / (z0[r] - z0[l - 1])
        r = l - 1
    return cb, d[b], bounds, seen


def histogram(kind, nbins, seed):
    rng = np.random.default_rng(seed)
    h = np.ones(nbins, dtype=np.uint64)
    if kind == "bell":
        x = np.linspace(-1, 1, nbins)
        h += rng.poisson(2e4 * np.exp(-8 * x * x)).astype(np.uint64)
    elif kind == "flat":
        h *= np.uint64(rng.integers(1, 10 ** 6))
    elif kind == "spikes":
        h[rng.integers(0, nbins, 12)] = 10 ** 9
    elif kind == "centre":
        h += rng.integers(0, 3, nbins).astype(np.uint64)
        h[nbins // 2 - 1:nbins // 2 + 1] = 4 * 10 ** 9
    elif kind == "two_scales":
        h[nbins // 2:] = 10 ** 8
    elif kind == "comb":
        h[::16] = 10 ** 6
    elif kind == "gaps":
        h = np.where(rng.random(nbins) < 0.4, rng.integers(1, 1000, nbins), 0).astype(np.uint64)
        h[0] = h[-1] = 5
    return h


def heavy_top(nbins, k, fill, seed, big):
    """1 to 3 counts in each of the last `fill` bins, but `big` in two of the last k."""
    rng = np.random.default_rng(seed)
    h = np.zeros(nbins, dtype=np.uint64)
    h[nbins - fill:] = rng.integers(1, 4, fill).astype(np.uint64)
    h[nbins - 2 - rng.integers(0, min(k, fill) - 4, 2)] = big
    return h


# (nbins, k, fill, seed, big)
HEAVY = [(4096, 64, 80, 14, 5 * 10 ** 10), (4096, 64, 80, 11, 2 * 10 ** 10),
         (4096, 256, 300, 3, 10 ** 11)]
KINDS = ["bell", "flat", "spikes", "centre", "two_scales", "comb", "gaps"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nbins,k", [(256, 16), (320, 64), (193, 5)])
def test_pruned_scan_equals_the_full_scan(kind, nbins, k):
    h = histogram(kind, nbins, seed=nbins + k)
    cb, cost, bounds, seen = pruned_dp(h, k)
    cb_ref, cost_ref, bounds_ref, st = oracle.dp_codebook(h, k)
    assert st == 0
    np.testing.assert_array_equal(cb, cb_ref)
    assert cost == cost_ref
    np.testing.assert_array_equal(bounds, bounds_ref)
    b = int(np.count_nonzero(h))
    assert seen < sum(r - j + 1 for j in range(2, k) for r in range(j, b - k + j + 1)) + b


@pytest.mark.parametrize("nbins,k,fill,seed,big", HEAVY)
def test_bounds_handed_past_heavy_bins(nbins, k, fill, seed, big):
    h = heavy_top(nbins, k, fill, seed, big)
    cb, cost, bounds, _ = pruned_dp(h, k)
    cb_ref, cost_ref, bounds_ref, st = oracle.dp_codebook(h, k)
    assert st == 0
    np.testing.assert_array_equal(cb, cb_ref)
    assert cost == cost_ref
    np.testing.assert_array_equal(bounds, bounds_ref)


def test_prefix_sums_are_sequential():
    """np.cumsum adds in order, as the definition's running sums do."""
    x = np.random.default_rng(0).standard_normal(5000)
    acc, out = 0.0, []
    for v in x:
        acc += v
        out.append(acc)
    np.testing.assert_array_equal(np.cumsum(x), out)
