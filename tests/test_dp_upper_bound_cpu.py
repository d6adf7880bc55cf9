"""The DP's upper bound on the candidates (Alg. 3, App. D), checked on the CPU against the
oracle's full scan: inside a tile of rows, no row needs a candidate above the largest one
that lies within the rounding slack of the minimum of the tile's highest row. Codebook, cost
and interval starts bit for bit, with the lower bound of the level before."""
import numpy as np
import pytest

import oracle
from test_dp_prune_cpu import HEAVY, KINDS, heavy_top, histogram


def bounded_dp(hist, k, tile):
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
    cut = 0
    for j in range(2, k + 1):
        rmax = b - k + j
        new, nlow, hi = np.full(b + 1, np.inf), np.zeros(b + 1, dtype=np.int64), b
        for r in range(rmax, (b if j == k else j) - 1, -1):   # a tile's highest row first
            top = r == rmax or r % tile == 0
            lo = j if j in (2, k) else max(j, low[r] if r < rmax else low[r - 1])
            up = r if top or j == k else min(r, hi)
            cut += r - up
            l = np.arange(lo, up + 1)
            s0, s1, s2 = z0[r] - z0[l - 1], z1[r] - z1[l - 1], z2[r] - z2[l - 1]
            w = s2 - 2.0 * s1 + s0 if j == k else s2 - s1 * s1 / s0
            cand = d[l - 1] + w
            i = int(np.argmin(cand))
            new[r], split[j, r] = cand[i], lo + i
            slack = 2.0 ** -53 * (256.0 * (z0[b] if r == rmax else z0[r]) + 32.0 * k * cand[i])
            near = np.nonzero(cand <= cand[i] + slack)[0]
            nlow[r] = lo + int(near[0])
            if top:
                hi = lo + int(near[-1])
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
    return cb, d[b], bounds, cut


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nbins,k,tile", [(256, 16, 16), (320, 64, 16), (193, 5, 64)])
def test_bounded_scan_equals_the_full_scan(kind, nbins, k, tile):
    h = histogram(kind, nbins, seed=nbins + 3 * k)
    cb, cost, bounds, cut = bounded_dp(h, k, tile)
    cb_ref, cost_ref, bounds_ref, st = oracle.dp_codebook(h, k)
    assert st == 0
    np.testing.assert_array_equal(cb, cb_ref)
    assert cost == cost_ref
    np.testing.assert_array_equal(bounds, bounds_ref)
    if kind == "bell":
        assert cut > 0


@pytest.mark.parametrize("nbins,k,fill,seed,big", HEAVY)
def test_bounds_handed_past_heavy_bins(nbins, k, fill, seed, big):
    h = heavy_top(nbins, k, fill, seed, big)
    cb, cost, bounds, _ = bounded_dp(h, k, 16)
    cb_ref, cost_ref, bounds_ref, st = oracle.dp_codebook(h, k)
    assert st == 0
    np.testing.assert_array_equal(cb, cb_ref)
    assert cost == cost_ref
    np.testing.assert_array_equal(bounds, bounds_ref)
