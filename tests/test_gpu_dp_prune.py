"""The library's DP with its pruned rows (gefen_dp_codebook) against the oracle's full scan,
bit for bit: exact ties, plateaus beside spikes, windows that span several 64-candidate
chunks, level counts around the backtrack's checkpoints (every 16 levels), as many bins as
entries, and counts too large to prune, which take the full scan."""
import numpy as np
import pytest
import torch

import oracle
from test_dp_prune_cpu import HEAVY, KINDS, heavy_top, histogram

pytestmark = pytest.mark.gpu

gf = pytest.importorskip("paper_2606_13894_amd")


def _check(h, k):
    cb, cost, status = gf.dp_codebook(torch.from_numpy(h.view(np.int64).copy()).cuda(), k)
    cb_ref, cost_ref, _, st_ref = oracle.dp_codebook(h, k)
    assert status == st_ref
    np.testing.assert_array_equal(cb.cpu().numpy(), cb_ref)
    assert cost == cost_ref


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nbins,k", [(4096, 256), (1000, 34), (256, 16)])
def test_dp_kinds(kind, nbins, k):
    _check(histogram(kind, nbins, seed=nbins + 7 * k), k)


@pytest.mark.parametrize("nbins,k,fill,seed,big", HEAVY)
def test_dp_heavy_bins(nbins, k, fill, seed, big):
    """Rows that later levels add, with far larger sums than the row whose bound they take."""
    _check(heavy_top(nbins, k, fill, seed, big), k)


@pytest.mark.parametrize("seed", range(40))
def test_dp_random_spikes(seed):
    """A few counts a bin beside up to four bins near the largest counts that still prune."""
    rng = np.random.default_rng(seed)
    nbins, k = int(rng.choice([256, 1024, 4096])), int(rng.choice([9, 16, 33, 64, 100]))
    fill = int(rng.integers(k + 2, 250))
    at = [np.arange(nbins - fill, nbins), np.arange(fill),
          np.sort(rng.choice(nbins, fill, replace=False))][seed % 3]
    h = np.zeros(nbins, dtype=np.uint64)
    h[at] = rng.integers(1, 4, fill).astype(np.uint64)
    n = int(rng.integers(1, 5))
    most = 0.9 * 2.0 ** 50 / nbins / n
    for _ in range(n):
        h[at[rng.integers(0, fill)]] = int(min(most, 10 ** rng.uniform(8, np.log10(most))))
    _check(h, k)


@pytest.mark.parametrize("k", [2, 3, 16, 17, 18, 19, 32, 33, 34, 50])
def test_dp_level_counts(k):
    _check(histogram("bell", 130, seed=k), k)
    _check(histogram("bell", k, seed=k), k)           # one bin per entry
    h = histogram("bell", k + 5, seed=k)
    h[1:7] = 0                                         # one bin fewer than entries
    _check(h, k)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33])
def test_dp_few_bins(n):
    """Running sums over fewer terms than a batch, and around whole batches."""
    h = np.zeros(64, dtype=np.uint64)
    h[np.random.default_rng(n).permutation(64)[:n]] = 1 + np.arange(n, dtype=np.uint64)
    _check(h, 8)


def test_dp_counts_too_large_to_prune():
    h = histogram("bell", 512, seed=3) * np.uint64(10 ** 10)
    assert float(h.sum()) * 512 > 2.0 ** 50
    _check(h, 24)
