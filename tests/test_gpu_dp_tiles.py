"""The DP's levels in one launch (gefen_dp_codebook) against the oracle's full scan, bit for
bit: bins and entries around the 16-row tiles and the first level of that launch, tiles that
a level reaches late, windows longer than a chunk with and without pruning, two DPs at
once on two streams, and waits between the tiles that run out."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from test_dp_prune_cpu import histogram
from test_gpu_dp_prune import _check

pytestmark = pytest.mark.gpu

gf = pytest.importorskip("paper_2606_13894_amd")


@pytest.mark.parametrize("k", [7, 8, 9, 10, 12])
@pytest.mark.parametrize("b", [15, 16, 17, 31, 33, 48, 200])
def test_tile_edges(b, k):
    _check(histogram("bell", b, seed=b + k), k)


@pytest.mark.parametrize("b,k", [(300, 250), (1024, 250), (2000, 9), (4096, 12)])
def test_late_tiles_and_long_windows(b, k):
    _check(histogram("flat", b, seed=b), k)
    _check(histogram("comb", b, seed=b), k)


def test_long_windows_without_pruning():
    h = histogram("bell", 1500, seed=5) * np.uint64(10 ** 10)
    assert float(h.sum()) * 1500 > 2.0 ** 50
    _check(h, 11)


@pytest.mark.parametrize("kind", ["bell", "flat", "comb", "gaps"])
@pytest.mark.parametrize("nbins,k", [(48, 9), (500, 64), (2000, 40), (4096, 256)])
def test_whole_windows(nbins, k, kind):
    """Counts too large to prune: every candidate of every row, ties included."""
    h = histogram(kind, nbins, seed=nbins + k)
    h *= np.uint64(int(2.0 ** 51 / nbins / float(h.sum())) + 1)
    assert float(h.sum()) * nbins > 2.0 ** 50
    _check(h, k)


def test_two_streams():
    hs = [histogram(kind, 4096, seed=9) for kind in ("bell", "two_scales")]
    dev = [torch.from_numpy(h.view(np.int64).copy()).cuda() for h in hs]
    streams = [torch.cuda.Stream() for _ in hs]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        for d, s in zip(dev, streams):
            with torch.cuda.stream(s):
                got.append(gf.dp_codebook(d, 256, stream=s))
        torch.cuda.synchronize()
        for h, (cb, cost, status) in zip(hs, got):
            ref = oracle.dp_codebook(h, 256)
            assert status == ref[3] and cost == ref[1]
            np.testing.assert_array_equal(cb.cpu().numpy(), ref[0])


@pytest.mark.parametrize("nbins,k", [(40, 9), (200, 50), (1000, 34), (1024, 256)])
@pytest.mark.parametrize("kind", ["bell", "gaps"])
def test_waits_that_run_out(nbins, k, kind):
    """Every wait between the row tiles given up at once (a poll limit below none): one
    workgroup takes the levels instead, with the same result."""
    h = histogram(kind, nbins, seed=nbins + k)
    d = torch.from_numpy(h.view(np.int64).copy()).cuda()
    cb = torch.empty(k, dtype=torch.float64, device="cuda")
    cost = torch.empty(1, dtype=torch.float64, device="cuda")
    status = torch.empty(1, dtype=torch.int32, device="cuda")
    call = gf.load_library().gefen_internal_dp_codebook
    p = ctypes.c_void_p
    assert call(p(d.data_ptr()), ctypes.c_int32(nbins), ctypes.c_int32(k), p(cb.data_ptr()),
                p(cost.data_ptr()), p(status.data_ptr()), ctypes.c_int32(-1),
                p(torch.cuda.current_stream().cuda_stream)) == 0
    ref = oracle.dp_codebook(h, k)
    assert status.item() == ref[3]
    np.testing.assert_array_equal(cb.cpu().numpy(), ref[0])
    assert cost.item() == ref[1]
