"""Block inference (gefen_partition_scores, the inference of gefen_init) against the oracle
over the shapes its plan treats differently: chunks with a remainder, primes that the base
divisor lacks, sub-sums of a large prime factor, several tensors in one call, sizes whose sums
would not fit the room for them, tensors that take several plans. Scores are
float64 sums of at most 4e5 terms in another order: 1e-9 relative, as the other partition
tests."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

gf = pytest.importorskip("paper_2606_13894_amd")


def _grad(n, dtype, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randn(n, generator=gen, device="cuda").to(dtype)


def _bits(g):
    from parity import grad_bits
    return grad_bits(g)


@pytest.mark.parametrize("n", [2, 6, 2047, 2048, 2049, 4096, 15838, 80018, 49155, 98304, 49152,
                               180180, 50257, 166368, 65231, 98466, 46189])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_scores_over_sizes(n, dtype):
    g = _grad(n, dtype, n)
    divs, scores, period = gf.partition_scores(g, 1e-8)
    d_ref, s_ref, p_ref = oracle.partition(_bits(g), 1e-8)
    np.testing.assert_array_equal(divs, d_ref)
    np.testing.assert_allclose(scores, s_ref, rtol=1e-9, atol=1e-300)
    assert period == p_ref


def test_blocks_that_repeat_have_score_zero():
    """Equal blocks are summed alike, whatever path their divisor takes."""
    row = _grad(29 * 96, torch.float32, 5)
    divs, scores, _ = gf.partition_scores(row.repeat(40), 1e-8)
    zero = (divs % row.numel() == 0)
    assert zero.sum() > 3 and not scores[zero].any()


def test_several_tensors_in_one_call():
    sizes = [(768, torch.float32), (3072 * 5, torch.bfloat16), (1, torch.float32),
             (29 * 1733, torch.float32), (97, torch.bfloat16), (4096 * 3, torch.float32)]
    grads = [_grad(n, dt, 3 + i) for i, (n, dt) in enumerate(sizes)]
    st = gf.GefenState(grads)
    assert st.periods == [oracle.partition(_bits(g), 1e-8)[2] for g in grads]


@pytest.mark.parametrize("n,dtype", [(7207200, torch.float32), (9699690, torch.bfloat16),
                                     (24504480, torch.float32), (73513440, torch.bfloat16)])
def test_scores_with_little_stored(n, dtype):
    """So many divisors that the small ones are summed and contrasted straight from the
    gradient (up to 1023 elements: 1, 4 and 16 lanes a block), against float64
    sums of torch's logarithms."""
    g = _grad(n, dtype, n)
    divs, scores, period = gf.partition_scores(g, 1e-8)
    z = g.double().square_().add_(1e-8).log_()
    ref = []
    for p in map(int, divs):
        mu = z.view(-1, p).sum(1) / p
        ref.append(((mu[1:] - mu[:-1]).abs_().sum() / max(mu.numel() - 1, 1)).item())
    ref = np.array(ref)
    np.testing.assert_allclose(scores, ref, rtol=1e-9, atol=1e-300)
    peaks = [i for i in range(1, len(ref) - 1) if ref[i] > ref[i - 1] and ref[i] > ref[i + 1]]
    assert period == divs[max(peaks, key=lambda i: ref[i])]
    row = g[:n // 180]
    divs, scores, _ = gf.partition_scores(row.repeat(180), 1e-8)
    assert not scores[divs % row.numel() == 0].any()


def test_tensors_over_several_plans():
    """Tensors of 15 MB of sums each, between smaller ones: two plans."""
    sizes = [768, 1081080, 1081080, 97, 1081080, 3072 * 5, 1081080, 1081080, 1081080, 50257]
    grads = [_grad(n, torch.float32, 11 + i) for i, n in enumerate(sizes)]
    st = gf.GefenState(grads)
    assert st.periods == [oracle.partition(_bits(g), 1e-8)[2] for g in grads]
