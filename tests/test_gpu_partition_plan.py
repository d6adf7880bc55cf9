"""Block inference (gefen_partition_scores, the inference of gefen_init) against the oracle
over the shapes its plan treats differently: chunks with a remainder, primes that the base
divisor lacks, sub-sums of a large prime factor, several tensors in one call. Scores are
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
