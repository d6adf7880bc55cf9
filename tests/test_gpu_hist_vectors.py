"""The histogram kernel's register path (uniform blocks of whole 4-element vectors) at the
edges of its vector counts, at both gradient types, aligned or not, against the same bins in
float64 on the CPU; whole counts, so exactly. With zero blocks and infinite gradients.
"""
import pytest

pytestmark = pytest.mark.gpu

# vectors of a block: lane groups (<= 32), 1, 2, 4 and 8 a lane, longer (by vectors only where
# the shorter blocks hold at least as many elements), and a streamed one
PERIODS = [4, 8, 36, 128, 132, 256, 260, 512, 516, 1024, 1028, 2048, 2052, 6148, 8192, 8196, 30]


def _expect(grads, periods, bins):
    import torch
    h = torch.zeros(bins, dtype=torch.int64)
    for g, p in zip(grads, periods):
        x = g.detach().cpu().double().view(-1, p)
        a = x.abs().amax(1, keepdim=True)
        x = (x / a)[(a > 0).view(-1)].reshape(-1)
        x = x[~x.isnan()]
        at = ((x + 1.0) * (0.5 * bins)).floor().long().clamp(max=bins - 1)
        h += torch.bincount(at, minlength=bins)
    return h


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("rows", [41, 400])   # the longer blocks hold most elements, or the fewer
def test_histogram_of_uniform_blocks(bf16, shift, bits, rows):
    import torch

    import paper_2606_13894_amd as gf
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    dt = torch.bfloat16 if bf16 else torch.float32
    grads = []
    for i, p in enumerate(PERIODS):
        n = p * (rows if p < 1000 else 7)
        buf = torch.randn(n + shift, generator=gen, device="cuda").mul_(10.0 ** (i % 5 - 2)).to(dt)
        g = buf[shift:]
        g[p:2 * p] = 0.0            # a zero block counts nothing
        g[2 * p] = -g[2 * p:3 * p].abs().max() * 2   # the block's maximum in its first element
        grads.append(g)
    st = gf.GefenState(grads, period_override=PERIODS, code_bits=bits)
    got = st.histogram(grads).cpu()
    assert torch.equal(got, _expect(grads, PERIODS, 16 << bits))


def test_infinite_gradients():
    import torch

    import paper_2606_13894_amd as gf
    periods = [64, 768, 4096]
    grads = [torch.linspace(-1.0, 1.0, 4 * p, device="cuda") for p in periods]
    st = gf.GefenState(grads, period_override=periods)
    for g in grads:
        g[3] = float("inf")
    got = st.histogram(grads).cpu()
    want = _expect(grads, periods, 4096)
    # inf / inf has no bin of its own: the conversion of NaN gives bin 0
    want[0] += len(periods)
    assert torch.equal(got, want)
