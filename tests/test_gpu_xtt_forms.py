"""X^T T for r > 16 in its two forms: four waves to a panel, or a wave to a panel.  Both add the shares of four waves in wave order."""
import numpy as np
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


def _layer(X, r):
    return binding.make_layer(torch.empty(16, X.shape[1], device="cuda", dtype=torch.bfloat16), X, r)


@pytest.mark.parametrize("n,d,r", [(16384, 1024, 17), (16384, 1024, 64), (8192, 16384, 33), (8192, 16384, 64)])
def test_a_waves_share_is_summed_by_itself(n, d, r):
    """Whole numbers whose sum over a share (every fourth step of 32 tokens, 8 of a range's 32) stays below 2^24 and over a range
    does not.  The tokens of a share repeat in each of its steps, so that its sum is a multiple of 8 and adding four of them is
    exact too: 8 x 4 x 32 x 255^2 < 2^27.  Token counts and widths make ranges of 1024."""
    rng = np.random.default_rng(r)
    base = rng.integers(140, 256, (128, d))
    X = torch.from_numpy(np.tile(base, (n // 128, 1)).astype(np.float32)).cuda().bfloat16()
    Q = torch.zeros(d, r, device="cuda")
    Q[torch.arange(r), torch.arange(r)] = 1.0                      # X Q: the first columns of X
    S = torch.empty(d, r, device="cuda")
    ctx = binding.Context()
    ctx.layer_forward_sketch(_layer(X, r), None, X, None, binding.SKETCH_POWER, Q, 0, S, None, None)
    ctx.check()
    want = (base.T @ base[:, :r]) * (n // 128)
    assert np.array_equal(S.double().cpu().numpy(), want.astype(np.float64))


@pytest.mark.parametrize("r", [17, 33, 64])
@pytest.mark.parametrize("n,d", [(333, 2568), (1152, 2560), (129, 6144)])
def test_both_forms_give_the_same_bits(n, d, r):
    """Six layers in one call give each wave a panel, one alone does not; ranges of four steps, of three, and of one"""
    ctx = binding.Context()
    X = [torch.randn(n, d, device="cuda").bfloat16() for _ in range(6)]
    many = [torch.empty(d, r, device="cuda") for _ in X]
    ctx.basis_many([(_layer(x, r), x, 40 + i, None, b) for i, (x, b) in enumerate(zip(X, many))], 1, 0)
    for i, (x, b) in enumerate(zip(X, many)):
        one = torch.empty_like(b)
        ctx.basis_many([(_layer(x, r), x, 40 + i, None, one)], 1, 0)
        assert torch.equal(one, b), i
    ctx.check()
