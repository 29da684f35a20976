"""X Q for more than 32 columns (rows of X straight to registers, planes of Q through LDS): every number of 64-wide slices around the
pipeline's depth, widths that slices do not divide, tokens that workgroups do not, one workgroup per token block and several."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


def _layer(X, r):
    return binding.make_layer(torch.empty(16, X.shape[1], device="cuda", dtype=torch.bfloat16), X, r)


@pytest.mark.parametrize("r", [33, 48, 49, 64])
@pytest.mark.parametrize("n,d", [(64, 64), (65, 72), (130, 128), (129, 192), (200, 248), (131, 320), (66, 392), (190, 448), (333, 1024), (97, 1104)])
def test_power_sketch(n, d, r):
    """S = X^T (X Q): both products accumulate in fp32, over d and n terms, from exact bf16 products of the three planes of a
    factor: sqrt(terms) 2^-24 of the size of a column each"""
    ctx = binding.Context()
    X = torch.randn(n, d, device="cuda").bfloat16()
    Q = torch.randn(d, r, device="cuda")
    S = torch.empty(d, r, device="cuda")
    ctx.layer_forward_sketch(_layer(X, r), None, X, None, binding.SKETCH_POWER, Q, 0, S, None, None)
    ctx.check()
    want = X.double().T @ (X.double() @ Q.double())
    err = (S.double() - want).norm(dim=0) / want.norm(dim=0)
    assert err.max() < 4 * (n + d) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("r", [40, 64])
@pytest.mark.parametrize("n,d", [(4096, 136), (4100, 1048)])
def test_many_layers_take_twice_the_tokens(n, d, r):
    """Eight layers together give every compute unit a workgroup of 128 tokens, one alone does not: the same bits"""
    ctx = binding.Context()
    X = [torch.randn(n, d, device="cuda").bfloat16() for _ in range(8)]
    many = [torch.empty(d, r, device="cuda") for _ in X]
    ctx.basis_many([(_layer(x, r), x, 40 + i, None, b) for i, (x, b) in enumerate(zip(X, many))], 2, 0)
    for i, (x, b) in enumerate(zip(X, many)):
        one = torch.empty_like(b)
        ctx.basis_many([(_layer(x, r), x, 40 + i, None, one)], 2, 0)
        assert torch.equal(one, b), i
    ctx.check()
