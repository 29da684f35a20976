"""A basis of one column of fp32 activations: the projection finds the norm of the column that it multiplies with and divides its result by it.
Widths below, at and past the chunks of both forms and the line between them, rows that are no 16-byte vectors, alone and in company."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (5, 3), (17, 16), (40, 63), (300, 250), (33, 257), (100, 1000), (61, 1020), (300, 1023), (300, 1024), (7, 1027), (130, 2052), (600, 4100)]


def _randn(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *shape: torch.randn(*shape, device="cuda", generator=g)


def _want(X, q, K):
    q = q.double() / q.double().norm()
    for _ in range(K):
        q = X.double().T @ (X.double() @ q)
        q = q / q.norm()
    return q


@pytest.mark.parametrize("of_s0", [1.0, 1e-30, 1e30])
@pytest.mark.parametrize("n,d", SHAPES)
def test_from_a_given_sketch(n, d, of_s0):
    """against fp64: a power step rounds T and the sketch to fp32 once each, 2^-24 of a vector's norm; two steps and the last rounding"""
    ctx = binding.Context()
    randn = _randn(1000 * n + d)
    X, S0 = randn(n, d), of_s0 * randn(d, 1)
    L = binding.make_layer(torch.empty(16, d, device="cuda"), X, 1)
    B, many, other = torch.full((d, 1), 9.0, device="cuda"), torch.full((d, 1), 9.0, device="cuda"), torch.empty(72, 1, device="cuda")
    ctx.basis(L, X, 2, 3, S0, 0, B)
    # of unit length whatever was given, and along X^T X X^T X S0 up to the roundings as X's condition lets them grow
    want = _want(X, S0, 2)
    first = (X.double() @ (S0.double() / S0.double().norm())).norm() * torch.linalg.matrix_norm(X.double(), 2) / (X.double().T @ (X.double() @ (S0.double() / S0.double().norm()))).norm()
    second = torch.linalg.matrix_norm(X.double(), 2) ** 2 / (X.double().T @ (X.double() @ _want(X, S0, 1))).norm()
    assert (B.double() - want).norm() <= 2.0 ** -23 * (1 + 2 * second * (1 + first))
    Xo = randn(50, 72)
    ctx.basis_many([(L, X, 3, S0, many), (binding.make_layer(torch.empty(16, 72, device="cuda"), Xo, 1), Xo, 4, randn(72, 1), other)], 2, 0)
    ctx.check()
    assert torch.equal(B, many)


@pytest.mark.parametrize("d", [64, 1024])
def test_no_column_is_reported(d):
    ctx = binding.Context()
    X, B = _randn(d)(100, d), torch.empty(d, 1, device="cuda")
    L = binding.make_layer(torch.empty(16, d, device="cuda"), X, 1)
    ctx.basis(L, X, 1, 3, torch.zeros(d, 1, device="cuda"), 0, B)
    with pytest.raises(binding.AgzoError):
        ctx.check()
    ctx.basis(L, X, 1, 3, None, 0, B)
    ctx.check()
