"""A lone bf16 layer's basis of one column: its projection adds up the partial sums of a short column by itself, and one workgroup normalises the last one.
Columns below, at and past the widths and token counts where either ends, alone and beside a layer that takes the other launches: the same bits,
and the column that fp64 finds."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu

# (tokens, width): blocks of 256 rows, two and more turns of partial sums, a workgroup a compute unit and one more
SHAPES = [(1, 8), (40, 248), (300, 256), (300, 264), (2049, 504), (2048, 512), (432, 520), (432, 1016), (432, 1024), (1000, 1024), (100, 1032), (4096, 256), (4097, 256)]


@pytest.mark.parametrize("K", [1, 3])
@pytest.mark.parametrize("n,d", SHAPES)
def test_alone_and_in_company(n, d, K):
    ctx = binding.Context()
    g = torch.Generator(device="cuda").manual_seed(10 * n + d)
    X, other = (torch.randn(t, w, device="cuda", generator=g).bfloat16() for t, w in ((n, d), (500, 2048)))
    lay = [binding.make_layer(torch.empty(16, x.shape[1], device="cuda", dtype=torch.bfloat16), x, 1) for x in (X, other)]
    alone, many, beside = torch.full((d, 1), 9.0, device="cuda"), torch.full((d, 1), 9.0, device="cuda"), torch.empty(2048, 1, device="cuda")
    ctx.basis(lay[0], X, K, 5, None, 0, alone)
    ctx.basis_many([(lay[0], X, 5, None, many), (lay[1], other, 6, None, beside)], K, 0)
    ctx.check()
    assert torch.equal(alone, many)
    # from the first sketch on (X^T of the column that a basis without power steps starts from): each step rounds the column and T to fp32
    first = torch.empty_like(alone)
    ctx.basis(lay[0], X, 0, 5, None, 0, first)
    q = first.double()
    for _ in range(K):
        q = X.double().T @ (X.double() @ q)
        q = q / q.norm()
    assert (alone.double() - q).norm() <= (K + 1) * 4e-6


@pytest.mark.parametrize("n,d", [(300, 264), (432, 1024)])
def test_no_activations_are_reported(n, d):
    ctx = binding.Context()
    X, B = torch.zeros(n, d, device="cuda", dtype=torch.bfloat16), torch.empty(d, 1, device="cuda")
    ctx.basis(binding.make_layer(torch.empty(16, d, device="cuda", dtype=torch.bfloat16), X, 1), X, 2, 3, None, 0, B)
    with pytest.raises(binding.AgzoError):
        ctx.check()


@pytest.mark.parametrize("d", [1, 63, 255, 256, 257, 1000, 1024, 1025])
def test_one_column(d):
    """against fp64: the column is rounded once"""
    ctx = binding.Context()
    Y, Q = torch.randn(d, 1, device="cuda", generator=torch.Generator(device="cuda").manual_seed(d)), torch.full((d, 1), 9.0, device="cuda")
    ctx.qr(Y, Q)
    ctx.check()
    want = Y.double() / Y.double().norm()
    assert ((Q.double() - want).abs() <= 2.0 ** -23 * want.abs()).all()
