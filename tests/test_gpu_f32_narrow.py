"""X Q of fp32 layers for one to four columns and rows of 1024 values or more: widths that chunks do not divide, rows that are not
16-byte vectors, tokens that workgroups do not divide.  fp64 sums, rounded once: P enters the stored output below through
eps P G^T, whose coefficient is large enough to show an error of one rounding."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("n,d,pad", [(4, 1024, 0), (5, 1028, 4), (7, 1027, 0), (33, 1281, 3), (130, 2303, 1), (66, 3072, 0)])
def test_projection(n, d, pad, r):
    ctx = binding.Context()
    X = torch.randn(n, d + pad, device="cuda")[:, :d]
    W, B = torch.zeros(24, d, device="cuda"), torch.randn(d, r, device="cuda")
    Y = torch.empty(n, 24, device="cuda")
    ctx.perturbed_forward(binding.make_layer(W, X, r, Y=Y), W, X, B, 9, 1.0, Y, None, None)
    ctx.check()
    G = torch.from_numpy(oagzo.gaussian_factor(9, 24, r)).cuda().double()
    P = (X.double() @ B.double()).float().double()
    want, size = P @ G.T, P.abs() @ G.abs().T
    # one rounding of P (a tie may fall the other way), one of Y, and the generator's 1e-6 of a normal
    assert ((Y.double() - want).abs() <= size * (2.0 ** -23 + 2e-6)).all()
    S = torch.empty(d, r, device="cuda")
    ctx.layer_forward_sketch(binding.make_layer(W, X, r), None, X, None, binding.SKETCH_POWER, B, 0, S, None, None)
    ctx.check()
    want = X.double().T @ P
    assert ((S.double() - want).norm(dim=0) <= 2.0 ** -22 * want.norm(dim=0)).all()
