"""Orthonormalisations take different launches by what is in them: one workgroup a problem for few rows and up to 16 columns, Gram partials
summed ahead of the factorisation where there are many.  A layer's basis has the same bits whichever it is, that is whatever layers it
shares a call with; and the QR of explicit matrices at the edges of the one-workgroup form against fp64."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


# tokens, widths of the layers that are small alone, and of one that makes the call take the other launches
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,r,widths,other", [(300, 3, (8, 120, 128, 136, 256, 512), 520), (257, 16, (64, 248, 256, 500, 512), 2048), (2100, 9, (256, 264), 4096),
                                              (300, 64, (640, 72), 4104), (300, 20, (9728, 64), 264), (300, 20, (12288, 64), 264)])
def test_basis_in_any_company(n, r, widths, other, dtype):
    ctx = binding.Context()
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X = [torch.randn(n, d // 8 * 8, device="cuda").to(dt) for d in widths + (other,)]
    ranks = [min(r, x.shape[1]) for x in X]
    lay = [binding.make_layer(torch.empty(16, x.shape[1], device="cuda", dtype=dt), x, k) for x, k in zip(X, ranks)]
    many = [torch.full((x.shape[1], k), 9.0, device="cuda") for x, k in zip(X, ranks)]
    ctx.basis_many([(l, x, 3 + i, None, b) for i, (l, x, b) in enumerate(zip(lay, X, many))], 2, 0)
    for i, (l, x, b) in enumerate(zip(lay, X, many)):
        one = torch.full_like(b, 9.0)
        ctx.basis(l, x, 2, 3 + i, None, 0, one)
        assert torch.equal(one, b), (i, x.shape)
        assert (b.double().T @ b.double() - torch.eye(b.shape[1], device="cuda")).norm() < 1e-5
    ctx.check()


@pytest.mark.parametrize("d,r", [(2, 2), (15, 15), (100, 7), (256, 16), (257, 4), (383, 16), (511, 3), (512, 16), (513, 16)])
def test_qr(d, r):
    rng = np.random.default_rng(d + r)
    Y = (rng.standard_normal((d, r)) @ np.diag(np.logspace(0, -2, r))).astype(np.float32)
    Q = torch.full((d, r), 9.0, device="cuda")
    ctx = binding.Context()
    ctx.qr(torch.from_numpy(Y).cuda(), Q)
    ctx.check()
    want, _ = oagzo.qr_pos(Y.astype(np.float64))
    got = Q.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - want) < 1e-5 * np.linalg.norm(want)
    # no pivot at all is reported, as by the other launches
    ctx.qr(torch.from_numpy(np.zeros_like(Y)).cuda(), Q)
    with pytest.raises(binding.AgzoError):
        ctx.check()


@pytest.mark.parametrize("d", [300, 700])
@pytest.mark.parametrize("r", [1, 4, 5, 8, 9, 12, 13, 20, 21, 36, 49])
def test_ranks_that_fill_part_of_a_block(d, r):
    """the factorisation ends behind the last four columns that are there.  Bounds as above"""
    rng = np.random.default_rng(d + r)
    Y = (rng.standard_normal((d, r)) @ np.diag(np.logspace(0, -2, r))).astype(np.float32)
    Q = torch.full((d, r), 9.0, device="cuda")
    ctx = binding.Context()
    ctx.qr(torch.from_numpy(Y).cuda(), Q)
    ctx.check()
    want, _ = oagzo.qr_pos(Y.astype(np.float64))
    assert np.linalg.norm(Q.cpu().numpy().astype(np.float64) - want) < 1e-5 * np.linalg.norm(want)
    Y[:, r - 1] = 0.0                                              # the last pivot, of the last four columns
    ctx.qr(torch.from_numpy(Y).cuda(), Q)
    with pytest.raises(binding.AgzoError):
        ctx.check()
