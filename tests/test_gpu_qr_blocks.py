"""QR at the edges of its blocking: ranks around multiples of sixteen (blocks of the factorisation), row counts around multiples
of 128 (a workgroup's rows), square inputs.  The fp64 factorisation is exact to fp32 rounding: tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 127, 128, 129, 4231])
@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64])
def test_qr(d, r):
    rng = np.random.default_rng(100 * d + r)
    Y = rng.standard_normal((d, r)) @ np.diag(np.logspace(0, -3 if d > 64 else -1, r))
    Y = Y.astype(np.float32)
    Q = torch.full((d, r), 9.0, dtype=torch.float32, device="cuda")
    ctx = binding.Context()
    ctx.qr(torch.from_numpy(Y).cuda(), Q)
    ctx.check()
    want, _ = oagzo.qr_pos(Y.astype(np.float64))
    got = Q.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got.T @ got - np.eye(r)) < 1e-5
    assert np.linalg.norm(got - want) < 1e-5 * np.linalg.norm(want)
