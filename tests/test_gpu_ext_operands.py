"""The rank-r term alone (W = 0) over ranks around the eights and sixteens of its operands' segments, both signs and both schedules: losses against
fp64 with the basis that the step used.  The term enters as bf16 hi / lo pairs: 2^-16 of it."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu
EPS = 0.5


@pytest.mark.parametrize("n,d_in,d_out", [(300, 1032, 264), (1000, 2048, 520)])
@pytest.mark.parametrize("r", [1, 7, 8, 9, 16, 17, 24, 33, 48, 49, 64])
def test_losses(n, d_in, d_out, r):
    g = torch.Generator(device="cuda").manual_seed(r)
    x = torch.randn(n, d_in, device="cuda", generator=g).bfloat16()
    w = torch.zeros(d_out, d_in, device="cuda", dtype=torch.bfloat16)
    t = torch.randn(n, d_out, device="cuda", generator=g).bfloat16()
    G = torch.from_numpy(oagzo.gaussian_factor(9, d_out, r)).cuda().double()
    ctx = binding.Context()
    for flags in (0, binding.SHARED_FORWARD):
        out, b = torch.zeros(4, dtype=torch.float64, device="cuda"), torch.empty(d_in, r, device="cuda")
        ctx.step_no_update(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 1, EPS, 9, flags, out, b)
        ctx.check()
        D = (x.double() @ b.double()) @ G.T
        want = np.array([((s * EPS * D - t.double()) ** 2).mean().item() for s in (0, 1, -1)])
        assert np.all(np.abs(out[:3].cpu().numpy() - want) < 1e-4 * want), (flags, out, want)
