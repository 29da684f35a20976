"""Squared errors of several layers whose 256 x 256 tiles share a launch, workgroups walking lists that go through all of them: every
loss, scalar and weight has the bits of launches of their own (timing a kernel class makes every forward one), also of layers that take
128 x 128 tiles when alone, and the losses agree with fp64.

Tolerance of L0: bf16 products accumulate in fp32 over d_in, a few 1e-6 of a loss of comparable residuals."""
import pytest
import torch

from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = 1e-3, 1e-3

# tokens, r, (d_in, d_out) per layer, target: layers of 160 tiles and more with ends that no tile divides; d_in that slices do not
# divide; target rows off 16 bytes (fp64 squares), a last half tile that overlaps by no multiple of 16, by one, by all; layers of few deep tiles
RAGGED = [(512, 4096), (520, 3600), (2048, 1111), (4096, 1024), (4096, 1040), (3072, 264), (128, 3000)]
# tiles in numbers that neither 8 nor a round of them divides; two problems of one depth
ALIGNED = [(256, 2816), (512, 2560), (1024, 3072), (512, 256)]


@pytest.mark.parametrize("flags", [0, binding.ONE_SIDED])
@pytest.mark.parametrize("n,r,shapes", [(3001, 16, RAGGED), (2690, 17, RAGGED), (4096, 8, ALIGNED), (300, 64, RAGGED[2:6])])
def test_same_as_launches_of_their_own(n, r, shapes, flags):
    given = []
    for i, (d_in, d_out) in enumerate(shapes):
        x = synth.device_powerlaw_x(70 + i, n, d_in)
        given.append((x,) + synth.device_weights_and_target(170 + i, x, d_out))
    got = []
    for mask in (0, 1 << binding.PROF_GEMM):
        ctx = binding.Context()
        ctx.profile_enable(mask)
        w = [g[1].clone() for g in given]
        out = torch.full((2, len(given), 4), float("nan"), dtype=torch.float64, device="cuda")
        for k in range(2):
            ctx.step_many([(binding.make_layer(w[i], x, r), w[i], x, binding.make_loss(t), 40 + i + 100 * k, out[k, i], None)
                           for i, (x, _, t) in enumerate(given)], 1, EPS, LR, flags)
        ctx.check()
        got.append([out] + w)
        ctx.close()
    assert torch.isfinite(got[0][0]).all()
    assert all(torch.equal(a, b) for a, b in zip(*got))
    for i, (x, w0, t) in enumerate(given):
        y = x.double() @ w0.double().T
        want = ((y - t.double()) ** 2).mean().item()
        assert abs(got[0][0][0, i, 0].item() - want) < 5e-6 * want, i
