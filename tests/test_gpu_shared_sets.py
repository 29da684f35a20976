"""The shared schedule (f0, f+ and f- from one pass) over several layers in one launch: every layer's losses, scalar and weights are
those of a launch of its own, bit for bit, and agree with Alg. 2 in fp64.

Tolerances as for the forwards in 128 x 128 tiles: bf16 products accumulate in fp32 over d_in, a few 1e-6 of a loss; g is an
eps-sized difference of two of them."""
import numpy as np
import pytest
import torch

from launches import kernels
from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_out, d_in, r (of one padded rank or two), target: one tile; tiles in numbers that 8 does not divide; shapes that tiles do not
# divide; several extension slices; depths in another order than the list's
SHAPES = [(256, 256, 128, 16, "bf16"), (768, 768, 192, 9, "bf16"), (512, 256, 704, 64, "f32"), (300, 520, 136, 16, "bf16"), (257, 769, 320, 33, "f32"),
          (256, 2816, 256, 16, "bf16")]


@pytest.mark.parametrize("count", [1, 2, len(SHAPES)])
def test_layers_share_a_launch(count):
    ctx = binding.Context()
    probs = []
    for i, (n, d_out, d_in, r, target) in enumerate(SHAPES[-count:]):
        W, X, T = synth.single_layer_problem(140 + i, n, d_in, d_out, kind="rmsnorm", storage="bf16", target_storage=target)
        dev = [torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (W, X)]
        probs.append((W, X, T, r, *dev, torch.from_numpy(T).cuda().to(torch.bfloat16 if target == "bf16" else torch.float32)))
    out = torch.zeros(2, count, 4, dtype=torch.float64, device="cuda")
    together = [p[4].clone() for p in probs]
    ctx.step_many([(binding.make_layer(w, p[5], p[3]), w, p[5], binding.make_loss(p[6]), 60 + i, out[0, i], None)
                   for i, (p, w) in enumerate(zip(probs, together))], 1, EPS, LR, binding.SHARED_FORWARD)
    for i, p in enumerate(probs):
        W, X, T, r, Wd, Xd, Td = p
        ctx.step(binding.make_layer(Wd, Xd, r), Wd, Xd, binding.make_loss(Td), 1, EPS, LR, 60 + i, binding.SHARED_FORWARD, out[1, i])
        assert torch.equal(Wd, together[i]), i
        o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 60 + i, storage="bf16")
        got = out[1, i].cpu().numpy()
        assert abs(got[0] - o["L0"]) < 5e-6 * o["L0"] and abs(got[2] - o["Lm"]) < 5e-6 * o["Lm"], (i, got, o["L0"], o["Lm"])
        assert abs(got[3] - o["g"]) < 2e-2 * abs(o["g"]) + 1e-7 * o["L0"] / EPS, (i, got[3], o["g"])
    ctx.check()
    assert torch.equal(out[0], out[1])


# a head; layers short of a tile in each direction; one that the persistent kernel takes
@pytest.mark.parametrize("n,d_out,d_in,r,ce,reads", [(300, 1000, 264, 1, True, False), (700, 4000, 512, 16, True, False), (200, 512, 2048, 16, False, False), (512, 200, 512, 1, False, False),
                                                     (512, 512, 64, 40, False, False), (512, 512, 128, 16, False, True), (257, 769, 1024, 1, False, True)])
def test_operands_are_made_where_a_forward_reads_them(n, d_out, d_in, r, ce, reads):
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    w, x = (torch.randn(s, device="cuda").bfloat16() for s in ((d_out, d_in), (n, d_in)))
    t = torch.randint(0, d_out, (n,), device="cuda", dtype=torch.int32) if ce else torch.randn(n, d_out, device="cuda").bfloat16()
    out = torch.zeros(4, dtype=torch.float64, device="cuda")
    item = (binding.make_layer(w, x, r), w, x, binding.make_loss(t, kind=binding.LOSS_CE if ce else binding.LOSS_MSE), 3, out, None)
    torch.cuda.synchronize()

    def call():
        ctx.step_many([item], 1, EPS, LR, binding.SHARED_FORWARD)
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
    names, _ = kernels(stream, call)
    assert any("_ext_kernel" in name or "ext_prep" in name for name in names) == reads, names
    ctx.check()
    assert torch.isfinite(out).all()
    ctx.close()
