"""The 128 x 128 forward kernel at the edges of its range, alone and with several layers in one launch, against fp64.

Tolerances: bf16 products are exact in fp32 and accumulate in fp32 over d_in (and 3 r) terms, so outputs agree to about
sqrt(d_in) 2^-24 of their size before the rounding to bf16 (2^-9) and losses to a few 1e-6; the rank-r term enters as
bf16 hi / lo pairs, 2^-16 of an eps-sized term."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_out, d_in, r: one tile; a tile and one row or sixteen columns more; the shortest pipeline and one with a slice for
# every stage; ranks of one and several extension slices; more tiles than one band; a d_in that its last slice does not fill and
# rows of odd length
SHAPES = [(128, 128, 128, 1), (129, 144, 192, 16), (255, 272, 320, 17), (257, 400, 704, 64), (1100, 1168, 256, 8), (130, 2064, 128, 4),
          (200, 131, 136, 4), (128, 300, 712, 16), (333, 1001, 248, 5)]


def _problem(i, n, d_out, d_in, pad, target):
    W, X, T = synth.single_layer_problem(70 + i, n, d_in, d_out, kind="rmsnorm", storage="bf16", target_storage=target)

    def dev(a, dt):
        t = torch.full((a.shape[0], a.shape[1] + pad), 3.0, device="cuda", dtype=dt)
        t[:, :a.shape[1]] = torch.from_numpy(a).cuda().to(dt)
        return t[:, :a.shape[1]]
    return W, X, T, dev(W, torch.bfloat16), dev(X, torch.bfloat16), dev(T, torch.bfloat16 if target == "bf16" else torch.float32)


@pytest.mark.parametrize("flags", [0, binding.ONE_SIDED])
def test_layers_of_all_shapes_in_one_call(flags):
    ctx = binding.Context()
    probs = [_problem(i, n, do, di, 8 * (i % 2), "bf16" if i % 3 else "f32") + (r,) for i, (n, do, di, r) in enumerate(SHAPES)]
    out = torch.zeros(len(probs), 4, dtype=torch.float64, device="cuda")
    ctx.step_many([(binding.make_layer(Wd, Xd, r), Wd, Xd, binding.make_loss(Td), 900 + i, out[i], None)
                   for i, (_, _, _, Wd, Xd, Td, r) in enumerate(probs)], 1, EPS, LR, flags)
    ctx.check()
    for i, (W, X, T, Wd, _, _, r) in enumerate(probs):
        o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 900 + i, storage="bf16", one_sided=bool(flags & binding.ONE_SIDED))
        got = out[i].cpu().numpy()
        assert abs(got[0] - o["L0"]) < 5e-6 * o["L0"], (i, got, o["L0"])
        assert abs(got[1] - o["Lp"]) < 5e-6 * o["Lp"], (i, got, o["Lp"])
        # (the accumulated rounding is common to the evaluations: what is left of it, over 2 eps)
        assert abs(got[3] - o["g"]) < 2e-2 * abs(o["g"]) + 1e-7 * o["L0"] / EPS, (i, got[3], o["g"])


@pytest.mark.parametrize("n,d_out,d_in,r", SHAPES)
def test_stored_outputs(n, d_out, d_in, r):
    ctx = binding.Context()
    W, X, _, Wd, Xd, _ = _problem(3, n, d_out, d_in, 8, "bf16")
    Y = torch.full((n, d_out + 8), 7.0, device="cuda", dtype=torch.bfloat16)
    L = binding.make_layer(Wd, Xd, r, Y=Y[:, :d_out])
    B = torch.linalg.qr(torch.randn(d_in, r, device="cuda"))[0].contiguous()
    ctx.perturbed_forward(L, Wd, Xd, B, 5, EPS, Y[:, :d_out], None, None)
    ctx.check()
    Yo = X.astype(np.float64) @ W.astype(np.float64).T
    Yo += EPS * (X.astype(np.float64) @ B.double().cpu().numpy()) @ oagzo.gaussian_factor(5, d_out, r).T
    got = Y.double().cpu().numpy()
    assert np.all(got[:, d_out:] == 7.0)
    err = np.abs(got[:, :d_out] - Yo)
    rms = np.sqrt(np.mean(Yo ** 2))
    assert np.all(err <= 2.0 ** -8 * np.abs(Yo) + 1e-5 * rms)       # one rounding to bf16
    assert np.linalg.norm(err) < 2.0 ** -8 * np.linalg.norm(Yo)
