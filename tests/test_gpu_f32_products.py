"""fp32 storage: the fp64 matrix-core forward and tall-skinny products at the edges of their tiles, against the oracle.

Tolerances: every product accumulates in fp64 and is rounded once to fp32 (2^-24), so losses agree to about 1e-7 and bases,
whose columns amplify the rounding of the sketches by their conditioning, to 1e-4 through the projector."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_in, d_out, r, row padding: around the 64 x 64 tile and the 32-wide slice, rows that do and do not start on 16 bytes,
# one and several blocks of 16 columns, fewer chunks of 16 and groups of 4 than the 16 waves, and more than one round of them
SHAPES = [(64, 32, 64, 1, 0), (63, 31, 65, 1, 0), (65, 33, 63, 4, 3), (129, 36, 127, 16, 0), (200, 100, 70, 17, 4), (150, 260, 66, 33, 0),
          (130, 77, 64, 64, 1), (1100, 1032, 72, 8, 0), (1, 5, 3, 1, 0)]


def _problem(i, n, d_in, d_out, pad):
    W, X, T = synth.single_layer_problem(40 + i, n, d_in, d_out, kind="rmsnorm", storage="f32")

    def dev(a):
        t = torch.zeros(a.shape[0], a.shape[1] + pad, device="cuda")
        t[:, :a.shape[1]] = torch.from_numpy(a).cuda()
        return t[:, :a.shape[1]]
    return W, X, T, dev(W), dev(X), dev(T)


@pytest.mark.parametrize("flags", [0, binding.SHARED_FORWARD, binding.ONE_SIDED])
def test_layers_of_all_shapes_in_one_call(flags):
    ctx = binding.Context()
    probs = [_problem(i, n, di, do, pad) + (r,) for i, (n, di, do, r, pad) in enumerate(SHAPES)]
    out = torch.zeros(len(probs), 4, dtype=torch.float64, device="cuda")
    ctx.step_many([(binding.make_layer(Wd, Xd, r), Wd, Xd, binding.make_loss(Td), 500 + i, out[i], None)
                   for i, (_, _, _, Wd, Xd, Td, r) in enumerate(probs)], 1, EPS, LR, flags)
    ctx.check()
    for i, (W, X, T, Wd, _, _, r) in enumerate(probs):
        o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 500 + i, one_sided=bool(flags & binding.ONE_SIDED))
        got = out[i].cpu().numpy()
        assert abs(got[0] - o["L0"]) < 1e-6 * o["L0"], (i, got, o["L0"])
        assert abs(got[1] - o["Lp"]) < 1e-6 * o["Lp"], (i, got, o["Lp"])
        assert abs(got[3] - o["g"]) < 1e-3 * abs(o["g"]) + 1e-6 * o["L0"] / EPS, (i, got[3], o["g"])
        moved = o["W_new"] - W
        assert np.linalg.norm((Wd.cpu().numpy() - W) - moved) < 5e-3 * np.linalg.norm(moved) + 1e-7 * np.linalg.norm(W), i


@pytest.mark.parametrize("shape", SHAPES)
def test_outputs_and_basis(shape):
    n, d_in, d_out, r, pad = shape
    ctx = binding.Context()
    W, X, _, Wd, Xd, _ = _problem(7, n, d_in, d_out, pad)
    Y = torch.full((n, d_out + pad), 7.0, device="cuda")[:, :d_out]
    B = torch.empty(d_in, r, device="cuda")
    L = binding.make_layer(Wd, Xd, r, Y=Y)
    ctx.basis(L, Xd, 1, 9, None, 0, B)
    ctx.perturbed_forward(L, Wd, Xd, B, 9, EPS, Y, None, None)
    ctx.check()
    Bh = B.double().cpu().numpy()
    want = oagzo.subspace_extract(X, r, 1, 9)["B"]
    assert np.linalg.norm(Bh @ Bh.T - want @ want.T) < 1e-4 * np.sqrt(r)
    Yo = X.astype(np.float64) @ W.astype(np.float64).T + EPS * (X.astype(np.float64) @ Bh) @ oagzo.gaussian_factor(9, d_out, r).T
    assert np.linalg.norm(Y.double().cpu().numpy() - Yo) < 5e-7 * np.linalg.norm(Yo)
