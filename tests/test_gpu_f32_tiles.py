"""fp32 forwards in both tile sizes, at the edges of either and around the number of tiles that decides: losses and outputs from fp64
accumulators, so they agree with fp64 to its rounding (losses) and to one rounding to fp32 (outputs)."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_out, d_in, r: tiles of 32 (one, a row or column more, ranks past a slice, d_in below, at and past the slices in flight,
# rows that are not 16-byte vectors), 127 and 128 tiles of 64
SHAPES = [(32, 32, 32, 1), (33, 65, 31, 4), (64, 31, 129, 33), (100, 96, 160, 16), (1, 7, 5, 1), (95, 33, 257, 64), (127 * 64, 64, 36, 2), (8192, 61, 68, 3)]


@pytest.mark.parametrize("n,d_out,d_in,r", SHAPES)
def test_step_and_stored_output(n, d_out, d_in, r):
    r = min(r, n, d_in)
    ctx = binding.Context()
    W, X, T = synth.single_layer_problem(11, n, d_in, d_out, kind="rmsnorm", storage="f32")
    Wd, Xd, Td = (torch.from_numpy(a).cuda() for a in (W, X, T))
    Y = torch.empty(n, d_out, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    L = binding.make_layer(Wd, Xd, r, Y=Y)
    ctx.layer_forward_sketch(L, Wd, Xd, Y, binding.SKETCH_NONE, None, 0, None, binding.make_loss(Td), loss)
    ctx.check()
    want = X.astype(np.float64) @ W.astype(np.float64).T
    assert np.all(np.abs(Y.double().cpu().numpy() - want) <= 2.0 ** -24 * np.abs(want) + 1e-13 * np.abs(want).max())
    l0 = np.mean((want - T.astype(np.float64)) ** 2)
    assert abs(loss.item() - l0) <= 1e-12 * l0
    out = torch.zeros(2, 4, dtype=torch.float64, device="cuda")
    Ws = Wd.clone()
    ctx.step(binding.make_layer(Wd, Xd, r), Wd, Xd, binding.make_loss(Td), 1, EPS, LR, 5, 0, out[0])
    ctx.step(binding.make_layer(Ws, Xd, r), Ws, Xd, binding.make_loss(Td), 1, EPS, LR, 5, binding.SHARED_FORWARD, out[1])
    ctx.check()
    o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 5, storage="f32")
    for got in out.cpu().numpy():
        assert abs(got[0] - o["L0"]) <= 1e-9 * o["L0"] and abs(got[1] - o["Lp"]) <= 1e-6 * o["Lp"]
        assert abs(got[3] - o["g"]) <= 2e-3 * abs(o["g"]) + 1e-9 * o["L0"] / EPS
