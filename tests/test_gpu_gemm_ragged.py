"""The persistent 256 x 256 forward kernel where tiles and slices do not divide the layer, in each of its output forms, against
fp64.  Tiles that would hang over an edge start earlier and leave out what their neighbour has counted; a last slice that d_in
does not fill reads zeros past it; rows of target or output need no alignment.

Tolerances as in test_gpu_gemm_mid.py: fp32 sums over d_in (and 3 r) terms, one rounding of a stored output, and for the
cross-entropy fp32 sums of 128 exponentials."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_out, d_in, r, padding of the rows of target or output: one tile; one row / column more or fewer; a whole number of
# slices, one chunk more, one chunk fewer; the shortest d_in; ranks of one and of several extension slices; more tiles than one band
SHAPES = [(256, 256, 128, 1, 0), (257, 259, 136, 4, 0), (511, 513, 248, 17, 1), (300, 777, 200, 64, 3), (2400, 264, 192, 16, 8),
          (512, 512, 328, 8, 0), (512, 300, 320, 5, 4), (270, 4099, 152, 8, 0)]


def _dev(a, dt, pad, fill=3.0):
    t = torch.full((a.shape[0], a.shape[1] + pad), fill, device="cuda", dtype=dt)
    t[:, :a.shape[1]] = torch.from_numpy(a).cuda().to(dt)
    return t[:, :a.shape[1]]


def _large(L):
    L.tiling = binding.TILING_LARGE
    return L


@pytest.mark.parametrize("target", ["bf16", "f32"])
@pytest.mark.parametrize("n,d_out,d_in,r,pad", SHAPES)
def test_squared_error(n, d_out, d_in, r, pad, target):
    W, X, T = synth.single_layer_problem(n, n, d_in, d_out, kind="rmsnorm", storage="bf16", target_storage=target)
    # rows behind d_in hold values that would show (X) or spread (NaN) if a last slice read them
    Xd = _dev(X, torch.bfloat16, 8, float("nan"))
    Td = _dev(T, torch.bfloat16 if target == "bf16" else torch.float32, pad)
    o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 900, storage="bf16")
    ctx = binding.Context()
    for flags in (0, binding.SHARED_FORWARD):
        Wd = _dev(W, torch.bfloat16, 8, float("nan"))
        out = torch.zeros(4, dtype=torch.float64, device="cuda")
        ctx.step(_large(binding.make_layer(Wd, Xd, r)), Wd, Xd, binding.make_loss(Td), 1, EPS, LR, 900, flags, out)
        ctx.check()
        got = out.cpu().numpy()
        assert abs(got[0] - o["L0"]) < 5e-6 * o["L0"], (flags, got, o["L0"])
        assert abs(got[1] - o["Lp"]) < 5e-6 * o["Lp"], (flags, got, o["Lp"])
        assert abs(got[3] - o["g"]) < 2e-2 * abs(o["g"]) + 1e-7 * o["L0"] / EPS, (flags, got[3], o["g"])


@pytest.mark.parametrize("n,d_out,d_in,r,pad", SHAPES)
def test_stored_outputs_and_cross_entropy(n, d_out, d_in, r, pad):
    ctx = binding.Context()
    W, X, _ = synth.single_layer_problem(7, n, d_in, d_out, kind="rmsnorm", storage="bf16")
    Wd, Xd = _dev(W, torch.bfloat16, 8, float("nan")), _dev(X, torch.bfloat16, 8, float("nan"))
    Y = torch.full((n, d_out + pad), 7.0, device="cuda", dtype=torch.bfloat16)
    B = torch.linalg.qr(torch.randn(d_in, r, device="cuda"))[0].contiguous()
    ctx.perturbed_forward(_large(binding.make_layer(Wd, Xd, r, Y=Y[:, :d_out])), Wd, Xd, B, 5, EPS, Y[:, :d_out], None, None)
    ids = torch.arange(n, dtype=torch.int32, device="cuda") * 37 % d_out
    ids[::5] = -1
    ids[0], ids[-1] = d_out - 1, 0
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.perturbed_forward(_large(binding.make_layer(Wd, Xd, r)), Wd, Xd, B, 5, EPS, None, binding.make_loss(ids, kind=binding.LOSS_CE), out)
    ctx.check()
    Yo = X.astype(np.float64) @ W.astype(np.float64).T
    Yo += EPS * (X.astype(np.float64) @ B.double().cpu().numpy()) @ oagzo.gaussian_factor(5, d_out, r).T
    got = Y.double().cpu().numpy()
    assert np.all(got[:, d_out:] == 7.0)
    err = np.abs(got[:, :d_out] - Yo)
    assert np.all(err <= 2.0 ** -8 * np.abs(Yo) + 1e-5 * np.sqrt(np.mean(Yo ** 2)))
    y, keep = torch.from_numpy(Yo), (ids >= 0).cpu()
    want = (torch.logsumexp(y, 1)[keep] - y[keep, ids.cpu()[keep].long()]).mean().item()
    assert abs(out.item() - want) < 1e-5 * max(1.0, abs(want)), (out.item(), want)


@pytest.mark.parametrize("target", ["bf16", "f32"])
@pytest.mark.parametrize("r", [16, 64])
def test_shared_schedule_sums_every_term_of_the_perturbation(r, target):
    """L+ and L- of the shared schedule against those of three forwards, with an eps that makes the rank-r term most of the
    output: both add the same fp32 terms, in another order and with the target subtracted at another point.  Rounding: 2^-24 of an
    output for each of some twenty additions, independent over 131072 outputs, so some 1e-9 of a loss.  One lo term (2^-9 of the
    perturbation) left out in one of a wave's 64 blocks: 1e-6."""
    n, d_out, d_in = 512, 257, 136
    _, X, T = synth.single_layer_problem(n + r, n, d_in, d_out, kind="rmsnorm", storage="bf16", target_storage=target)
    W, _, _ = synth.single_layer_problem(r, n, d_in, d_out, kind="rmsnorm", storage="bf16")
    Xd, Td = _dev(X, torch.bfloat16, 0), _dev(T, torch.bfloat16 if target == "bf16" else torch.float32, 0)
    ctx = binding.Context()
    got = []
    for flags in (0, binding.SHARED_FORWARD):
        Wd = _dev(W, torch.bfloat16, 0)
        out = torch.zeros(4, dtype=torch.float64, device="cuda")
        ctx.step(_large(binding.make_layer(Wd, Xd, r)), Wd, Xd, binding.make_loss(Td), 1, 1.0, 0.0, 31, flags, out)
        ctx.check()
        got.append(out.cpu().numpy())
    for i in range(3):
        assert abs(got[1][i] - got[0][i]) < 1e-7 * got[0][i], (i, got)
