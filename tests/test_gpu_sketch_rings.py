"""The range sketch emitted by the 128 x 128 forward kernel in each of its LDS rings: more tiles than compute units, fewer, and the
shares of d_in that a stored output of few tiles takes (a share sketches its own slices)."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu

# tokens, d_in, d_out, r: 21 x 16 tiles, 2 x 129 (129 workgroups of two tokens' tiles); shares of 8 slices and a last one that d_in
# does not fill, with more and with fewer output tiles than slices in a share; two slices.  (Stored, the former run in 64 x 64 tiles whose waves share
# d_in; past their line:) shares of eight and nine slices, of thirteen and fourteen, of eight and nine for more output tiles than that
SHAPES = [(2600, 200, 2000, 5), (129, 136, 16500, 16), (300, 1100 - 4, 300, 16), (3001, 2056, 264, 13), (140, 1032, 1300, 1), (256, 128, 256, 7),
          (300, 4168, 300, 16), (3001, 2632, 264, 13), (140, 2664, 1300, 1)]


@pytest.mark.parametrize("out", ["y", "mse_bf16", "mse_f32"])
@pytest.mark.parametrize("n,d_in,d_out,r", SHAPES)
def test_fused_range_sketch(n, d_in, d_out, r, out):
    W, X, T = synth.single_layer_problem(n, n, d_in, d_out, kind="rmsnorm", storage="bf16", target_storage="f32")
    Xd = torch.full((n, d_in + 8), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :d_in]
    Xd.copy_(torch.from_numpy(X))
    Wd = torch.from_numpy(W).cuda().bfloat16()
    Td = torch.from_numpy(T).cuda().to(torch.float32 if out == "mse_f32" else torch.bfloat16)
    loss = None if out == "y" else binding.make_loss(Td)
    ctx, got = binding.Context(), []
    for mode in (binding.SKETCH_RANGE, binding.SKETCH_RANGE_FUSED):
        Y = torch.full((n, d_out), 3.0, device="cuda", dtype=torch.bfloat16) if out == "y" else None
        S, f = torch.empty(d_in, r, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        ctx.layer_forward_sketch(binding.make_layer(Wd, Xd, r, Y=Y), Wd, Xd, Y, mode, None, 91, S, loss, f if loss else None)
        ctx.check()
        got.append((Y, f.item(), S.double().cpu().numpy()))
    assert got[0][1] == got[1][1]
    assert out != "y" or torch.equal(got[0][0], got[1][0])
    # fp32 sums of n products: 2^-24 sqrt(n) of the norms at most
    want = oagzo.range_sketch(X.astype(np.float64), r, 91)
    for _, _, S in got:
        assert np.linalg.norm(S - want) < 4e-6 * np.linalg.norm(want)
