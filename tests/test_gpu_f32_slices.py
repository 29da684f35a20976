"""fp32 forwards in 64 x 64 tiles around the pairs of whole slices that their loop takes: no whole slice to a few, an odd one left over, an end that
is no whole slice, rows of wider matrices.  fp64 sums: the loss to 1e-12 of it (2^-53 d_in products, their order)."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in", [4, 32, 36, 64, 96, 100, 128, 160, 164, 192, 102, 161])
def test_loss(d_in):
    g = torch.Generator(device="cuda").manual_seed(d_in)
    n, d_out = 1030, 1025          # 17 x 17 tiles, the last of both directions ragged
    x, w = (torch.randn(rows, d_in + 8, device="cuda", generator=g)[:, 4:d_in + 4] for rows in (n, d_out))
    t = torch.randn(n, d_out, device="cuda", generator=g)
    ctx, out = binding.Context(), torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.layer_forward_sketch(binding.make_layer(w, x, 1), w, x, None, binding.SKETCH_NONE, None, 0, None, binding.make_loss(t), out)
    ctx.check()
    want = ((x.double() @ w.double().T - t.double()) ** 2).mean().item()
    assert abs(out.item() - want) < 1e-12 * want
