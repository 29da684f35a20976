"""Token cross-entropy from chunk statistics where the merge can go wrong: a last chunk without a column, fewer chunks than the
merge has lanes, more than it holds in flight, token counts around its groups of sixteen, skipped tokens.

Tolerance: the statistics are fp32 sums of 128 exponentials on fp32 logits (relative error about 128 2^-24 per token, averaged),
the merge is fp64."""
import numpy as np
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu

# tokens, d_out, d_in
SHAPES = [(1, 5, 64), (15, 128, 64), (16, 257, 64), (17, 384, 72), (33, 2049, 128), (300, 16640, 64), (257, 40000, 64), (256, 33024, 128)]


@pytest.mark.parametrize("n,d_out,d_in", SHAPES)
def test_loss_against_fp64(n, d_out, d_in):
    g = torch.Generator().manual_seed(n + d_out)
    x = torch.randn(n, d_in, generator=g).to(torch.bfloat16)
    w = (torch.randn(d_out, d_in, generator=g) * 0.5).to(torch.bfloat16)
    ids = torch.randint(0, d_out, (n,), generator=g, dtype=torch.int32)
    if n > 2:
        ids[::7] = -1
        ids[1] = d_out                                       # no such output: skipped like a negative id
    ctx = binding.Context()
    xd, wd, td = x.cuda(), w.cuda(), ids.cuda()
    out = torch.full((1,), 3.0, dtype=torch.float64, device="cuda")
    for _ in range(2):
        ctx.layer_forward_sketch(binding.make_layer(wd, xd, 1), wd, xd, None, binding.SKETCH_NONE, None, 0, None,
                                 binding.make_loss(td, kind=binding.LOSS_CE), out)
    ctx.check()
    y = x.double() @ w.double().T
    keep = (ids >= 0) & (ids < d_out)
    want = (torch.logsumexp(y[keep], 1) - y[keep, ids[keep].long()]).mean().item()
    assert abs(out.item() - want) < 1e-5 * max(1.0, abs(want)), (out.item(), want)
