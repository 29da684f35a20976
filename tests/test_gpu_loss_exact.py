"""Squared error whose squares do not fit into fp32: with small whole numbers in X and W every output and every difference from
the target is a whole number below 2^24, so the loss is exact if the squares are taken and added in 64 bits - which all forwards do
for target rows that do not start on 16 bytes and in the columns behind the last full 16.  (Elsewhere four squares are added in
fp32, exact too as long as they stay below 2^24.)  Only the final scaling rounds."""
import numpy as np
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, binding.SHARED_FORWARD])
@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("n,d_out,pad,big_from", [(257, 256, 1, 0), (300, 272, 4, 0), (256, 259, 6, 0), (256, 259, 5, 256), (384, 264, 0, 256), (259, 520, 8, 512)])
def test_loss(n, d_out, pad, big_from, large, flags):
    """pad: rows of the target are that much longer (and so off 16 bytes, unless a multiple of 8); big_from: the first column whose
    difference is large"""
    d_in = 136
    rng = np.random.default_rng(n + d_out)
    X, W = rng.integers(-8, 9, (n, d_in)), rng.integers(-8, 9, (d_out, d_in))
    Y = X @ W.T
    T = Y + rng.integers(-7, 8, Y.shape)
    T[:, big_from:] = Y[:, big_from:] - 4097 - rng.integers(0, 4, Y[:, big_from:].shape)
    Td = torch.zeros(n, d_out + pad, device="cuda")
    Td[:, :d_out] = torch.from_numpy(T).cuda().float()
    Xd, Wd = torch.from_numpy(X).cuda().bfloat16(), torch.from_numpy(W).cuda().bfloat16()
    ctx, out = binding.Context(), torch.zeros(4, dtype=torch.float64, device="cuda")
    L = binding.make_layer(Wd, Xd, 4)
    if large:
        L.tiling = binding.TILING_LARGE
    ctx.step(L, Wd, Xd, binding.make_loss(Td[:, :d_out]), 1, 1e-3, 0.0, 3, flags, out)
    ctx.check()
    want = float(((Y - T).astype(np.int64) ** 2).sum()) / (n * d_out)
    assert abs(out[0].item() - want) < 4e-16 * want, (out[0].item(), want)
