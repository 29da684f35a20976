"""Normals of every stream against the oracle's (64 bits, rounded once): the radius of a Box-Muller pair to 1.49e-7 of it and the sine
and cosine to 5.1e-8 (measured over all their arguments), a product's rounding and the oracle's, 2^-24 of the value each."""
import numpy as np
import pytest
import torch

from oracle import philox as ophilox
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tag", [binding.TAG_G, 3])
@pytest.mark.parametrize("rows,cols,seed", [(65536, 32, 1), (3, 8, (1 << 63) + 5), (70001, 4, 9)])
def test_normals(rows, cols, seed, tag):
    dst = torch.empty(rows, cols, device="cuda")
    binding.Context().fill_normal(dst, seed, tag)
    got = dst.cpu().numpy().astype(np.float64)
    want = ophilox.normal(seed, tag, rows, cols).astype(np.float64)
    pair = want.reshape(rows, cols // 2, 2)
    radius = np.repeat(np.sqrt((pair ** 2).sum(axis=2)), 2, axis=1)
    assert np.all(np.abs(got - want) <= np.abs(want) * (1.49e-7 + 2.0 ** -23) * 1.01 + radius * 5.1e-8 * 1.01)
    assert abs(got.mean()) < 6 / np.sqrt(got.size) and abs(got.var() - 1) < 9 / np.sqrt(got.size)


# (sums of what sqrtf(-2 logf(u)) and sincospif gave; the second draw alone has every u of 23 bits among its radii)
@pytest.mark.parametrize("rows,cols,seed,tag,want", [(1 << 22, 32, 1, 0, 0x5d2430bce86e2f8b), (1 << 22, 32, 2, 3, 0x2576f7897db68adc), (70001, 7, 9, 2, 0xc84b907b7ce67e1c)])
def test_bits(rows, cols, seed, tag, want):
    """A seed stands for its perturbations and updates: not one bit of a normal may change.  Every word counts with a weight of its own"""
    dst = torch.empty(rows, cols, device="cuda")
    binding.Context().fill_normal(dst, seed, tag)
    bits, total, step = dst.view(torch.int32).reshape(-1), 0, 1 << 25
    for i in range(0, bits.numel(), step):
        part = bits[i:i + step].to(torch.int64)
        total += (part * (2 * torch.arange(i, i + part.numel(), device="cuda") + 1)).sum().item()
    assert total % (1 << 64) == want
