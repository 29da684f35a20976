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
