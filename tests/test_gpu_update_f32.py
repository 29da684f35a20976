"""The fp32 sweep of several matrices in one launch: tiles of 32 x 256 that hang over either edge, ranks that are not whole runs of
four, rows that are not aligned, more matrices than a launch takes."""
import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from launches import kernels
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu

# d_out, d_in, row stride, r (the last three: aligned rows that end inside a run of four)
SHAPES = [(1, 1, 1, 1), (31, 4, 8, 4), (32, 256, 256, 16), (33, 260, 260, 3), (65, 255, 256, 2), (64, 513, 513, 17), (7, 1028, 1032, 64), (300, 131, 131, 5),
          (40, 254, 256, 1), (33, 515, 520, 2), (5, 1021, 1024, 33)]


@pytest.mark.parametrize("copies", [1, 3])
def test_sweeps_of_one_call(copies):
    """One rounding of W, and r products and the coefficient in fp32: (r + 3) 2^-24 of |c| |G| |B| on top of it"""
    ctx = binding.Context()
    rng = np.random.default_rng(copies)
    items, checks = [], []
    for m, (d_out, d_in, ld, r) in enumerate(SHAPES * copies):
        buf = torch.full((d_out, ld), 3.0, device="cuda")
        W = rng.standard_normal((d_out, d_in)).astype(np.float32)
        buf[:, :d_in] = torch.from_numpy(W).cuda()
        B = rng.standard_normal((d_in, r)).astype(np.float32)
        g = None if m % 3 == 0 else torch.tensor([-0.7], dtype=torch.float64, device="cuda")
        items.append((buf[:, :d_in], torch.from_numpy(B).cuda(), 50 + m, 0.25, g))
        Z, G = oagzo.perturbation(B.astype(np.float64), 50 + m, d_out)
        c = 0.25 * (1.0 if g is None else -0.7)
        bound = 2.0 ** -24 * np.abs(W.astype(np.float64) - c * Z) + (r + 3) * 2.0 ** -23 * abs(c) * (np.abs(G) @ np.abs(B.T))
        checks.append((buf, W.astype(np.float64) - c * Z, bound, d_in))
    ctx.update_many(items)
    ctx.check()
    for buf, want, bound, d_in in checks:
        assert (buf[:, d_in:] == 3.0).all()
        # G itself comes from fp32 logarithms and angles: 2^-20 of a value
        assert (np.abs(buf[:, :d_in].cpu().numpy().astype(np.float64) - want) <= bound * 8 + 1e-30).all()


def test_rows_of_every_kind_share_a_launch():
    """aligned rows of whole runs of four, aligned rows that end inside one, and others"""
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    items = [(torch.zeros(d_out, ld, device="cuda")[:, :d_in], torch.zeros(d_in, r, device="cuda"), 5, 0.1, None) for d_out, d_in, ld, r in SHAPES]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx.update_many(items)
        stream.synchronize()
    names, _ = kernels(stream, lambda: ctx.update_many(items))
    assert len(names) == 1 and "update_f32_kernel" in names[0], names
    ctx.close()
