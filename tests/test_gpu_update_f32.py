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
    """One rounding of the result; r fused products and two roundings of the coefficient, 2^-24 of |c| |G| |B| each; and what G itself may
    be off the oracle's (test_gpu_generator.py: 2.7e-7 of a value and 5.1e-8 of its pair's radius, which is 5.8 at most).  The bits are
    those of agzo_update, and nothing behind d_in is written"""
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
        alone = buf.clone()
        ctx.update(binding.make_layer(alone[:, :d_in], alone[:, :d_in], r), alone[:, :d_in], items[-1][1], 50 + m, 0.25, g)
        Z, G = oagzo.perturbation(B.astype(np.float64), 50 + m, d_out)
        c = 0.25 * (1.0 if g is None else -0.7)
        want, absB = W.astype(np.float64) - c * Z, np.abs(B.T.astype(np.float64))
        inner = abs(c) * ((r + 2) * 2.0 ** -24 * (np.abs(G) @ absB) + (2.7e-7 * np.abs(G) + 5.8 * 5.1e-8) @ absB)
        checks.append((buf, alone, want, (2.0 ** -24 * (np.abs(want) + inner) + inner) * (1 + 1e-5), d_in))
    ctx.update_many(items)
    ctx.check()
    for buf, alone, want, bound, d_in in checks:
        assert (buf[:, d_in:] == 3.0).all()
        assert torch.equal(buf, alone)
        assert (np.abs(buf[:, :d_in].cpu().numpy().astype(np.float64) - want) <= bound).all()


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
