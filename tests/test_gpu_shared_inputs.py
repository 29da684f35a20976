"""Layers of a call that read the same activations share the loads of them in the extraction's products: two to five of them (four share at most),
beside layers of their own, other ranks, token counts and widths that no tile divides, and with too few workgroups for it.  Every basis has the
bits of a call of its own, every step those of one in a single stream."""
import pytest
import torch

from launches import kernels
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, binding.INIT_FEATURE])
@pytest.mark.parametrize("shared,sets", [("", [(300, 256, (4, 4)), (129, 1000, (16, 5, 9)), (77, 520, (2,))]),
                                         ("xtt xq", [(5001, 1000, (16, 5, 9)), (4000, 520, (2,)), (4001, 2056, (3, 4))]),
                                         ("xtt xq", [(3001, 2056, (8, 8, 8, 8, 8)), (64, 64, (16, 16)), (1000, 1024, (3,))]),
                                         ("xtt xq", [(8000, 4168, (16,)), (16200, 4168, (1, 16, 7, 2))]),
                                         ("xtt xq", [(8200, 2640, (1, 1)), (9000, 1544, (1, 1, 1))]),
                                         ("xtt", [(3000, 3640, (1, 1)), (2500, 1544, (1, 1, 1))])])
def test_same_bits_as_alone(shared, sets, flags):
    g = torch.Generator(device="cuda").manual_seed(len(sets))
    stream = torch.cuda.Stream()
    ctx, items = binding.Context(stream), []
    for n, d, ranks in sets:
        x = torch.randn(n, d + 16, device="cuda", generator=g).bfloat16()[:, 8:d + 8]
        w = torch.empty(16, d, device="cuda", dtype=torch.bfloat16)
        items += [(binding.make_layer(w, x, r), x, 7 * len(items) + r, None, torch.full((d, r), 9.0, device="cuda")) for r in ranks]
    order = torch.randperm(len(items), generator=torch.Generator().manual_seed(3)).tolist()
    items = [items[i] for i in order]
    torch.cuda.synchronize()
    ctx.basis_many(items, 2, flags)
    ctx.check()
    got = [b.clone() for *_, b in items]
    names, _ = kernels(stream, lambda: ctx.basis_many(items, 2, flags))
    for kind in ("xtt", "xq"):
        assert any(kind + "_group_kernel" in s for s in names) == (kind in shared.split()), names
    for i, ((layer, x, seed, _, b), want) in enumerate(zip(items, got)):
        one = torch.full_like(b, 5.0)
        torch.cuda.synchronize()
        ctx.basis(layer, x, 2, seed, None, flags, one)
        ctx.check()
        assert torch.equal(one, want), (i, x.shape, layer.r)


@pytest.mark.parametrize("f32_target", [False, True])
def test_steps(f32_target):
    """Beside forwards on compute units of their own, and (an fp32 target) on half of every one"""
    n, r = 2900, 12
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream)
    xs = [synth.device_powerlaw_x(5, n, 1024), synth.device_powerlaw_x(6, n, 2048)]
    layers = []
    for i, (x, d_out) in enumerate([(xs[0], 2048), (xs[0], 1024), (xs[1], 1024), (xs[0], 1024), (xs[1], 2560)]):
        w, t = synth.device_weights_and_target(20 + i, x, d_out)
        layers.append((w, x, t.float() if f32_target and i == 1 else t))
    w0 = [w.clone() for w, _, _ in layers]
    out = torch.zeros(len(layers), 4, dtype=torch.float64, device="cuda")
    got = []
    for mask in (0, 1 << binding.PROF_FILL):
        for (w, _, _), s in zip(layers, w0):
            w.copy_(s)
        torch.cuda.synchronize()
        ctx.profile_enable(mask)
        ctx.step_many([(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 50 + i, out[i], None) for i, (w, x, t) in enumerate(layers)], 2, 1e-3, 1e-3, 0)
        ctx.check()
        got.append([out.clone()] + [w.clone() for w, _, _ in layers])
    assert all(torch.equal(a, b) for a, b in zip(*got)) and not torch.equal(got[0][1], w0[0])
