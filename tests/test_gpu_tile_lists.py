"""Squared errors of several layers whose 256 x 256 tiles share a launch, workgroups walking lists that go through all of them: every
loss, scalar and weight has the bits of launches of their own (timing a kernel class makes every forward one), also of layers that take
128 x 128 tiles when alone, and the losses agree with fp64.

Tolerance of L0: bf16 products accumulate in fp32 over d_in, a few 1e-6 of a loss of comparable residuals."""
import pytest
import torch

from launches import kernels
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = 1e-3, 1e-3

# tokens, r, (d_in, d_out) per layer, target: layers of 160 tiles and more with ends that no tile divides; d_in that slices do not
# divide; target rows off 16 bytes (fp64 squares), a last half tile that overlaps by no multiple of 16, by one, by all
RAGGED = [(512, 4096), (520, 3600), (2048, 1111), (4096, 1024), (4096, 1040), (3072, 264), (128, 3000)]
# tiles in numbers that neither 8 nor a round of them divides; two problems of one depth
ALIGNED = [(256, 2816), (512, 2560), (1024, 3072), (512, 256)]
# more than two rounds of an XCD's workgroups and a rest that 8 does not divide: 540 tiles (5000 tokens), 525 (5376), beside one of a round
ROUNDS, ROUNDS_ALIGNED = [(128, 6900), (192, 3000), (136, 6900)], [(128, 6400), (256, 3072), (128, 6400)]
# few deep tiles, which layers of 300 tokens take beside the extraction only
DEEP = [(9728, 2560), (8192, 1100), (9600, 2048), (6144, 2056)]


def _strided(a, pad):
    """a in rows that lie `pad` values further apart, NaN between them"""
    buf = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), device="cuda", dtype=a.dtype)
    buf[:, :a.shape[1]] = a
    return buf


def _given(n, shapes, strides, f32_target=None):
    """(x, w, t) per layer, in rows of their own strides where `strides`, and d_in, d_out"""
    got = []
    for i, (d_in, d_out) in enumerate(shapes):
        x = synth.device_powerlaw_x(70 + i, n, d_in)
        w, t = synth.device_weights_and_target(170 + i, x, d_out)
        if i == f32_target:
            t = t.float()
        pads = (8 * (i % 3), 8 * ((i + 1) % 4), (0, 3, 8, 5)[i % 4]) if strides else (0, 0, 0)
        got.append(tuple(_strided(a, pad) for a, pad in zip((x, w, t), pads)) + (d_in, d_out))
    return got


def _items(given, w, out, r, k):
    return [(binding.make_layer(w[i][:, :d_in], x[:, :d_in], r), w[i][:, :d_in], x[:, :d_in], binding.make_loss(t[:, :d_out]), 40 + i + 100 * k, out[k, i], None)
            for i, (x, _, t, d_in, d_out) in enumerate(given)]


def _lists(names):
    return sum("gemm_bf16_aligned_kernelILi0ELb0ELi1E" in name and "ELi16E" in name for name in names)


# lists: launches of them in a step (base forwards beside the extraction; perturbed ones)
@pytest.mark.parametrize("flags", [0, binding.ONE_SIDED])
@pytest.mark.parametrize("n,r,shapes,strides,lists", [(3001, 16, RAGGED, False, 2), (2690, 17, RAGGED, True, 2), (4096, 8, ALIGNED, False, 1), (4096, 8, ALIGNED, True, 1),
                                                      (300, 64, DEEP, True, 1), (5000, 3, ROUNDS, True, 1), (5376, 16, ROUNDS_ALIGNED, False, 1),
                                                      (600, 8, RAGGED[:5] * 4, True, 2)])
def test_same_as_launches_of_their_own(n, r, shapes, strides, lists, flags):
    given = _given(n, shapes, strides)
    got, stream = [], torch.cuda.Stream()
    for mask in (0, 1 << binding.PROF_GEMM):
        ctx = binding.Context(stream=stream)
        ctx.profile_enable(mask)
        w = [g[1].clone() for g in given]
        out = torch.full((2, len(given), 4), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for k in range(2):
                ctx.step_many(_items(given, w, out, r, k), 1, EPS, LR, flags)
            ctx.check()
            stream.synchronize()
        got.append([out] + [a.view(torch.int16) for a in w])
        if mask == 0:
            spare = [a.clone() for a in w]
            names, _ = kernels(stream, lambda: ctx.step_many(_items(given, spare, out.clone(), r, 0), 1, EPS, LR, flags))
            assert _lists(names) >= lists, names
        ctx.close()
    assert torch.isfinite(got[0][0]).all()
    assert all(torch.equal(a, b) for a, b in zip(*got))
    for i, (x, w0, t, d_in, d_out) in enumerate(given):
        y = x[:, :d_in].double() @ w0[:, :d_in].double().T
        want = ((y - t[:, :d_out].double()) ** 2).mean().item()
        assert abs(got[0][0][0, i, 0].item() - want) < 5e-6 * want, i


def test_one_layer_that_lists_do_not_take():
    """base forwards then run beside the extraction as launches of their own, those of both signs in lists but for that layer's"""
    r, stream = 4, torch.cuda.Stream()
    given = _given(1500, [(2560, 4096), (2560, 1024), (4096, 2560), (2560, 3000), (3072, 2560)], True, f32_target=3)
    got = []
    for mask in (0, 1 << binding.PROF_GEMM):
        ctx = binding.Context(stream=stream)
        ctx.profile_enable(mask)
        w = [g[1].clone() for g in given]
        out = torch.full((1, len(given), 4), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ctx.step_many(_items(given, w, out, r, 0), 3, EPS, LR, 0)
            ctx.check()
            stream.synchronize()
        got.append([out] + [a.view(torch.int16) for a in w])
        if mask == 0:
            names, _ = kernels(stream, lambda: ctx.step_many(_items(given, [a.clone() for a in w], out.clone(), r, 0), 3, EPS, LR, 0))
            assert _lists(names) == 1, names
        ctx.close()
    assert torch.isfinite(got[0][0]).all()
    assert all(torch.equal(a, b) for a, b in zip(*got))
