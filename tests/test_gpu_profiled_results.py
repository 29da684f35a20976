"""Timing a kernel class changes which launches a call makes (every forward by itself, its operands prepared inside its time), and
must not change a bit of its results."""
import pytest
import torch

from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu

# tokens, d_out, d_in, r: the forward kernels of large, middling and small layers
SHAPES = [(512, 300, 328, 8), (4096, 2560, 192, 16), (100, 72, 64, 1)]


def _problem(n, d_out, d_in):
    W, X, T = synth.single_layer_problem(n, n, d_in, d_out, kind="rmsnorm", storage="bf16")
    return [torch.from_numpy(a).cuda().bfloat16() for a in (W, X, T)]


@pytest.mark.parametrize("flags,launches", [(0, 3), (binding.ONE_SIDED, 2), (binding.SHARED_FORWARD, 1)])
def test_step_many(flags, launches):
    got = []
    for mask in (0, 1 << binding.PROF_GEMM):
        ctx = binding.Context()
        ctx.profile_enable(mask)
        probs = [_problem(*s[:3]) for s in SHAPES]
        out = torch.zeros(len(probs), 4, dtype=torch.float64, device="cuda")
        ctx.step_many([(binding.make_layer(W, X, s[3]), W, X, binding.make_loss(T), 5 + i, out[i], None)
                       for i, ((W, X, T), s) in enumerate(zip(probs, SHAPES))], 1, 1e-3, 1e-2, flags)
        ctx.check()
        assert not mask or ctx.profile_read(binding.PROF_GEMM)[0] == launches * len(SHAPES)
        got.append([out] + [p[0] for p in probs])
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("n,d_out,d_in,r", SHAPES)
def test_perturbed_forward(n, d_out, d_in, r):
    W, X, T = _problem(n, d_out, d_in)
    B = torch.linalg.qr(torch.randn(d_in, r, device="cuda"))[0].contiguous()
    got = []
    for mask in (0, binding.PROF_ALL):
        ctx, out = binding.Context(), torch.zeros(1, dtype=torch.float64, device="cuda")
        ctx.profile_enable(mask)
        Y = torch.empty(n, d_out, device="cuda", dtype=torch.bfloat16)
        ctx.perturbed_forward(binding.make_layer(W, X, r), W, X, B, 5, 1e-3, None, binding.make_loss(T), out)
        ctx.perturbed_forward(binding.make_layer(W, X, r, Y=Y), W, X, B, 5, -1e-3, Y, None, None)
        ctx.check()
        assert not mask or ctx.profile_read(binding.PROF_GEMM)[0] == 2
        got.append((out, Y))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
