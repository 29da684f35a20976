"""The attention core on rows of wider tensors: whole and partial tiles of keys, the same bits as from contiguous ones."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,H,Hkv", [(3, 64, 2, 1), (2, 150, 6, 3), (1, 17, 1, 1)])
def test_strided_rows(n_seq, T, H, Hkv):
    g = torch.Generator(device="cuda").manual_seed(T)
    n, ctx = n_seq * T, binding.Context()
    q, k, v = (torch.randn(n, w * 128, device="cuda", generator=g).bfloat16() for w in (H, Hkv, Hkv))

    def wide(x, before, behind):      # the same values in rows with NaN on either side
        buf = torch.full((n, before + x.shape[1] + behind), float("nan"), device="cuda", dtype=torch.bfloat16)
        return buf[:, before:before + x.shape[1]].copy_(x)
    want, got = torch.empty_like(q), wide(torch.zeros_like(q), 24, 8)
    ctx.glue_attention(q, k, v, want, n_seq, T)
    ctx.glue_attention(wide(q, 8, 0), wide(k, 0, 16), wide(v, 40, 8), got, n_seq, T)
    ctx.check()
    assert torch.isfinite(want).all() and torch.equal(got, want)
    assert torch.isnan(got._base[:, :24]).all() and torch.isnan(got._base[:, 24 + q.shape[1]:]).all()
