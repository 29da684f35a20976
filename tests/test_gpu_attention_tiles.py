"""The attention core around its tiles: a key more or fewer than 64, queries of the last wave only, head counts that the
four heads of a preparation group do not divide.  Oracle, tolerances and the causality check of test_gpu_decoder.py."""
import pytest
import torch

import test_gpu_decoder
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,H,Hkv", [(2, 63, 1, 1), (1, 65, 6, 3), (1, 97, 2, 2), (1, 321, 5, 1)])
def test_attention_core(n_seq, T, H, Hkv):
    test_gpu_decoder.test_attention_core_matches_oracle(binding.Context(), n_seq, T, H, Hkv)


@pytest.mark.parametrize("at", [40, 104, 160, 201])
def test_values_behind_a_queries_group_do_not_reach_it(at):
    """An infinite value at token `at` stays out of every output before its group of 32 tokens: later keys are no part of those
    sums.  (Inside the group its probability is 0 for the earlier queries, and 0 x inf is NaN.)"""
    T, H = 202, 3
    ctx = binding.Context()
    q, k, v = (torch.randn(T, w * 128, device="cuda").bfloat16() for w in (H, 1, 1))
    want, got, v2 = torch.empty_like(q), torch.empty_like(q), v.clone()
    v2[at] = float("inf")
    ctx.glue_attention(q, k, v, want, 1, T)
    ctx.glue_attention(q, k, v2, got, 1, T)
    ctx.check()
    first = at // 32 * 32
    assert torch.equal(got[:first], want[:first]) and not torch.isfinite(got[at:]).any()
