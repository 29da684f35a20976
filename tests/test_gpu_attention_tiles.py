"""The attention core around its tiles: a key more or fewer than 64, queries of the last wave only, head counts that the
four heads of a preparation group do not divide.  Oracle, tolerances and the causality check of test_gpu_decoder.py."""
import pytest

import test_gpu_decoder
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,H,Hkv", [(2, 63, 1, 1), (1, 65, 6, 3), (1, 97, 2, 2), (1, 321, 5, 1)])
def test_attention_core(n_seq, T, H, Hkv):
    test_gpu_decoder.test_attention_core_matches_oracle(binding.Context(), n_seq, T, H, Hkv)
