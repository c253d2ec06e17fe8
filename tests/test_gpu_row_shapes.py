"""Launch shapes that depend on the number of rows: the LM head of a large vocabulary, the K-split down projection of nine to sixteen rows.  Whole steps against the oracle."""
import dataclasses

import pytest

from paper_2503_00784_amd import inputs
from tests.gpu_util import say
from tests.test_gpu_parity import _check_step, _engine_and_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


# 4008 tiles of 32 entries and a ragged last workgroup (100003 entries: 3126 tiles)
@pytest.mark.parametrize("vocab,n,k", [(128256, 1, 9), (100003, 1, 20), (128256, 3, 13), (100003, 4, 16), (128256, 5, 16)])
def test_lm_head_of_a_large_vocabulary(B, vocab, n, k):
    s = dataclasses.replace(inputs.MID, n_layers=1, vocab=vocab)
    say(f"LM head vocab={vocab} n={n} k={k}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, 40, 160, seed=n, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=-1)


# d_ff on both sides of the rule, and K ranges that the eight splits do not divide
@pytest.mark.parametrize("d_ff", [8160, 8192, 8224, 11040])
@pytest.mark.parametrize("k,root", [(8, -1), (8, 3), (12, -1), (16, -1), (16, 3)])
def test_down_projection_of_nine_to_sixteen_rows(B, d_ff, k, root):
    s = dataclasses.replace(inputs.MID, n_layers=2, d_ff=d_ff)
    say(f"down projection d_ff={d_ff} k={k} root={root}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, 40, 96, seed=k, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, 1, k, seed=k, mode=0, root_token=root)
