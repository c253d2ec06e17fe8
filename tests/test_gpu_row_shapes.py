"""Launch shapes that depend on the number of rows: attention over five and over seventeen to twenty query tiles per KV head,
the LM head of a large vocabulary, the K-split down projection of nine to sixteen rows.  Whole steps against the oracle."""
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


# heads of 64 in groups of four (tiles = rows * 4 / 16): 16, 17, 18, 20 tiles, a short and a longer prefix
@pytest.mark.parametrize("P", [30, 700])
@pytest.mark.parametrize("n,k,root", [(4, 16, -1), (4, 16, 5), (3, 23, 1), (5, 16, -1)])
def test_attention_beyond_sixteen_tiles(B, P, n, k, root):
    say(f"MID P={P} n={n} k={k} root={root}")
    w, oshape, eng, cache = _engine_and_oracle(B, inputs.MID, P, (P + 96 + 31) // 32 * 32, seed=P, synthetic_cache=True)
    _check_step(B, inputs.MID, w, oshape, eng, cache, n, k, seed=n, mode=0, root_token=root)


# no groups: 65..80 rows are five tiles; 64 blocks of 32 keys is where the two teams of five take over
@pytest.mark.parametrize("shape", ["NARROW64", "NARROW128"])
@pytest.mark.parametrize("P,n,k,root", [(1940, 4, 16, 5), (1968, 5, 16, -1), (1984, 4, 16, 5), (3001, 6, 13, -1)])
def test_attention_of_five_tiles(B, shape, P, n, k, root):
    s = inputs.ModelShape(2, 320, 5, 5, 64, 640, 1000) if shape == "NARROW64" else inputs.ModelShape(1, 384, 3, 3, 128, 512, 1000)
    say(f"{shape} P={P} n={n} k={k} root={root}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, P, (P + 96 + 31) // 32 * 32, seed=P, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=n, mode=0, root_token=root)


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
