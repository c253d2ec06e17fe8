"""The eight-wave form of the weight-streaming kernel behind projections other than the LM head: gate/up beyond 16384 channels and
Q/K/V beyond 2048 bands, with a ragged last workgroup.  Whole steps against the oracle."""
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


# 16416 channels are 1026 tiles, two past a whole workgroup of eight; 9..80 rows are one to five row tiles
@pytest.mark.parametrize("n,k,root", [(1, 9, -1), (3, 7, 4), (4, 10, -1), (5, 12, 4), (5, 16, -1)])
def test_gate_up_of_many_channels(B, n, k, root):
    s = dataclasses.replace(inputs.MID, n_layers=1, d_ff=16416)
    say(f"gate/up d_ff={s.d_ff} n={n} k={k} root={root}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, 40, 128, seed=n, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)


# 171 heads of 64 without groups are 2052 bands, 1026 tiles of two
@pytest.mark.parametrize("n,k,root", [(1, 9, -1), (3, 7, 4), (4, 10, -1), (5, 16, -1)])
def test_qkv_of_many_bands(B, n, k, root):
    s = inputs.ModelShape(1, 256, 171, 171, 64, 512, 1000)
    say(f"Q/K/V heads={s.n_q_heads} n={n} k={k} root={root}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, 33, 128, seed=n, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)
