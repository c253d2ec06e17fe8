"""Operand layout of 17..80 rows whose last row tile holds one to eight rows: that tile holds their lo halves too.  Whole steps against the
oracle at both edges of every tile count, in the launch shapes of a small model (two waves per band group) and of the 7B layer (three
band groups per workgroup, split projections, partial results of Q/K/V), and the layout's map by itself (the library's own,
compiled for the host)."""
import dataclasses

import pytest

from paper_2503_00784_amd import inputs
from tests.gpu_util import say
from tests.launch_rules import rules
from tests.test_gpu_parity import _check_step, _engine_and_oracle


@pytest.mark.parametrize("M", list(range(1, 82)) + [333, 1024])
def test_every_half_has_a_row_of_its_own(M):
    tiles, lo = rules().operand_tiles(M), [rules().lo_row(M, m) for m in range(M)]
    assert len(set(lo) | set(range(M))) == 2 * M and max(lo) < 16 * tiles <= 2 * 16 * ((M + 15) // 16)
    assert tiles == -(-2 * M // 16) or M > 80 or (M - 1) % 16 >= 8  # no tile more than 2 M rows need where the last tile is shared
    if M > 16:  # a lane's hi and lo sums have the same position in their tiles, or are eight rows apart in the last one
        shared = bool(rules().shared_last_tile(M))
        assert all(r - m == 8 if shared and m // 16 == (M - 1) // 16 else (r - m) % 16 == 0 for m, r in enumerate(lo))


ROWS = [(1, 16, 3), (3, 6, -1), (3, 8, -1), (5, 5, -1), (4, 8, -1), (4, 8, 3), (5, 8, -1), (5, 8, 3), (6, 8, 3), (7, 8, -1), (7, 8, 3), (4, 16, 3), (6, 12, -1), (6, 12, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,root", ROWS)
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_small_model_at_the_edges_of_the_tiles(n, k, root, dtype):
    from paper_2503_00784_amd import binding as B
    if dtype == "fp16" and (n * k) % 8:
        pytest.skip("the other element type at half of the edges")
    say(f"MID {dtype} rows={n * k + (root >= 0)}")
    w, oshape, eng, cache = _engine_and_oracle(B, inputs.MID, 60, 160, seed=n, synthetic_cache=True, dtype=dtype)
    _check_step(B, inputs.MID, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,root", [(1, 16, 3), (4, 8, 3), (5, 8, -1), (6, 8, 3), (7, 8, -1), (4, 16, 3), (6, 12, -1)])
def test_layer_of_the_large_model(n, k, root):
    from paper_2503_00784_amd import binding as B
    say(f"WIDE7 rows={n * k + (root >= 0)}")
    w, oshape, eng, cache = _engine_and_oracle(B, inputs.WIDE7, 60, 160, seed=n, synthetic_cache=True)
    _check_step(B, inputs.WIDE7, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


def _step(B, s, n, k, root):
    w, oshape, eng, cache = _engine_and_oracle(B, s, 40, 160, seed=n, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)


# The eight-wave kernel at four and five row tiles, both edges of either: an LM head of 4008 tiles, a gate/up projection of 1026
@pytest.mark.gpu
@pytest.mark.parametrize("vocab,d_ff", [(128256, 512), (1000, 16416)])
@pytest.mark.parametrize("n,k,root", [(6, 8, 3), (7, 8, -1), (4, 16, 3), (6, 12, -1)])
def test_eight_waves(B, vocab, d_ff, n, k, root):
    say(f"vocab={vocab} d_ff={d_ff} rows={n * k + (root >= 0)}")
    _step(B, dataclasses.replace(inputs.MID, n_layers=1, vocab=vocab, d_ff=d_ff), n, k, root)


# Two band groups of two waves each, whose partial sums are added before the halves: gate/up of 258 tiles at every number of row
# tiles, Q/K/V of 384 bands at two and three (beyond that its partial results take another kernel)
@pytest.mark.gpu
@pytest.mark.parametrize("n,k,root", [(1, 16, 3), (3, 8, -1), (4, 8, 3), (5, 8, -1), (6, 8, 3), (7, 8, -1), (4, 16, 3), (6, 12, -1)])
def test_two_groups_of_two_waves(B, n, k, root):
    say(f"Q/K/V of 384 bands, d_ff=4128, rows={n * k + (root >= 0)}")
    _step(B, inputs.ModelShape(1, 256, 64, 16, 64, 4128, 1000), n, k, root)
