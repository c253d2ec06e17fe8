"""Attention of up to sixteen (row, query head) pairs per kv head: both sides of every line between the kernel without a loop and the staged
kernel in chunks.  Whole steps against the oracle."""
import pytest

from paper_2503_00784_amd import inputs
from tests.gpu_util import say
from tests.test_gpu_parity import _check_step, _engine_and_oracle

pytestmark = pytest.mark.gpu


# keys of the pass (prefix and own rows); heads of 128 on 3, 65, 96 and 97 kv heads, heads of 64 with and without groups
@pytest.mark.parametrize("heads,kv,D,keys", [(3, 3, 128, 640), (3, 3, 128, 641), (3, 3, 128, 906), (3, 3, 128, 1024), (3, 3, 128, 1025), (12, 3, 128, 700),
                                             (65, 65, 128, 768), (65, 65, 128, 769), (97, 97, 128, 800), (97, 97, 128, 1024), (97, 97, 128, 1025),
                                             (8, 2, 64, 768), (8, 2, 64, 800), (5, 5, 64, 1000), (8, 2, 64, 1024), (8, 2, 64, 1025)])
@pytest.mark.parametrize("k,root", [(4, -1), (3, 5)])
def test_both_sides_of_the_lines(heads, kv, D, keys, k, root):
    from paper_2503_00784_amd import binding as B
    s = inputs.ModelShape(1, 256, heads, kv, D, 512, 1000)
    P = keys - k - (root >= 0)
    say(f"heads {heads}/{kv} x {D} keys={keys} rows={k + (root >= 0)}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, P, (keys + 31) // 32 * 32, seed=keys, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, 1, k, seed=k, mode=0, root_token=root)


# The merge of chunks, eight rows of a head in one workgroup (129 and 160 such groups) or in eight (126 and fewer), rows that do not fill the last
@pytest.mark.parametrize("heads,kv,D,P,n,k,root", [(43, 43, 128, 1100, 2, 8, 3), (42, 42, 128, 1100, 2, 8, 3), (32, 8, 64, 1400, 3, 11, -1), (12, 4, 128, 1400, 1, 9, -1),
                                                   (6, 2, 64, 6000, 1, 5, -1)])
def test_merge_of_chunks(heads, kv, D, P, n, k, root):
    from paper_2503_00784_amd import binding as B
    s = inputs.ModelShape(1, 256, heads, kv, D, 512, 1000)
    say(f"merge: heads {heads}/{kv} x {D} P={P} rows={n * k + (root >= 0)}")
    w, oshape, eng, cache = _engine_and_oracle(B, s, P, (P + 80 + 31) // 32 * 32, seed=P, synthetic_cache=True)
    _check_step(B, s, w, oshape, eng, cache, n, k, seed=k, mode=0, root_token=root)
