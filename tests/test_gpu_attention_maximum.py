"""The online softmax's running maximum, its exchange between lane groups and the rescaling of what has been added up: prefixes whose
scores climb, fall and jump from one block of 32 keys to the next, in every attention launch shape.  Whole steps against the oracle."""
import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say
from tests.test_gpu_parity import _check_step

pytestmark = pytest.mark.gpu

G64, H128 = inputs.ModelShape(1, 512, 8, 2, 64, 512, 1000), inputs.ModelShape(1, 512, 3, 3, 128, 512, 1000)


def _key_scales(pattern, P):
    """One factor per slot; a key scaled by 30 scores up to about 2^60 above or below the mean."""
    if pattern == "climb":
        return np.geomspace(0.05, 30.0, P)
    if pattern == "fall":
        return np.geomspace(30.0, 0.05, P)
    return np.random.default_rng(P).choice([0.1, 1.0, 4.0, 30.0], (P + 31) // 32).repeat(32)[:P]


# query tiles (rows x group / 16) and contexts: one and two tiles, teams of two, four and five waves and one team of eight
@pytest.mark.parametrize("pattern", ["climb", "fall", "jump"])
@pytest.mark.parametrize("shape,P,n,k,root", [(G64, 1500, 1, 4, -1), (H128, 1500, 1, 8, -1), (H128, 1500, 2, 8, -1), (G64, 500, 1, 8, -1), (H128, 500, 2, 16, -1),
                                              (H128, 1500, 2, 16, -1), (G64, 1500, 1, 12, 3), (H128, 1500, 4, 12, 3), (H128, 2200, 4, 16, 5),
                                              (G64, 900, 3, 8, -1), (G64, 900, 4, 16, 5)])
def test_scores_that_move_between_blocks(shape, P, n, k, root, pattern):
    from paper_2503_00784_amd import binding as B
    say(f"{pattern} heads {shape.n_q_heads}/{shape.n_kv_heads} x {shape.head_dim} P={P} n={n} k={k} root={root}")
    max_seq = (P + 96 + 31) // 32 * 32
    w = inputs.make_weights(shape, seed=P, threads=8)
    kb, vb, rl = inputs.make_synthetic_cache(shape, P, max_seq, seed=P)
    scaled = O.bf16_bits_to_f64(kb)
    scaled[:, :, :P] *= _key_scales(pattern, P)[:, None]
    kb = (np.ascontiguousarray(scaled.astype(np.float32)).view(np.uint32) >> 16).astype(np.uint16)
    eng = B.VerifyEngine(shape, w, max_seq)
    eng.load_cache(kb, vb, P, rl)
    oshape = O.shape_from(shape)
    _check_step(B, shape, w, oshape, eng, O.OracleCache.from_bits(oshape, kb, vb, P, rl), n, k, seed=n, mode=0, root_token=root)
