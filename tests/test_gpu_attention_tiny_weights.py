"""Softmax weights below the smallest normal 32-bit number, where one and two query tiles per kv head compute them: they are kept, and values
large enough make them visible.  Against the oracle's whole step."""
import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _bf16(x):
    return (np.asarray(x, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _inputs(shape, P, max_seq):
    """Every token's queries and keys are one vector a (1, .., 1), so that a row scores its own key at about 127.7 in powers of two, the prefix
    (zero keys) at 0; a row's own values are zero, those of the prefix in the last block before the drafts of the order of 2^124."""
    a = 2.796875 if shape.head_dim == 128 else 3.328125
    w = inputs.make_weights(shape, seed=P, threads=8)
    w["embed"] = np.full_like(w["embed"], _bf16(0.0625))
    w["g_attn"] = [np.full_like(w["g_attn"][0], _bf16(1.0))]
    w["wv"] = [np.zeros_like(w["wv"][0])]
    w["w_down"] = [np.zeros_like(w["w_down"][0])]
    for name in ("wq", "wk"):
        w[name] = [np.zeros_like(w[name][0])]
        w[name][0][:, 0] = _bf16(a)
    k = np.zeros((1, shape.n_kv_heads, max_seq, shape.head_dim), np.uint16)
    v = np.zeros_like(k)
    channels = 2.0 ** 124 * (1.0 + np.arange(shape.n_kv_heads * shape.head_dim) % 5).reshape(shape.n_kv_heads, 1, shape.head_dim)
    v[0, :, P // 32 * 32:P] = _bf16(channels)
    return w, k, v, np.zeros(shape.vocab, np.float32)


# the kernel without a loop (heads of 64 and 128), one tile of the staged kernel in chunks, two tiles in one chunk
@pytest.mark.parametrize("D,P,k", [(128, 500, 1), (64, 500, 4), (64, 980, 2), (128, 1500, 1), (128, 700, 5), (64, 1500, 8), (128, 300, 20)])
def test_weights_below_the_normal_range(D, P, k):
    import torch

    from paper_2503_00784_amd import binding as B
    shape = inputs.ModelShape(1, 512, 2, 2, D, 512, 1000)
    say(f"heads of {D} P={P} k={k}")
    max_seq = (P + k + 31) // 32 * 32
    w, kb, vb, root = _inputs(shape, P, max_seq)
    eng = B.VerifyEngine(shape, w, max_seq)
    eng.load_cache(kb, vb, P, root)
    oshape = O.shape_from(shape)
    q, toks, u = inputs.make_draft(shape.vocab, 1, k, seed=1)
    logits = torch.empty((k, shape.vocab), dtype=torch.float32, device="cuda")
    eng.verify(to_dev(toks), to_dev(q), to_dev(u), logits_out=logits)
    assert eng.results(1)["status"] == 0
    _, want = O.oracle_verify(oshape, w, O.OracleCache.from_bits(oshape, kb, vb, P, root), toks, q, u)
    err = np.linalg.norm(logits.cpu().numpy() - want, axis=1) / np.linalg.norm(want, axis=1)
    say(f"  relative error of the rows' logits {err.max():.2e}")
    # a weight of 2^-128 has five bits as a bf16 number below the normal range: half of the last is 2^-6; without such weights the
    # attention's part of the residual stream, ten times the rest, is missing
    assert (err < 0.05).all()
