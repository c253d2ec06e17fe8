"""Attention of a prompt chunk in every launch shape (two teams of four and of five waves, one team of eight; one chunk of keys and
more), at sizes where the launch rule, restated here, picks that shape.  Two layers, so that every row's
attention shows in the second layer's cache: the chunk against the same rows in chunks of 48, which take the kernels of a verify step
that the oracle pins elsewhere."""
import numpy as np
import pytest

from paper_2503_00784_amd import inputs
from tests.gpu_util import say


def picked(D, Hkv, group, M, P, max_chunks=8):
    NB, MQ, best = (P + M + 31) // 32, M * group, None
    for nwv, ksplit, stage in ((8, 2, 1.02), (10, 2, 1.27), (8, 1, 1.06)):
        rows = nwv // ksplit * 16
        groups = -(-MQ // rows)
        seen = lambda z: min(NB, (P + (min(MQ, (z + 1) * rows) - 1) // group) // 32 + 1)
        for t in range(1, max_chunks + 1):
            bl = max(2, -(-NB // t))
            n = -(-NB // bl)
            cost = Hkv * groups * (6 * n + stage * 0.5 * (seen(0) + seen(groups - 1)) / ksplit) / 256
            for r in range(-(-Hkv * groups * n // 256)):
                cost = max(cost, (r + 1) * (6 + stage * -(-min(bl, seen(groups - 1 - r * 256 // (n * Hkv))) // ksplit)))
            cost *= 0.68 if D == 64 else 1.0
            cost += 4 + 1.5e-6 * n * MQ * Hkv * D if n > 1 else 0
            if best is None or cost < best[0]:
                best = (cost, (nwv, ksplit, t))
    return best[1]


# (head width, KV heads, group, rows, prefix)
CASES = [(64, 2, 1, 81, 0), (128, 8, 4, 97, 33), (64, 4, 4, 500, 700), (128, 1, 8, 257, 700), (64, 8, 8, 257, 0), (128, 8, 8, 257, 5),
         (64, 8, 4, 97, 1500), (128, 8, 4, 97, 1500), (128, 4, 4, 257, 1500), (64, 16, 8, 200, 0), (64, 16, 8, 333, 100), (128, 16, 8, 200, 31)]


def test_the_sizes_reach_every_shape():
    shapes = {(D, *picked(D, *c)[:2], picked(D, *c)[2] > 1) for D, *c in CASES}
    assert {(D, 8, 2, many) for D in (64, 128) for many in (False, True)} <= shapes
    assert {(D, 10, 2, many) for D in (64, 128) for many in (False, True)} <= shapes
    assert {(64, 8, 1, False), (128, 8, 1, False)} <= shapes


@pytest.mark.gpu
@pytest.mark.parametrize("D,Hkv,group,M,P", CASES)
def test_prompt_attention_in_every_shape(D, Hkv, group, M, P):
    import torch
    from paper_2503_00784_amd import binding as B
    say(f"prompt attention D={D} heads={Hkv}x{group} M={M} P={P}: {picked(D, Hkv, group, M, P)}")
    s = inputs.ModelShape(2, 256, Hkv * group, Hkv, D, 512, 300)
    weights = B.DeviceWeights(s, inputs.make_weights(s, seed=M, threads=8))
    max_seq = (P + M + 31) // 32 * 32
    kb, vb, root = inputs.make_synthetic_cache(s, max(P, 1), max_seq, seed=P + 1)
    ids = np.random.default_rng(M).integers(0, s.vocab, M).tolist()
    out = []
    for chunk in (M, 48):
        eng = B.VerifyEngine(s, None, max_seq, weights=weights, max_prefill_rows=M)
        eng.load_cache(kb, vb, P, root)
        eng.prefill(ids, chunk=chunk)
        torch.cuda.synchronize()
        assert int(eng.status.cpu()[0]) == 0 and int(eng.prefix_len.cpu()[0]) == P + M
        out.append((eng.root_logits.cpu().double(), eng.k.view(torch.bfloat16).cpu().double(), eng.vT.view(torch.bfloat16).cpu().double()))
    (la, ka, va), (lb, kb2, vb2) = out
    # The first layer's cached rows come before any attention and may round the other way where a product's sum differs in its last
    # bits; attention's weights and outputs carry 16 bits and more, so the second layer's rows differ by a few 2^-16 of their size
    # before they are rounded, a bf16 step (2^-8, twice that across a power of two) where that moves them, and few do.
    assert (la - lb).norm() <= 1e-3 * lb.norm()
    for a, b in ((ka, kb2), (va, vb2)):
        assert ((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-3).all()
        assert (a[0] != b[0]).double().mean() < 0.01 and (a[1] != b[1]).double().mean() < 0.05
