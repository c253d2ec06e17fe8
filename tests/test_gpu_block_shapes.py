"""The many-row projection kernel in every block shape its launch can pick (row tiles and bands per wave), at sizes where
that shape is the one picked: ragged rows and bands, an odd number of K steps, and the fused epilogues through whole layers."""
import dataclasses

import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


# (bands of 16 columns, rows): picks (4,12) (4,10) (4,8) (4,6) (4,5) (4,4) (4,3) (4,2), (3,12) .. (3,2), (2,8) .. (2,2)
SHAPES = [(1281, 393), (1225, 393), (1281, 289), (851, 289), (1025, 198), (851, 198), (513, 198), (385, 198),
          (1361, 289), (1025, 289), (1021, 263), (1361, 133), (1025, 133), (769, 133), (1025, 81), (513, 81),
          (1281, 133), (513, 289), (513, 133), (513, 107), (1, 81)]


@pytest.mark.parametrize("bands,rows", SHAPES)
def test_block_gemm_in_every_shape(B, bands, rows):
    import torch
    N, K = 16 * bands - 3, 96
    say(f"block gemm bands={bands} rows={rows}")
    g = np.random.default_rng(bands + rows)
    a = g.normal(0, 1, (rows, K)).astype(np.float32)
    hi = inputs.f32_to_bf16_bits(a)
    lo = inputs.f32_to_bf16_bits((a.astype(np.float64) - O.bf16_bits_to_f64(hi)).astype(np.float32))
    w = inputs.f32_to_bf16_bits(g.normal(0, 0.02, (N, K)).astype(np.float32))
    y = B.block_gemm(to_dev(hi.view(np.int16)), to_dev(lo.view(np.int16)), to_dev(w.view(np.int16)))
    torch.cuda.synchronize()
    ref = (O.bf16_bits_to_f64(hi) + O.bf16_bits_to_f64(lo)) @ O.bf16_bits_to_f64(w).T
    # 2K = 192 products added in fp32: at most 192 roundings of 2^-24 of a running sum no larger than sum |x w|
    bound = 192 * 2.0 ** -24 * (np.abs(O.bf16_bits_to_f64(hi)) @ np.abs(O.bf16_bits_to_f64(w)).T) + 1e-7
    assert (np.abs(y.cpu().numpy() - ref) <= bound).all()


# one layer with rotary, cache, SwiGLU and residual epilogues: the rows of a chunk through the block kernels against the same rows
# in chunks of 48 through the weight-streaming kernels, which the oracle pins elsewhere
@pytest.mark.parametrize("m", [81, 107, 133, 198, 263, 289, 333, 393, 522, 700, 1000])
@pytest.mark.parametrize("shape", ["WIDE1", "WIDE7"])
def test_chunk_of_any_size_matches_small_chunks(B, m, shape):
    import torch
    say(f"prefill {shape} m={m}")
    s = dataclasses.replace(getattr(inputs, shape), n_layers=1)
    key = shape
    if key not in _WEIGHTS:
        _WEIGHTS.clear()
        _WEIGHTS[key] = B.DeviceWeights(s, inputs.make_weights(s, seed=3))
    ids = np.random.default_rng(m).integers(0, s.vocab, m).tolist()
    out = []
    for chunk in (m, 48):
        eng = B.VerifyEngine(s, None, 1056, weights=_WEIGHTS[key], max_prefill_rows=m)
        eng.prefill(ids, chunk=chunk)
        torch.cuda.synchronize()
        assert int(eng.status.cpu()[0]) == 0 and int(eng.prefix_len.cpu()[0]) == m
        out.append((eng.root_logits.cpu().double(), eng.k.view(torch.bfloat16).cpu().double(), eng.vT.view(torch.bfloat16).cpu().double()))
    (la, ka, va), (lb, kb, vb) = out
    # activations carry 16 mantissa bits (2^-17 per rounding) through a handful of steps: 1e-4 of the logits' size; and up to
    # one in a hundred cached values rounds the other way (below), by 2^-8 of itself: sqrt(0.01) * 2^-8 = 4e-4 of what attention adds
    assert (la - lb).norm() <= 5e-4 * lb.norm()
    for a, b in ((ka, kb), (va, vb)):  # cached values may round the other way: one bf16 step (2^-8), and only a few of them
        assert ((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-3).all()
        assert (a != b).double().mean() < 0.01


_WEIGHTS = {}
