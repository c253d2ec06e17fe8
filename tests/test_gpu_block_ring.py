"""The many-row projection kernel in every block shape over a K range several times as long as its ring of stage buffers, so that
every buffer is refilled while others are read; and, from the launch rule restated here, that the sizes reach every shape."""
import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev
from tests.test_gpu_block_shapes import SHAPES

PICKS = [(4, 12), (4, 10), (4, 8), (4, 6), (4, 5), (4, 4), (4, 3), (4, 2), (3, 12), (3, 10), (3, 8), (3, 6), (3, 5), (3, 4), (3, 3),
         (3, 2), (2, 8), (2, 6), (2, 4), (2, 3), (2, 2)]


def picked(bands, rows):
    """The row tiles and bands per wave that the launch chooses: the fewest rounds of 256 workgroups times the time of a K step."""
    mh, best = (rows + 15) // 16, None
    for wm, wn in PICKS:
        wgs = -(-bands // (2 * wn)) * -(-mh // (2 * wm))
        cost = -(-wgs // 256) * (0.18 + wn * (0.006 + 0.0186 * wm))
        if best is None or cost < best[0] - 1e-9:
            best = (cost, (wm, wn))
    return best[1]


def test_the_sizes_reach_every_shape():
    assert len(SHAPES) == 21 and {picked(b, r) for b, r in SHAPES} == set(PICKS)


@pytest.mark.gpu
@pytest.mark.parametrize("bands,rows", SHAPES)
def test_block_gemm_refills_its_ring(bands, rows):
    import torch
    from paper_2503_00784_amd import binding as B
    N, K = 16 * bands - 3, 32 * 13  # 13 K steps, 13 or 7 stages through a ring of three
    say(f"block gemm {picked(bands, rows)} bands={bands} rows={rows} K={K}")
    g = np.random.default_rng(bands * 3 + rows)
    a = g.normal(0, 1, (rows, K)).astype(np.float32)
    hi = inputs.f32_to_bf16_bits(a)
    lo = inputs.f32_to_bf16_bits((a.astype(np.float64) - O.bf16_bits_to_f64(hi)).astype(np.float32))
    w = inputs.f32_to_bf16_bits(g.normal(0, 0.02, (N, K)).astype(np.float32))
    y = B.block_gemm(to_dev(hi.view(np.int16)), to_dev(lo.view(np.int16)), to_dev(w.view(np.int16)))
    torch.cuda.synchronize()
    h, l, wt = O.bf16_bits_to_f64(hi), O.bf16_bits_to_f64(lo), O.bf16_bits_to_f64(w)
    # 2K products added in fp32: at most 2K roundings of 2^-24 of a running sum no larger than sum |x w|
    bound = 2 * K * 2.0 ** -24 * (np.abs(h) @ np.abs(wt).T) + 1e-7
    assert (np.abs(y.cpu().numpy() - (h + l) @ wt.T) <= bound).all()
