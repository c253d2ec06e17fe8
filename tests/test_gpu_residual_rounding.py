"""The residual stream takes a projection's result in one rounding, however many ways the projection's K range is split: the parts
are added to each other first.  A stream of +-384 (fp32 step 2^-15) and a down projection whose eight equal stretches of K each
contribute 3/8 of a step: added one by one to the stream they would all vanish, their sum is three steps."""
import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

SHAPE = inputs.ModelShape(1, 256, 2, 2, 64, 8192, 256)
STEP = 2.0 ** -15


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


def _weights(dtype):
    s = SHAPE
    pack = (lambda a: np.asarray(a, dtype=np.float16)) if dtype == "fp16" else (lambda a: inputs.f32_to_bf16_bits(np.asarray(a, dtype=np.float32)))
    zeros = lambda *dims: pack(np.zeros(dims))
    sign = np.where(np.arange(s.d_model) % 2, -1.0, 1.0)
    gate, up, down = np.zeros((s.d_ff, s.d_model)), np.zeros((s.d_ff, s.d_model)), np.zeros((s.d_model, s.d_ff))
    gate[:, 0] = 4.0                                            # silu(4) = 3.928 for every channel: the normalised stream is +-1
    up[:, 0] = 0.375 * 2.0 ** -5 / (4.0 / (1.0 + np.exp(-4.0)))
    down[:, 512::1024] = 2.0 ** -10                             # one channel in the middle of each eighth of K
    return {"embed": pack(np.tile(384.0 * sign, (s.vocab, 1))), "lm_head": pack(np.ones((s.vocab, s.d_model))),
            "g_final": pack(np.ones(s.d_model)), "wq": [zeros(s.q_dim, s.d_model)], "wk": [zeros(s.kv_dim, s.d_model)],
            "wv": [zeros(s.kv_dim, s.d_model)], "wo": [zeros(s.d_model, s.q_dim)], "w_gate": [pack(gate)], "w_up": [pack(up)],
            "w_down": [pack(down)], "g_attn": [pack(np.ones(s.d_model))], "g_ffn": [pack(np.ones(s.d_model))]}


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("M", [4, 8, 9, 16, 17, 33, 64, 80, 81, 200, 1000])
def test_split_projection_rounds_the_stream_once(B, dtype, M):
    import torch
    say(f"residual rounding {dtype} M={M}")
    s, w = SHAPE, _weights(dtype)
    eng = B.VerifyEngine(s, w, 1056, max_prefill_rows=1024)
    tokens = (np.arange(M) % s.vocab).astype(np.int32)
    want = O.verify_forward(O.shape_from(s), w, O.OracleCache(O.shape_from(s), 96), tokens[None, :2])[-1]  # every row is the same
    if M > 80:
        eng.prefill(tokens.tolist(), chunk=M)
        got = eng.root_logits.cpu().numpy()[None]
    else:
        logits = torch.zeros((M, s.vocab), dtype=torch.float32, device="cuda")
        q = torch.full((1, M, s.vocab), 1.0 / s.vocab, device="cuda")
        eng.verify(to_dev(tokens[None]), q, torch.full((1, M + 1), 0.5, device="cuda"), logits_out=logits)
        got = logits.cpu().numpy()
    # every logit is the sum of the 256 entries of the stream over its size: +-384 cancel, three steps per entry remain.  One
    # rounding is half a step per entry; everything else (activations of 16 bits and more, products in fp32) is below 2^-12 of it
    exact = s.d_model * 3 * STEP / 384.0
    assert np.abs(want - exact).max() <= 0.01 * exact
    err = np.abs(got - want).max() / (s.d_model * STEP / 384.0)
    say(f"  error {err:.4f} steps of the stream")
    assert err <= 0.5 * (1 + 2.0 ** -10)
