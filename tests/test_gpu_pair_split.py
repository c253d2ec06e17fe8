"""An activation's two 16-bit halves belong to each other: the low half is what is left of the value when the stored high half is
taken away.  The LM head is the identity here, so that a logit is one entry of the last norm's operand (times its row's factor),
and attention contributes nothing: every entry must come out to the precision of the pair, none to that of a single half."""
import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

D_MODEL = 1024


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


@pytest.fixture(scope="module", params=["bf16", "fp16"])
def model(request, B):
    s = inputs.ModelShape(1, D_MODEL, 2, 2, 64, 8192, D_MODEL)
    dtype = request.param
    pack = (lambda a: a.astype(np.float16)) if dtype == "fp16" else (lambda a: inputs.f32_to_bf16_bits(a.astype(np.float32)))
    g = np.random.default_rng(17)
    draw = lambda *dims: pack(g.normal(0, 0.02, dims))
    w = {"embed": pack(g.normal(0, 1.0, (s.vocab, s.d_model))), "lm_head": pack(np.eye(s.d_model)),
         "g_final": pack(g.normal(1, 0.1, s.d_model)), "wq": [draw(s.q_dim, s.d_model)], "wk": [draw(s.kv_dim, s.d_model)],
         "wv": [draw(s.kv_dim, s.d_model)], "wo": [pack(np.zeros((s.d_model, s.q_dim)))], "w_gate": [draw(s.d_ff, s.d_model)],
         "w_up": [draw(s.d_ff, s.d_model)], "w_down": [draw(s.d_model, s.d_ff)], "g_attn": [pack(g.normal(1, 0.1, s.d_model))],
         "g_ffn": [pack(g.normal(1, 0.1, s.d_model))]}
    oshape = O.shape_from(s)
    x = O.embed_rows(w, list(range(s.vocab)))  # a row depends on its own token alone
    h = O.rmsnorm(x, O._w(w, "g_ffn", 0), s.rms_eps)
    x = x + (O.silu(h @ O._w(w, "w_gate", 0).T) * (h @ O._w(w, "w_up", 0).T)) @ O._w(w, "w_down", 0).T
    return dtype, s, w, B.DeviceWeights(s, w), O.rmsnorm(x, O._w(w, "g_final"), oshape.rms_eps)


@pytest.mark.parametrize("M", [8, 16, 33, 64, 80, 81, 400])
def test_halves_belong_to_each_other(B, model, M):
    import torch
    dtype, s, w, weights, want_all = model
    say(f"pair split {dtype} M={M}")
    eng = B.VerifyEngine(s, None, 448, weights=weights, max_prefill_rows=max(M, 80))
    worst = 0.0
    for first in range(0, s.vocab - M + 1, M if M <= 80 else 64):  # M = 80: 12 passes, 980 thousand entries
        tokens = np.arange(first, first + M, dtype=np.int32)
        eng.set_prefix_len(0)
        if M > 80:
            eng.prefill(tokens.tolist(), chunk=M)
            got, want = eng.root_logits.cpu().numpy()[None], want_all[first + M - 1:first + M]
        else:
            logits = torch.zeros((M, s.vocab), dtype=torch.float32, device="cuda")
            eng.verify(to_dev(tokens[None]), torch.full((1, M, s.vocab), 1.0 / s.vocab, device="cuda"), torch.full((1, M + 1), 0.5, device="cuda"),
                       logits_out=logits)
            got, want = logits.cpu().numpy(), want_all[first:first + M]
        worst = max(worst, float((np.abs(got - want) / np.maximum(np.abs(want), 0.25)).max()))
    # a pair carries 2 * 8 (bf16) or 2 * 11 (fp16) bits; what it is made from went through one layer of pairs, whose errors add up to
    # a few times 2^-16 (bf16: 8192 products of pairs of 2^-17, a sum of size 2) or to fp32 rounding.  A high half that is not the
    # stored one is off by a whole step of it: 2^-8 and 2^-11 of a value at least.
    say(f"  worst entry {worst:.2e}")
    assert worst <= (2.0 ** -12 if dtype == "bf16" else 2.0 ** -15)
