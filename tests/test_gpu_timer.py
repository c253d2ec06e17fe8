"""The per-kernel timer counts every launch it times once and nothing else: whole steps on both sides of the vocabulary sizes
where the sampling launches change."""
import dataclasses

import numpy as np
import pytest

from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    return binding


def _engine(B, vocab):
    s = dataclasses.replace(inputs.MID, n_layers=1, vocab=vocab)
    eng = B.VerifyEngine(s, inputs.make_weights(s, seed=1, threads=4), 96)
    eng.prefill(inputs.make_prefix_ids(s, 20, seed=1).tolist())
    return s, eng


# sampling launches of one step: (vocabulary, rule, top_p) -> independent sequences below 8192 entries and the sequential rule below
# 12288 are one kernel; above, row statistics + sums + search, and row statistics + a launch per sequence (two here) + search; the
# nucleus is one launch more below 8192 entries, two above
@pytest.mark.parametrize("vocab,rule,top_p,launches", [
    (4099, "longest", 0.0, 1), (4099, "paper", 0.0, 1), (4099, "deferred", 0.0, 1),
    (4099, "longest", 0.9, 2), (4099, "paper", 0.9, 2), (4099, "deferred", 0.9, 2),
    (8192, "longest", 0.0, 3), (8192, "paper", 0.0, 1), (8192, "deferred", 0.9, 3),
    (12288, "longest", 0.9, 5), (12288, "paper", 0.0, 4), (12288, "deferred", 0.0, 4), (12288, "paper", 0.9, 6)])
def test_timer_counts_the_launches_of_a_step(B, vocab, rule, top_p, launches):
    import torch
    say(f"timer vocab={vocab} {rule} top_p={top_p}")
    s, eng = _engine(B, vocab)
    n, k = 2, 3
    q, toks, u = (to_dev(a) for a in inputs.make_draft(vocab, n, k, seed=2))
    torch.cuda.synchronize()
    B.profile_enable(True)
    try:
        if rule == "deferred":
            eng.verify_deferred(toks[0].contiguous(), q[0].contiguous(), u[0].contiguous(), toks[:, 0].contiguous(),
                                q[:, 0].contiguous(), u[:, 0].contiguous(), top_p=top_p)
        else:
            eng.verify(toks, q, u, select_mode=1 if rule == "paper" else 0, top_p=top_p)
        assert B.profile_dropped() == 0
        prof = B.profile_read()
    finally:
        B.profile_enable(False)
    count = {c: p["launches"] for c, p in prof.items()}
    assert count["sample"] == launches
    assert count["commit"] == (0 if rule == "deferred" else 1)
    for c in ("setup", "qkv_rope", "attn", "o_proj", "gate_up_swiglu", "down_proj", "lm_head"):
        assert count[c] == 1, c
    for c, p in prof.items():
        assert (p["ms"] > 0) == (p["launches"] > 0), (c, p)
        assert np.isfinite(p["ms"]) and p["ms"] < 1e3
    assert eng.results(n)["status"] == 0
