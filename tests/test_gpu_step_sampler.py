"""The sampler's many-workgroup kernels behind an LM head, where they read row statistics that were merged once (and, in the sequential
rule, lie in the scratch that its last kernel overwrites): whole steps of one layer with vocabularies beyond the one-workgroup
kernels, decisions and tokens against the oracle's sampler on the logits that the step returned."""
import dataclasses

import numpy as np
import pytest

from oracle import duo_oracle as O
from paper_2503_00784_amd import inputs
from tests.gpu_util import say, to_dev
from tests.test_gpu_deferred import _gpu_outcome, _oracle_outcome
from tests.test_gpu_parity import _nucleus_margin

pytestmark = pytest.mark.gpu

P, T = 20, 0.9
_ENGINES = {}


@pytest.fixture(scope="module")
def B():
    from paper_2503_00784_amd import binding
    binding.load()
    yield binding
    _ENGINES.clear()


def _engine(B, V):
    if V not in _ENGINES:
        s = dataclasses.replace(inputs.MID, n_layers=1, vocab=V)
        eng = B.VerifyEngine(s, inputs.make_weights(s, seed=4, threads=8), 96)
        eng.prefill(inputs.make_prefix_ids(s, P, seed=4).tolist())
        _ENGINES[V] = eng
    return _ENGINES[V]


def _step(eng, toks, q, u, mode, root, top_p):
    import torch
    R, (n, k), V = int(root >= 0), toks.shape, eng.shape.vocab
    lg = torch.zeros((R + n * k, V), dtype=torch.float32, device="cuda")
    eng.set_prefix_len(P)
    eng.verify(to_dev(toks), to_dev(q), to_dev(u), temperature=T, select_mode=mode, root_token=root, logits_out=lg, top_p=top_p)
    got = eng.results(n)
    assert got["status"] == 0
    return got, lg.cpu().numpy(), eng.root_logits.cpu().numpy()


def _compare(got, gl, groot, toks, q, u, mode, root, top_p):
    n, k = toks.shape
    ref = O.speculative_verify(gl, groot, toks, q, u, prefix_len=P, temperature=T, select_mode=mode, has_root=root >= 0, top_p=top_p)
    if (top_p and _nucleus_margin(gl, groot, root >= 0, n, k, T, top_p) <= 1e-12) or ref.commit_margin <= 1e-9 or \
            (mode == 0 and min(ref.accept_margins.min(), ref.draw_margins.min()) <= 1e-9):
        return None
    np.testing.assert_array_equal(got["accept_len"], ref.accept_len)
    np.testing.assert_array_equal(got["next_token"], ref.next_token)
    assert (got["selected"], got["commit_len"], got["commit_token"], got["new_prefix_len"], got["device_prefix_len"]) == \
           (ref.selected, ref.commit_len, ref.commit_token, ref.new_prefix_len, ref.new_prefix_len)
    return ref


@pytest.mark.parametrize("V", [8192, 12288, 32000])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("root", [-1, 7])
@pytest.mark.parametrize("top_p", [0.0, 0.9, 0.4])
def test_step_decides_as_the_oracle_does(B, V, mode, root, top_p):
    say(f"step V={V} mode={mode} root={root} top_p={top_p}")
    eng, compared = _engine(B, V), 0
    for n, k, seed in ((1, 4, 1), (3, 4, 2), (5, 3, 3)):
        q, toks, u = inputs.make_draft(V, n, k, seed=seed, easy_rows=inputs.easy_rows_for(n, k))
        got, gl, groot = _step(eng, toks, q, u, mode, root, top_p)
        compared += _compare(got, gl, groot, toks, q, u, mode, root, top_p) is not None
    assert compared >= 2


def _script_candidates(p, tokens, q, u, taken):
    """Candidates 0 .. taken-1 are rejected by p and its residuals, `taken` (if there is one) is accepted: their tokens, draft
    distributions [s][V] and uniforms are set in place."""
    for i in range(len(tokens)):
        tokens[i] = int(np.argmax(np.where(p < 0.25 * q[i], q[i], 0.0)))
        u[i] = 0.999999
    if taken < len(tokens):
        tokens[taken] = int(np.argmin(np.where(p > 0, q[taken] / np.maximum(p, 1e-30), np.inf)))
        q[:taken, tokens[taken]] = 0.0  # the rejected ones take nothing of it away
        u[taken] = 1e-3


AT = {"first": 0, "second": 1, "third": 2, "fifth": 4, "last": 5, "none": 6}  # three launches at 32000 entries, then the last kernel


@pytest.mark.parametrize("V", [32000, 40960])
@pytest.mark.parametrize("at", AT)
@pytest.mark.parametrize("root", [-1, 7])
@pytest.mark.parametrize("top_p", [0.0, 0.9])
def test_sequential_rule_of_a_step_at_every_candidate(B, V, at, root, top_p):
    say(f"sequential step V={V} at={at} root={root} top_p={top_p}")
    eng, n, k = _engine(B, V), 6, 2
    q, toks, u = inputs.make_draft(V, n, k, seed=11)
    _, gl, groot = _step(eng, toks, q, u, 1, root, top_p)  # the judging row does not depend on the draft
    first, first_q, first_u = toks[:, 0].copy(), q[:, 0].copy(), u[:, 0].copy()
    _script_candidates(O.target_probs(gl[0] if root >= 0 else groot, T, top_p), first, first_q, first_u, AT[at])
    toks[:, 0], q[:, 0], u[:, 0] = first, first_q, first_u
    got, gl, groot = _step(eng, toks, q, u, 1, root, top_p)
    ref = _compare(got, gl, groot, toks, q, u, 1, root, top_p)
    assert ref is not None and ref.selected == (AT[at] if at != "none" else -1)


@pytest.mark.parametrize("V", [12288, 32000])
@pytest.mark.parametrize("at", ["suffix", *AT])
@pytest.mark.parametrize("root", [-1, 7])
@pytest.mark.parametrize("top_p", [0.0, 0.9])
def test_deferred_round_at_every_candidate(B, V, at, root, top_p):
    import torch
    say(f"deferred round V={V} at={at} root={root} top_p={top_p}")
    eng, l, s, R = _engine(B, V), 3, 6, int(root >= 0)
    q, toks, u = inputs.make_draft(V, 1, l, seed=21)
    q, toks, u = q[0], toks[0].copy(), u[0].copy()
    fq, ftoks, fu = inputs.make_draft(V, s, 1, seed=22)
    fq, ftoks, fu = fq[:, 0].copy(), ftoks[:, 0].copy(), fu[:, 0].copy()
    u[:l] = 0.0  # accepted wherever the target has any probability

    def one_pass():
        lg = torch.zeros((R + l, V), dtype=torch.float32, device="cuda")
        eng.set_prefix_len(P)
        eng.verify_deferred(to_dev(toks), to_dev(q), to_dev(u), to_dev(ftoks), to_dev(fq), to_dev(fu), temperature=T, root_token=root,
                            logits_out=lg, top_p=top_p)
        got = eng.results(1)
        assert got["status"] == 0
        gl = lg.cpu().numpy()
        return got, [gl[0] if R else eng.root_logits.cpu().numpy()] + [gl[R + m] for m in range(l)]

    for j in range(l):  # a suffix of tokens that the target would have chosen
        toks[j] = int(np.argmax(one_pass()[1][j]))
    judge = one_pass()[1]
    if at == "suffix":
        p = O.target_probs(judge[1], T, top_p)
        toks[1] = int(np.argmax(np.where(p < 0.25 * q[1], q[1], 0.0)))
        u[1] = 0.999999
    else:
        _script_candidates(O.target_probs(judge[l], T, top_p), ftoks, fq, fu, AT[at])
    got, judge = one_pass()
    if top_p:
        assert min(O.nucleus(O.target_probs(r, T), top_p)[1] for r in judge) > 1e-12
    ref = _oracle_outcome([0], toks.tolist(), judge[:l], judge[l], q, u[:l], ftoks, fq, fu, u[l], T, top_p)
    res = {"accept_len": int(got["accept_len"][0]), "next_token": int(got["next_token"][0]), "selected": got["selected"],
           "commit_len": got["commit_len"], "commit_token": got["commit_token"]}
    assert res["accept_len"] == (1 if at == "suffix" else l)
    assert res["selected"] == (-1 if at in ("suffix", "none") else AT[at])
    assert got["new_prefix_len"] == got["device_prefix_len"] == P + R + res["accept_len"]
    assert _gpu_outcome([0], toks.tolist(), res, ftoks)[0] == ref[0]
