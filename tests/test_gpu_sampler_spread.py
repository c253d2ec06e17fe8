"""The sampler's many-workgroup kernels where they can go wrong: the nucleus cut among equal and nearly equal logits (every
stage of the search: bins, refinement in the list and over the row, ties by id) on both sides of the vocabulary sizes where the
launch changes, and the sequential rule with the decision on either side of the last launch of its own."""
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


def _logits(kind, V, g):
    if kind == "normal":
        return g.normal(0, 2.0, V).astype(np.float32)
    if kind == "equal":          # one key: the ids decide
        return np.full(V, -1.25, dtype=np.float32)
    if kind == "near":           # one bin, distinct keys: refinement over the whole row
        return (3.0 + g.normal(0, 1e-4, V)).astype(np.float32)
    if kind == "levels":         # a few values, each shared by many ids
        return g.integers(-6, 7, V).astype(np.float32)
    if kind == "masked":         # most ids masked out, by -inf and by the type's lowest value
        x = g.normal(0, 2.0, V).astype(np.float32)
        x[g.random(V) < 0.5] = -np.inf
        x[g.random(V) < 0.3] = np.finfo(np.float32).min
        x[0] = 1.0
        return x
    assert kind == "peak"        # nearly all mass on one id
    x = g.normal(0, 1.0, V).astype(np.float32)
    x[V // 3] = 60.0
    return x


@pytest.mark.parametrize("V", [50, 2049, 8191, 8192, 8200, 32000, 128256])
@pytest.mark.parametrize("kind", ["normal", "equal", "near", "levels", "masked", "peak"])
def test_nucleus_ends_at_the_right_token(B, V, kind):
    """Sequences of one token, judged by one distribution with uniform 0, are accepted exactly if their token is in the
    nucleus: the tokens around the cut, in the order of the definition, must be taken and left as the oracle does."""
    g = np.random.default_rng(V)
    x = _logits(kind, V, g)
    p = O.target_probs(x, 0.9)
    for top_p in (0.313, 0.9437):
        say(f"nucleus V={V} {kind} top_p={top_p}")
        kept, margin = O.nucleus(p, top_p)
        if margin <= 1e-12:
            continue
        order = np.lexsort((np.arange(V), -p))
        cut = int((kept > 0).sum())  # tokens kept
        ids = order[[i for i in (0, cut - 3, cut - 2, cut - 1, cut, cut + 1, cut + 2, V - 1) if 0 <= i < V]].astype(np.int32)
        n = len(ids)
        q = np.zeros((n, 1, V), dtype=np.float32)
        q[np.arange(n), 0, ids] = 1.0
        u = np.zeros((n, 2), dtype=np.float32)
        u[:, 1] = 0.9999999  # the draw behind it falls on the largest id of the distribution it is made from
        got = B.spec_sample(to_dev(np.zeros((n, V), dtype=np.float32)), to_dev(x), to_dev(ids[:, None]), to_dev(q), to_dev(u),
                            temperature=0.9, top_p=top_p)
        np.testing.assert_array_equal(got["accept_len"], (kept[ids] > 0).astype(np.int32))
        # a rejected token is not in the nucleus: the correction is a draw from the nucleus itself
        c = np.cumsum(kept)
        target = float(u[0, 1]) * c[-1]
        if np.abs(c - target).min() > 1e-9:
            want = int(np.searchsorted(c, target, side="right"))
            assert all(got["next_token"][i] == want for i in range(n) if not kept[ids[i]] > 0)


def _sequential_case(V, n, k, taken, T):
    g = np.random.default_rng(V + 100 * n + taken)
    logits = g.normal(0, 1.5, (n * k, V)).astype(np.float32)
    root = g.normal(0, 1.5, V).astype(np.float32)
    q, toks, u = inputs.make_draft(V, n, k, seed=n + taken)
    toks[:, 0] = np.argmax(q[:, 0], axis=-1)  # large draft probability: rejected with a large uniform
    u[:, 0] = 0.999999
    if taken < n:
        u[taken, 0] = 1e-3
        toks[taken, 0] = int(np.argmin(q[taken, 0]))  # small draft probability: accepted
        if T == 0.0:
            toks[taken, 0] = int(np.argmax(root))
    if T == 0.0 and taken > 0:  # a residual that vanishes: the draft has all of its mass where the one-hot target has its own
        q[0, 0] = 0.0
        q[0, 0, int(np.argmax(root))] = 1.0
        toks[0, 0] = (int(np.argmax(root)) + 1) % V
    return logits, root, q, toks, u


@pytest.mark.parametrize("V,n,k", [(12288, 20, 2), (32000, 18, 1), (128256, 12, 4), (12287, 16, 3), (20001, 3, 5)])
@pytest.mark.parametrize("at", ["first", "second", "last_launch", "tail_first", "last", "none"])
@pytest.mark.parametrize("T", [1.0, 0.0])
def test_sequential_rule_decides_at_every_launch(B, V, n, k, at, T):
    taken = {"first": 0, "second": 1, "last_launch": min(max(3, min(8, V // 8192)) - 1, n - 1), "tail_first": min(max(3, min(8, V // 8192)), n - 1), "last": n - 1, "none": n}[at]
    say(f"sequential V={V} n={n} k={k} taken={taken} T={T}")
    logits, root, q, toks, u = _sequential_case(V, n, k, taken, T)
    ref = O.speculative_verify(logits, root, toks, q, u, prefix_len=7, temperature=T, select_mode=1, has_root=False)
    got = B.spec_sample(to_dev(logits), to_dev(root), to_dev(toks), to_dev(q), to_dev(u), temperature=T, select_mode=1, prefix_len=7)
    if ref.commit_margin <= 1e-9 and T > 0:
        pytest.skip("a decision within rounding of a tie")
    np.testing.assert_array_equal(got["accept_len"], ref.accept_len)
    np.testing.assert_array_equal(got["next_token"], ref.next_token)
    assert (got["selected"], got["commit_len"], got["commit_token"], got["new_prefix_len"]) == \
           (ref.selected, ref.commit_len, ref.commit_token, ref.new_prefix_len)
    assert got["status"] == 0
    # the deferred form on the same candidates: an empty suffix, first tokens judged by the root logits
    dgot = B.deferred_sample(None, to_dev(root), None, None, to_dev(u[-1:, k].copy()), to_dev(toks[:, 0].copy()), to_dev(q[:, 0].copy()),
                             to_dev(u[:, 0].copy()), temperature=T, prefix_len=7)
    assert dgot["selected"] == ref.selected and dgot["accept_len"] == 0
    assert dgot["next_token"] == (-1 if ref.selected >= 0 else ref.commit_token)


def test_device_found_faults_reach_the_status_word(B):
    """A token id outside the vocabulary: a draft token (any workgroup count), a new sequence's first token."""
    for V in (4099, 32000):
        logits, root, q, toks, u = _sequential_case(V, 3, 2, 1, 1.0)
        bad = toks.copy()
        bad[2, 1] = V
        for mode in (0, 1):
            got = B.spec_sample(to_dev(logits), to_dev(root), to_dev(bad), to_dev(q), to_dev(u), select_mode=mode, prefix_len=7)
            assert got["status"] == 1 and got["selected"] == -1 and got["new_prefix_len"] == 7
        first = toks[:, 0].copy()
        first[2] = -1
        got = B.deferred_sample(to_dev(logits[:2]), to_dev(root), to_dev(toks[0]), to_dev(q[0]), to_dev(u[0]), to_dev(first),
                                to_dev(q[:, 0].copy()), to_dev(u[:, 0].copy()), prefix_len=7)
        assert got["status"] == 1 and got["selected"] == -1 and got["new_prefix_len"] == 7
