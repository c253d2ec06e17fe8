"""The sampler at the vocabulary sizes where a launch changes: the threads that hold a slice of a row in registers (32768, 65536,
131072 entries; beyond, a slice is read twice)."""
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


def _same(B, V, n, k, T, mode, seed, prepare=None):
    """One call on random logits against the oracle, decisions and tokens; False where the oracle is within rounding of a tie."""
    g = np.random.default_rng(seed)
    logits = g.normal(0, 2.0, (n * k, V)).astype(np.float32)
    root = g.normal(0, 2.0, V).astype(np.float32)
    q, toks, u = inputs.make_draft(V, n, k, seed=seed)
    if prepare:
        prepare(logits, root, q, toks, u)
    ref = O.speculative_verify(logits, root, toks, q, u, prefix_len=5, temperature=T, select_mode=mode, has_root=False)
    if T > 0 and (ref.commit_margin <= 1e-9 or (mode == 0 and min(ref.accept_margins.min(), ref.draw_margins.min()) <= 1e-9)):
        return False
    got = B.spec_sample(to_dev(logits), to_dev(root), to_dev(toks), to_dev(q), to_dev(u), temperature=T, select_mode=mode, prefix_len=5)
    np.testing.assert_array_equal(got["accept_len"], ref.accept_len)
    np.testing.assert_array_equal(got["next_token"], ref.next_token)
    assert (got["selected"], got["commit_len"], got["commit_token"], got["new_prefix_len"], got["status"]) == \
           (ref.selected, ref.commit_len, ref.commit_token, ref.new_prefix_len, 0)
    return True


@pytest.mark.parametrize("V", [8200, 32760, 32768, 32769, 32776, 65536, 65537, 131072, 131073, 140001])
@pytest.mark.parametrize("T", [1.0, 0.0])
def test_statistics_of_a_slice_of_every_length(B, V, T):
    def last_entry_counts(logits, root, q, toks, u):
        logits[:, V - 1] = logits.max(axis=1) + 1.0  # the ends of the row carry weight: a slice cut short would show
        logits[:, 0] = logits.max(axis=1)            # T = 0: two of the largest, the lower id wins
        root[V - 1] = root.max() + 2.0
        toks[:, 0] = V - 1

    say(f"statistics V={V} T={T}")
    assert sum(_same(B, V, 2, 3, T, mode, seed, last_entry_counts) for mode in (0, 1) for seed in (1, 2)) >= 3


# (vocabulary, candidates): on both sides of the sizes where the rule over so many candidates leaves one workgroup, and of the number
# of launches that it then has (three up to 32768 entries, one candidate more without the last kernel)
@pytest.mark.parametrize("V,n", [(12287, 3), (12288, 3), (16383, 4), (16384, 4), (28671, 5), (28672, 4), (28672, 5), (28672, 6),
                                 (40960, 6), (40960, 7), (65536, 8), (65536, 9)])
@pytest.mark.parametrize("at", ["first", "last", "none"])
@pytest.mark.parametrize("T", [1.0, 0.0])
def test_sequential_rule_on_both_sides_of_every_line(B, V, n, at, T):
    taken = {"first": 0, "last": n - 1, "none": n}[at]

    def decide(logits, root, q, toks, u):
        toks[:, 0] = np.argmax(q[:, 0], axis=-1)  # a large draft probability and a large uniform: rejected
        u[:, 0] = 0.999999
        if taken < n:
            u[taken, 0] = 1e-3
            toks[taken, 0] = int(np.argmax(root)) if T == 0.0 else int(np.argmin(q[taken, 0]))
            q[:taken, 0, toks[taken, 0]] = 0.0    # the rejected ones take nothing of it away

    say(f"sequential rule V={V} n={n} at={at} T={T}")
    assert sum(_same(B, V, n, 2, T, 1, seed, decide) for seed in (1, 2, 3)) >= 2
    g = np.random.default_rng(V + n)
    root = g.normal(0, 2.0, V).astype(np.float32)
    q, toks, u = inputs.make_draft(V, n, 1, seed=n)
    decide(None, root, q, toks, u)
    ref = O.speculative_verify(np.zeros((n, V), dtype=np.float32), root, toks, q, u, prefix_len=5, temperature=T, select_mode=1, has_root=False)
    for top_p in (0.0, 0.9) if T > 0 else (0.0,):  # the deferred form: the same candidates behind an empty suffix
        if top_p:
            p = O.target_probs(root, T, top_p)
            first_in = [i for i in range(n) if i == taken and p[toks[i, 0]] > 0]
            if taken < n and not first_in:
                continue  # the token is outside the nucleus: another decision
            x_new, _ = O.duodec_verify_alg2([1], [], [], [], p, [[int(t)] for t in toks[:, 0]], q[:, 0].astype(np.float64), [],
                                            [float(a) for a in u[:, 0]], float(u[-1, 1]))
        got = B.deferred_sample(None, to_dev(root), None, None, to_dev(u[-1:, 1].copy()), to_dev(toks[:, 0].copy()), to_dev(q[:, 0].copy()),
                                to_dev(u[:, 0].copy()), temperature=T, prefix_len=5, top_p=top_p)
        if top_p:
            emitted = int(toks[got["selected"], 0]) if got["selected"] >= 0 else got["next_token"]
            assert emitted == x_new[1]
        else:
            assert got["selected"] == ref.selected
            assert got["next_token"] == (-1 if ref.selected >= 0 else ref.commit_token)
