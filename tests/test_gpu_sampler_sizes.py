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
