"""Frontier engine, last level: with two pairs per device the goals behind a literal prefix are read off its parent's pair
state; with one pair a literal prefix is rebuilt from its instructions.  Lists and costs must not depend on it."""
import numpy as np
import pytest


# chunk sets and masks of one word, of different numbers of words, odd radices, groups beside a master's.  Six
# instructions are the fewest whose last one can stand behind a literal prefix
@pytest.mark.gpu
@pytest.mark.parametrize("card,k", [([2, 2, 2, 2], 0), ([2, 2, 2, 2], 48), ([3, 2, 2, 2], 0), ([2, 2, 2, 5], 0), ([2, 4, 2, 4], 0), ([3, 2, 4, 3], 0)])
def test_goals_behind_literal_prefixes(card, k):
    from paper_2110_10548_amd import binding as B
    n = int(np.prod(card))
    q = dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=6, n_chunks=k, engine=3,
             bw=[12.7e9, 50.3e9, 151e9, 307e9], alpha=[2.3e-5, 1.1e-5, 5.7e-6, 1.9e-6])
    two = B.p2_synthesize_batch([dict(q, frontier_pairs=2)], [3.0e8])[0]
    one = B.p2_synthesize_batch([dict(q, frontier_pairs=1)], [3.0e8])[0]
    assert 0 < two["stats"]["literal_reruns"] < one["stats"]["literal_reruns"]
    # (several of the runs of 2048 that ranks are found through)
    index = two["programs"]["index"]
    assert len(index) > 4 * 2048 and (index[1:] > index[:-1]).all()
    assert np.array_equal(two["programs"], one["programs"])
    # costs: at most some 24 terms (six steps, four levels), added in another order where a program is re-run
    assert np.allclose(two["cost"], one["cost"], rtol=24 * 2.3e-16, atol=0.0)
    for key in ("candidates", "valid"):                  # (what is applied to prune differs between the forms)
        assert two["stats"][key] == one["stats"][key], key


def _of(card, **more):
    n, levels = int(np.prod(card)), len(card)
    return dict(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], engine=3, bw=[12.7e9, 50.3e9, 151e9, 307e9][-levels:],
                     alpha=[2.3e-5, 1.1e-5, 5.7e-6, 1.9e-6][-levels:]), **more)


# The widest chunk sets and masks (4, 8 and 16 words), and the last level's literal prefixes of both origins: seven
# instructions are the fewest with children of literal prefixes beside those of pair states (2 x 2 x 2 x 2 devices: 49 of
# 464); where two-pair prefixes are handed over, six are (3 749 of 3 757)
@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,pairs", [([2, 4, 4, 4], 6, 2), ([2, 4, 4, 8], 6, 2), ([2, 4, 8, 8], 6, 2), ([2, 2, 2, 2], 7, 2), ([3, 2, 2, 2], 7, 2),
                                                ([2, 2, 2, 2], 6, 3), ([3, 2, 2, 2], 6, 3)])
def test_goals_behind_literal_prefixes_of_wide_groups_and_of_both_origins(card, max_len, pairs):
    from paper_2110_10548_amd import binding as B
    two, one = (B.p2_synthesize_batch([_of(card, max_len=max_len, frontier_pairs=p)], [3.0e8])[0] for p in (pairs, 1))
    assert len(two["programs"]) == two["stats"]["valid"] > 4 * 2048
    assert np.array_equal(two["programs"], one["programs"])
    # costs: at most some 28 terms (seven steps, four levels), added in another order where a program is re-run
    assert np.allclose(two["cost"], one["cost"], rtol=28 * 2.3e-16, atol=0.0)
    assert two["stats"]["candidates"] == one["stats"]["candidates"]
