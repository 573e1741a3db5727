"""Engine AUTO beside the shared-prefix engine's reach: large groups and levels that are no power of two are enumerated by
size with pruning where that is faster than a lane per candidate; the lists, costs and counts stay those of the walk."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,k,expect", [([80], 3, 0, 3), ([128], 2, 0, 2), ([9, 8], 3, 0, 3), ([3, 4, 6], 3, 0, 3), ([6, 8], 5, 0, 3),
                                                   ([6, 8], 3, 0, 2), ([3, 5], 5, 1, 2), ([2, 8, 8], 3, 96, 3), ([3, 2, 2], 5, 24, 3),
                                                   ([5, 2, 2, 6], 3, 0, 3)])
def test_auto_engine_matches_the_walk(card, max_len, k, expect):
    from paper_2110_10548_amd import binding as B
    n = int(np.prod(card))
    q = dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, n_chunks=k,
             bw=[12.7e9, 50.3e9, 151e9, 307e9][:len(card)], alpha=[2.3e-5, 1.1e-5, 5.7e-6, 1.9e-6][:len(card)])
    msg = [2.0 ** 20, 3.0e8]
    auto, walk, lit = B.p2_synthesize_batch([q, dict(q, engine=2), dict(q, topk=7)], msg)
    assert auto["stats"]["engine"] == expect and walk["stats"]["engine"] == 2
    assert np.array_equal(auto["programs"], walk["programs"])
    assert np.array_equal(auto["cost"], walk["cost"])          # (to the last bit: shortlists with ties stay as they were)
    for key in ("candidates", "steps_executed", "member_visits", "valid"):
        assert auto["stats"][key] == walk["stats"][key], key
    kk = min(7, len(auto["programs"]))
    for m in range(2):
        want = np.lexsort((auto["programs"]["index"], auto["cost"][:, m]))[:kk]
        assert np.array_equal(lit["programs"]["index"][m * kk:(m + 1) * kk], auto["programs"]["index"][want])


def _whole(card, max_len, **more):
    n = int(np.prod(card))
    return dict(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, bw=[12.7e9, 151e9, 307e9][:len(card)],
                     alpha=[2.3e-5, 5.7e-6, 1.9e-6][:len(card)]), **more)


# Enumerations run four at a time, the walk takes all groups in one launch: more than four small groups with few candidates
# that differ in structure are walked, the same group many times over, large groups and many candidates are enumerated
@pytest.mark.gpu
@pytest.mark.parametrize("cards,max_len,expect", [([[66], [70], [75], [80]], 4, 3), ([[66], [70], [75], [80], [90]], 4, 2),
                                                  ([[66], [70], [75], [80], [66], [70], [75], [80]], 4, 3), ([[8, 9], [9, 8], [7, 10], [6, 11], [12, 6], [5, 14], [3, 24]], 2, 2),
                                                  ([[8, 9], [9, 8], [7, 10], [6, 11], [12, 6], [5, 14], [3, 24]], 3, 3), ([[300], [310], [320], [330], [340], [350]], 3, 3)])
def test_auto_engine_over_a_batch_of_large_groups(cards, max_len, expect):
    from paper_2110_10548_amd import binding as B
    msg = [2.0 ** 20, 3.0e8]
    queries = [_whole(card, max_len) for card in cards]
    small = _whole([2, 2], 3)                                # (a query of another kind changes nothing)
    auto = B.p2_synthesize_batch(queries + [small], msg)
    walk = B.p2_synthesize_batch([dict(q, engine=2) for q in queries], msg)
    assert [a["stats"]["engine"] for a in auto] == [expect] * len(cards) + [5]
    for a, w, q in zip(auto, walk, queries):
        alone = B.p2_synthesize_batch([q], msg)[0]
        for other in (w, alone):
            assert np.array_equal(a["programs"], other["programs"]) and np.array_equal(a["cost"], other["cost"])
            for key in ("candidates", "steps_executed", "member_visits", "valid"):
                assert a["stats"][key] == other["stats"][key], key
