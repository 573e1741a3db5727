"""Frontier engine: the places of the valid programs in ascending index order, by counting for short lists and by sorted
runs for long ones; and the launches that this takes."""
import numpy as np
import pytest


# 1 .. 571 programs: one launch to rank them; 1 646 (one run) and 2 549 (two): two launches
@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,valid,launches", [([2, 4], 1, 1, 1), ([2, 4], 3, 35, 1), ([2, 2, 4], 3, 80, 1), ([2, 2, 4], 4, 571, 1),
                                                         ([2, 2, 2, 2], 4, 1646, 2), ([2, 2, 4], 5, 2549, 2)])
def test_ranks_of_short_and_long_lists(card, max_len, valid, launches):
    from paper_2110_10548_amd import binding as B
    n = int(np.prod(card))
    q = dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, engine=3, bw=[12.7e9, 50.3e9, 151e9, 307e9][-len(card):],
             alpha=[2.3e-5, 1.1e-5, 5.7e-6, 1.9e-6][-len(card):])
    B.p2_set_profiling(True)
    try:
        got = B.p2_synthesize_batch([q], [3.0e8])[0]
        prof = B.p2_get_profile()
    finally:
        B.p2_set_profiling(False)
    index = got["programs"]["index"]
    assert len(index) == valid and (index[1:] > index[:-1]).all()
    walk = B.p2_synthesize_batch([dict(q, engine=2)], [3.0e8])[0]
    assert np.array_equal(got["programs"], walk["programs"])
    assert prof["post_launches"] == launches + 1            # (and the rows of all programs in one)
