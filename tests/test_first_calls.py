"""What the first calls of a host thread pay for beside their work."""
import threading
import time

import pytest


@pytest.mark.gpu
def test_one_enumeration_does_not_wait_for_the_choice_of_four_streams():
    """Streams for four enumerations side by side are chosen by timing pairs of them, some milliseconds; a thread's first
    call with a single enumeration (which opens a stream and allocates its lists, 0.6 ms) comes before that, and the first
    call with two pays for it."""
    from paper_2110_10548_amd import binding as B
    links = dict(bw=[10e9, 100e9], alpha=[1e-5, 1e-6])
    one = [dict(card=[2, 2], axes=[4], placement=[[2, 2]], reduce_axes=[0], max_len=2, engine=3, **links)]
    two = one + [dict(card=[2, 3], axes=[6], placement=[[2, 3]], reduce_axes=[0], max_len=2, engine=3, **links)]
    want = [len(r["programs"]) for r in B.p2_synthesize_batch(two, [1e6])]
    times = []

    def calls():
        row = []
        for queries in (one, two, one):
            t0 = time.perf_counter()
            got = B.p2_synthesize_batch(queries, [1e6])
            row.append(time.perf_counter() - t0)
            assert [len(r["programs"]) for r in got] == want[:len(queries)]
        times.append(row)
        B.p2_release_thread()

    for _ in range(5):
        th = threading.Thread(target=calls)
        th.start()
        th.join()
    assert len(times) == 5                   # (a thread whose assertion fails adds none)
    first_one, first_two = min(t[0] for t in times), min(t[1] for t in times)
    assert 2.0 * first_one < first_two
