"""CPU-side checks of the C-ABI library: it loads, exports every declared symbol, and its
host-only entry points (placements, pattern description, argument errors) agree with the oracle.
No kernel is launched here."""
import ctypes
import itertools
import os
import re
import threading
import time

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def B():
    from paper_2110_10548_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.lib()
    return binding


def test_every_declared_symbol_is_exported(B):
    header = open(os.path.join(ROOT, "include", "p2.h")).read()
    declared = set(re.findall(r"\b(p2_[a-z_]+)\s*\(", header))
    declared -= {"p2_hierarchy", "p2_options", "p2_program", "p2_stats", "p2_query", "p2_search_row"}
    assert declared == set(B.EXPORTS)
    L = ctypes.CDLL(B.LIB_PATH)
    for name in declared:
        assert getattr(L, name) is not None
    assert ctypes.sizeof(B.p2_program) == 16


@pytest.mark.parametrize("card,axes", [([1, 2, 2, 4], [4, 4]), ([2, 4], [2, 4]), ([4, 2, 4], [4, 8]), ([2, 4, 8], [2, 4, 8]),
                                       ([4, 8, 8], [4, 8, 8]), ([2, 4, 8, 8], [2, 4, 8, 8]), ([6, 4], [3, 8]), ([4, 16], [8, 2, 4])])
def test_placements_match_oracle(B, oracle, card, axes):
    a, b = B.p2_enumerate_placements(card, axes), oracle.enumerate_placements(card, axes)
    assert a.shape == b.shape and (a == b).all()


@pytest.mark.parametrize("card,axes", [([2, 4], [2, 4]), ([4, 2, 4], [4, 8]), ([3, 2, 4], [6, 4]), ([2, 3, 2], [6, 2]),
                                       ([2, 2, 2, 2], [4, 4])])
def test_patterns_match_oracle(B, oracle, card, axes):
    for r in range(1, len(axes) + 1):
        for red in itertools.combinations(range(len(axes)), r):
            for fm in (7, 3, 5, 6, 4):
                for x in oracle.enumerate_placements(card, axes):
                    q = oracle.Query(card, axes, x, list(red), form_mask=fm)
                    assert B.p2_num_patterns(card, axes, x, list(red), form_mask=fm) == q.n_patterns
                    for pid in range(q.n_patterns):
                        d, o = B.p2_describe_pattern(card, axes, x, list(red), pid, form_mask=fm), q.pattern(pid)
                        assert (d["slice"], d["form"], d["form_level"]) == (o["slice"], o["form"], o["form_level"])
                        assert (d["group_of"] == o["group_of"]).all() and (d["rank"] == o["rank"]).all()


@pytest.mark.parametrize("kind", ["system", "column", "row", "reduction"])
@pytest.mark.parametrize("card,axes", [([2, 4], [2, 4]), ([4, 2, 4], [4, 8]), ([3, 2, 4], [6, 4]), ([2, 3, 2], [6, 2]),
                                       ([2, 2, 2, 2], [4, 4]), ([2, 6], [2, 3, 2])])
def test_patterns_of_the_other_hierarchies_match_oracle(B, oracle, card, axes, kind):
    """Sec. 3.4, hierarchies (a)-(c) and the uncollapsed reduction rows: same patterns in the same order, same
    groups on the full system, same ranks (the library numbers devices by synthesis level internally)."""
    for r in range(1, len(axes) + 1):
        for red in itertools.combinations(range(len(axes)), r):
            for fm in (7, 5):
                for x in oracle.enumerate_placements(card, axes):
                    q = oracle.Query(card, axes, x, list(red), form_mask=fm, hierarchy=kind)
                    assert B.p2_num_patterns(card, axes, x, list(red), form_mask=fm, hierarchy=kind) == q.n_patterns
                    for pid in range(q.n_patterns):
                        d = B.p2_describe_pattern(card, axes, x, list(red), pid, form_mask=fm, hierarchy=kind)
                        o = q.pattern(pid)
                        assert (d["slice"], d["form"], d["form_level"]) == (o["slice"], o["form"], o["form_level"])
                        assert (d["group_of"] == o["group_of"]).all() and (d["rank"] == o["rank"]).all()


def test_canonical_alphabet_is_L_squared(B):
    # L levels with factor > 1 give L*L distinct group sets
    for f in ([8], [2, 4], [2, 1, 4], [2, 2, 2], [2, 2, 2, 2], [2, 1, 2, 1, 2]):
        L = sum(1 for v in f if v > 1)
        assert B.p2_num_patterns(f, [int(np.prod(f))], [f], [0]) == L * L


def test_argument_errors(B):
    def code(fn, *a, **k):
        with pytest.raises(B.P2Error) as e:
            fn(*a, **k)
        return e.value.code
    assert code(B.p2_enumerate_placements, [2, 4], [3, 3]) == B.P2_EINVAL               # products differ
    assert code(B.p2_enumerate_placements, [2] * 9, [512]) == B.P2_EUNSUPPORTED         # 9 levels
    assert code(B.p2_describe_pattern, [2, 4], [2, 4], [[2, 1], [1, 4]], [0, 0], 0) == B.P2_EINVAL   # duplicate axis
    assert code(B.p2_describe_pattern, [2, 4], [2, 4], [[2, 1], [1, 4]], [2], 0) == B.P2_EINVAL      # axis out of range
    assert code(B.p2_describe_pattern, [2, 4], [2, 4], [[1, 2], [1, 4]], [0], 0) == B.P2_EINVAL      # violates Eq. (1)
    assert code(B.p2_describe_pattern, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 7) == B.P2_EINVAL      # no such pattern
    assert code(B.p2_describe_pattern, [4, 16, 16], [1024], [[4, 16, 16]], [0], 0) == B.P2_EUNSUPPORTED   # > 512 devices
    # planning errors come back before any device work
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 0) == B.P2_EINVAL            # max_len < 1
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 8) == B.P2_EUNSUPPORTED      # max_len > 7
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [], 3) == B.P2_EINVAL             # empty reduce set
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, [1e6]) == B.P2_EINVAL     # costs without links
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, max_row_classes=65) == B.P2_EINVAL
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, max_row_classes=-1) == B.P2_EINVAL
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, flags=4) == B.P2_EINVAL   # unknown flag
    assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, hierarchy=5) == B.P2_EUNSUPPORTED   # no such hierarchy
    for engine in (2, 3, 4, 5):       # the other hierarchies of Sec. 3.4 run on the literal engine only
        assert code(B.p2_synthesize, [2, 4], [2, 4], [[2, 1], [1, 4]], [0], 3, hierarchy="row", engine=engine) == B.P2_EUNSUPPORTED
    assert code(B.p2_synthesize, [2, 4, 4], [2, 4, 4], [[2, 1, 1], [1, 4, 1], [1, 1, 4]], [0], 7, hierarchy="row") == B.P2_EUNSUPPORTED   # > 2^30
    # the placement search checks its arguments and counts the placements before any device work
    assert code(B.p2_search_placements, [2, 4], [3, 3], [[0]], 3, 1e6) == B.P2_EINVAL                # products differ
    assert code(B.p2_search_placements, [2, 4], [2, 4], [], 3, 1e6) == B.P2_EINVAL                   # no reduction
    assert code(B.p2_search_placements, [2, 4], [2, 4], [[]], 3, 1e6) == B.P2_EINVAL                 # empty reduction
    assert code(B.p2_search_placements, [2, 4], [2, 4], [[0]], 3, -1.0) == B.P2_EINVAL               # negative bytes
    assert code(B.p2_topk, [0.0], [0], -1) == B.P2_EINVAL
    assert code(B.p2_topk, [0.0], [0], 5000) == B.P2_EUNSUPPORTED
    assert b"" == b"" and isinstance(B.lib().p2_last_error(), bytes)


def test_workloads_are_seeded(B):
    from paper_2110_10548_amd import workloads
    a, b = workloads.config(3), workloads.config(3)
    assert a == b and all(10e9 <= v <= 400e9 for v in a["bw"])
    cfg = workloads.config(5)
    pls = B.p2_enumerate_placements(cfg["card"], cfg["axes"])
    q1, q2 = workloads.expand(cfg, pls), workloads.expand(cfg, pls)
    assert q1 == q2 and len(q1) == 512 and len(pls) == 227
    counts = [len(workloads.expand(workloads.config(i), B.p2_enumerate_placements(workloads.config(i)["card"],
                                                                                  workloads.config(i)["axes"])))
              for i in (1, 2, 3, 4)]
    assert counts == [2, 10, 84, 140]


def test_what_the_library_refuses_gets_no_room(B):
    """More message sizes or a longer shortlist than a call may ask for: the library's error, not the lack of memory for it."""
    q = dict(card=[2, 2], axes=[4], placement=[[2, 2]], reduce_axes=[0], max_len=2, bw=[1e9, 1e10], alpha=[1e-5, 1e-6])
    for msg, topk in (([1.0] * 100_000, 0), ([1.0] * 64, 2 ** 31 - 1)):
        with pytest.raises(B.P2Error) as e:
            B.p2_synthesize(**q, msg_bytes=msg, topk=topk)
        assert e.value.code == B.P2_EUNSUPPORTED
        with pytest.raises(B.P2Error) as e:
            B.p2_synthesize_batch([dict(q, topk=topk)] * 3, msg)
        assert e.value.code == B.P2_EUNSUPPORTED


def test_a_kept_result_keeps_no_more_than_a_megabyte_beside_it(B):
    q = dict(card=[2, 2], axes=[4], placement=[[2, 2]], reduce_axes=[0], max_len=2)
    b = B.Batch([q] * 400, [1.0, 2.0, 3.0])
    rows = np.random.default_rng(5).choice([0, 0, 3, 700, 5000], size=400)
    rows[:2], rows[200] = 0, 60_000                     # (nothing at first; one query with more than a megabyte)
    offs = np.concatenate([[0], np.cumsum(rows)])
    b._alloc(int(offs[-1]) + 10)
    b._offs[:] = offs
    b._progs["index"] = np.arange(len(b._progs))
    b._cost[:] = np.arange(len(b._progs))[:, None] * [1, 2, 3]
    out = b.results()
    b._progs["index"], b._cost[:] = 7, 7.0              # (the results are copies)
    assert len(out) == 400
    for i, r in enumerate(out):
        want = np.arange(offs[i], offs[i + 1])
        assert np.array_equal(r["programs"]["index"], want) and np.array_equal(r["cost"], want[:, None] * [1, 2, 3])
        beside = r["programs"].base.nbytes + r["cost"].base.nbytes - r["programs"].nbytes - r["cost"].nbytes
        assert beside <= 1 << 20


def test_room_for_rows_is_kept_per_thread_and_bounded(B):
    B._own.__dict__.clear()
    first = B._take_room(1 << 17, 2)
    B._keep_room(first, 100)
    narrow = B._take_room(1 << 17, 1)                   # (another number of message sizes: the same buffers)
    assert all(a is b for a, b in zip(narrow, first))
    assert "room" not in B._own.__dict__                # (nobody else gets them while a call writes to them)
    assert B._take_room(10, 1)[0] is not first[0]
    B._keep_room(narrow, 1 << 25)                       # a long list: given back
    assert "room" not in B._own.__dict__
    B._keep_room(narrow, 100)
    large = B._take_room((1 << 17) + 1, 1)              # what a second call needs is not kept, the first call's room is
    B._keep_room(large, 100)
    wide = B._take_room(5, 1 << 17)                     # (more message sizes than there is room for: another buffer of costs)
    assert wide[0] is first[0] and wide[1] is not first[1] and len(wide[1]) == 5 << 17
    for progs, cost, progs_at, cost_at in (first, wide, large):
        assert progs_at.value == progs.ctypes.data and ctypes.addressof(cost_at.contents) == cost.ctypes.data


def test_rooms_that_are_lent_are_written_again_only_when_unused(B):
    """Buffers that a result is a view of: the thread's again once nobody refers to them, or to anything made of them."""
    B._own.__dict__.clear()

    def call():                                         # (as a call with a long list does)
        room = B._take_room(1 << 17, 1)
        room[0]["index"][:3] += 1
        B._lend_room(room, 1 << 21)
        return room[0][:50_000], room[1][:50_000].reshape(50_000, 1)

    first = call()
    at = first[0].ctypes.data
    column = first[0]["index"][5:]                      # (a view of a view)
    del first
    second = call()
    assert second[0].ctypes.data != at and second[0]["index"][0] == 1
    del column
    third = call()                                      # (now the first one's are free)
    assert third[0].ctypes.data == at and third[0]["index"][0] == 2 and second[0]["index"][0] == 1
    kept = [call() for _ in range(4)]                   # (each its own, two of them remembered)
    assert len({r[0].ctypes.data for r in kept + [second, third]}) == 6 and len(B._own.lent) == 2
    del third, second, kept
    B._own.__dict__.clear()


def test_pieces_of_results_are_written_again_only_when_unused(B):
    q = dict(card=[2, 2], axes=[4], placement=[[2, 2]], reduce_axes=[0], max_len=2)
    b = B.Batch([q] * 3, [1.0])
    b._alloc(300)
    b._offs[:] = [0, 100, 150, 300]

    def run(value):
        b._progs["index"], b._cost[:] = value, value
        return b.results()

    first = run(1)
    column = first[1]["cost"][:, 0]
    del first
    second = run(2)
    assert (column == 1.0).all() and (second[1]["cost"] == 2.0).all()
    del second, column
    third = run(3)
    assert (third[2]["programs"]["index"] == 3).all() and all(len(r["programs"]) == n for r, n in zip(third, (100, 50, 150)))
    del third
    fourth = run(4)
    b._offs[:] = [0, 100, 150, 250]                     # (another number of rows: other memory)
    fifth = run(5)
    assert (fourth[2]["programs"]["index"] == 4).all() and (fifth[2]["programs"]["index"] == 5).all() and len(fifth[2]["programs"]) == 100


def _ready_batch(B, offs, n_msg=1):
    """A batch as a call leaves it, `offs` its queries' rows."""
    q = dict(card=[2, 2], axes=[4], placement=[[2, 2]], reduce_axes=[0], max_len=2)
    b = B.Batch([q] * (len(offs) - 1), [1.0] * n_msg)
    b._alloc(offs[-1])
    b._offs[:] = offs
    b._progs["index"] = np.arange(offs[-1])
    b._cost[:] = np.arange(offs[-1])[:, None]
    return b


def test_results_that_were_interrupted_can_be_asked_for_again(B, monkeypatch):
    b = _ready_batch(B, [0, 60_000, 120_000, 180_000])
    first = b.results()
    del first
    copy, left = B._copy_rows, [1]

    def interrupted(to, rows):
        left[0] -= 1
        if left[0] < 0:
            raise KeyboardInterrupt
        return copy(to, rows)

    monkeypatch.setattr(B, "_copy_rows", interrupted)
    with pytest.raises(KeyboardInterrupt):
        b.results()
    monkeypatch.setattr(B, "_copy_rows", copy)
    for _ in range(2):
        again = b.results()
        assert [r["programs"]["index"][0] for r in again] == [0, 60_000, 120_000]


def test_results_asked_for_by_several_threads(B):
    b = _ready_batch(B, [0, 30_000, 60_000, 90_000])
    trouble = []

    def ask(me):
        try:
            for _ in range(60):
                out = b.results()
                column = out[1]["cost"][:, 0]
                del out
                assert column[0] == 30_000.0 and column[-1] == 59_999.0
                column[:] = me                          # (what is handed out is the caller's own)
                time.sleep(0)
                assert (column == me).all()
        except BaseException as e:
            trouble.append(e)

    threads = [threading.Thread(target=ask, args=(-i - 1.0,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not trouble


def test_a_result_keeps_no_more_than_some_times_its_size(B, monkeypatch):
    """A long list is handed out in the buffers that the library wrote, unless they are many times its size, the costs' buffer among them."""
    rows, real = [0], B.lib()

    class Library:
        def p2_synthesize(self, *a):
            a[-3]._obj.value = rows[0]
            return B.P2_OK

        def __getattr__(self, name):
            return getattr(real, name)

    monkeypatch.setattr(B, "lib", Library)
    B._own.__dict__.clear()

    def kept(n, n_msg):
        rows[0] = n
        r = B.p2_synthesize([2, 2], [4], [[2, 2]], [0], 2, [1.0] * n_msg)
        assert r["programs"].shape == (n,) and r["cost"].shape == (n, n_msg)
        whole = [a if a.base is None else a.base for a in (r["programs"], r["cost"])]
        return sum(a.nbytes for a in whole) / (n * (16 + 8 * n_msg)), r["programs"].base is not None

    assert kept(100_000, 1)[1]                           # (the buffers themselves)
    kept(100, 64)                                        # (a short list: the thread's buffers are as wide as this from now on)
    for n in (16_384, 20_000, 100_000):
        assert kept(n, 1)[0] <= 8.0, n
    B._own.__dict__.clear()


def test_copies_that_a_batch_keeps_are_bounded(B):
    """Memory of earlier results is kept for the next ones as far as buffers are kept elsewhere."""
    def kept(b):
        return sum(progs.nbytes + cost.nbytes for progs, cost in b._pieces)

    b = _ready_batch(B, list(range(0, 130_001, 1000)), n_msg=1)
    b.results()
    assert kept(b) == 130_000 * 24
    b = _ready_batch(B, list(range(0, 130_001, 1000)), n_msg=30)
    for _ in range(2):
        out = b.results()
        assert all((r["cost"][0] == 1000.0 * i).all() for i, r in enumerate(out)) and 0 < kept(b) <= B._KEEP_BYTES < 130_000 * 256
