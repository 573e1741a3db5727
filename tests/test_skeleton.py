"""Structures answered from the graph of their skeleton (as many levels, two devices each) beside their own devices' graphs and the
oracle: the same programs, costs and counts whatever the sizes of the levels."""
import itertools
import math
import random

import numpy as np
import pytest
import skeleton_rules

MOST = {1: 7, 2: 7, 3: 6, 4: 6, 5: 5, 6: 4}              # the size limits up to which skeletons are used, by levels
MSG = [2.0 ** 20, 3.0e8]


def _query(card, max_len, seed, **more):
    rng, L, n = random.Random(seed), len(card), int(np.prod(card))
    return dict(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, bw=[rng.uniform(1e9, 4e11) for _ in range(L)],
                     alpha=[rng.uniform(1e-6, 3e-5) for _ in range(L)]), **more)


def _same(a, b):
    assert np.array_equal(a["programs"], b["programs"]) and len(a["programs"]) > 0
    assert np.array_equal(a["cost"], b["cost"])          # (to the last bit: loads are whole numbers on either side, and added up in one order)
    for key in ("candidates", "steps_executed", "member_visits", "valid", "engine"):
        assert a["stats"][key] == b["stats"][key], key


# one level to six, twos, odd and prime sizes, sizes that divide their neighbours and such that do not, up to 512 devices; blocks of chunks
SIZES = [([2], 7, {}), ([511], 7, {}), ([2, 2], 7, {}), ([3, 170], 7, {}), ([17, 30], 6, dict(algo=1)), ([2, 2, 2], 6, {}), ([3, 4, 2], 6, {}), ([5, 3, 7], 5, dict(n_chunks=210)),
         ([8, 8, 8], 6, {}), ([3, 2, 85], 6, {}), ([2, 2, 2, 2], 6, {}), ([3, 4, 5, 2], 6, dict(n_chunks=480)), ([2, 4, 8, 8], 6, {}), ([5, 2, 3, 17], 4, {}),
         ([3, 4, 3, 4], 2, {}), ([2, 3, 2, 5, 2], 5, {}), ([2] * 6, 4, dict(algo=1)), ([3, 2, 2, 3, 2, 7], 4, {}), ([4, 3], 1, {})]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more", SIZES)
def test_skeleton_matches_the_devices(card, max_len, more):
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, 1, **more)
    # (every query by itself, which no skeleton is used for; small odd groups are walked, large ones enumerated)
    own = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY)], MSG)[0]
    auto, short = B.p2_synthesize_batch([q, dict(q, topk=3)], MSG)
    alone = B.p2_synthesize_batch([q], MSG)[0]           # (rows written straight to the host)
    for a in (auto, alone):
        _same(a, own)
    kk = min(3, len(own["programs"]))
    for m in range(len(MSG)):
        best = np.lexsort((own["programs"]["index"], own["cost"][:, m]))[:kk]
        assert np.array_equal(short["programs"]["index"][m * kk:(m + 1) * kk], own["programs"]["index"][best])


@pytest.mark.gpu
@pytest.mark.parametrize("levels", [2, 3, 4, 5, 6])
def test_structures_of_one_skeleton(levels):
    """Groups of many sizes in one batch, more than a wavefront's lanes of them, among other axes and with levels of one device: each as alone."""
    from paper_2110_10548_amd import binding as B
    rng = random.Random(levels)
    queries = []
    while len(queries) < (70 if levels <= 3 else 12):
        f = [rng.choice((2, 2, 3, 4, 5, 6, 8, 11)) for _ in range(levels)]
        for _ in range(rng.randrange(3)):
            f.insert(rng.randrange(len(f) + 1), 1)       # (a hardware level that the group does not span)
        g = [rng.choice((1, 1, 2, 3)) for _ in f]        # the other axis
        if len(f) > 8 or np.prod(f) * np.prod(g) > 512 or np.prod(f) < 66:
            continue
        card = [a * b for a, b in zip(f, g)]
        q = _query(card, min(MOST[levels], 4), len(queries), axes=[int(np.prod(f)), int(np.prod(g))], placement=[f, g], algo=rng.randrange(2), topk=rng.choice((0, 0, 4)))
        queries.append(q)
    together = B.p2_synthesize_batch(queries, MSG)
    apart = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY) for q in queries[:24]], MSG)
    for q, r, o in zip(queries, together, apart):
        _same(r, o)
    for q, r in list(zip(queries, together))[24:]:
        _same(r, B.p2_synthesize_batch([q], MSG)[0])
    assert {r["stats"]["route"] for r in together} <= {0, B.ROUTE_GRAPH} and sum(r["stats"]["steps_evaluated"] > 0 for r in together) < len(queries)


# chunks that are no multiple of the group's devices: how often rows can be cut is the group's own; chunks that divide for some levels, for none, one chunk
@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,chunks", [([80], 4, 16), ([8, 9], 5, 12), ([16, 8], 4, 8), ([4, 4], 5, 4), ([3, 4, 6], 4, 6), ([2, 4, 8], 5, 1), ([4, 4, 8], 4, 8), ([4, 2, 4], 6, 48),
                                                 ([2, 2, 2, 2], 5, 8), ([2, 3, 4, 5], 4, 30), ([2, 4, 8, 8], 4, 64)])
def test_rows_that_do_not_divide(card, max_len, chunks):
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, 2, n_chunks=chunks)
    other = dict(q, n_chunks=int(np.prod(card)))         # (the whole skeleton beside it)
    own = B.p2_synthesize_batch([dict(x, flags=B.FLAG_EVALUATE_EVERY_QUERY) for x in (q, other)], MSG)
    for a, o in zip(B.p2_synthesize_batch([q, other], MSG), own):
        _same(a, o)
    _same(B.p2_synthesize_batch([q], MSG)[0], own[0])


@pytest.mark.gpu
def test_sizes_drawn_from_all():
    """A draw of the 15 407 lists of one to six levels with up to 512 devices, at the largest size limits."""
    from paper_2110_10548_amd import binding as B
    rng = random.Random(11)
    for levels, n in ((1, 12), (2, 40), (3, 40), (4, 16), (5, 6), (6, 10)):
        cards = []
        while len(cards) < n:
            c = [min(int(2.0 ** rng.uniform(1.0, 10.0 - levels)), 512) for _ in range(levels)]
            if np.prod(c) <= 512:
                cards.append(c)
        queries = [_query(c, MOST[levels], i) for i, c in enumerate(cards)]
        for a in range(0, n, 2):
            own = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY) for q in queries[a:a + 2]], MSG[:1])
            for r, o in zip(B.p2_synthesize_batch(queries[a:a + 2], MSG[:1]), own):
                _same(r, o)


@pytest.mark.parametrize("levels,max_len,cards", [(1, 6, [[3], [8], [97]]), (2, 4, [[2, 3], [3, 2], [4, 6], [5, 5], [9, 2]]), (3, 3, [[2, 3, 2], [3, 2, 4], [2, 2, 5], [3, 3, 3]])])
def test_programs_do_not_depend_on_the_sizes(oracle, levels, max_len, cards):
    """What skeletons rest on, as the oracle sees it: programs and prefixes of any sizes are those of twos."""
    def of(card):
        o = oracle.Query(card, [int(np.prod(card))], [card], [0])
        r = o.synthesize(max_len)
        return r["index"].tolist(), o.eval_indices(max_len, start=0, count=o.num_candidates(max_len))[2]
    want = of([2] * levels)
    for card in cards:
        assert of(card) == want, card


# selections by wavefronts (up to ten), by blocks of 64, 256 and 1 024 threads; more asked for than there is; nothing valid; a graph of the devices themselves
@pytest.mark.gpu
@pytest.mark.parametrize("queries", [[([2, 2], 3, 1, {})], [([3, 4, 6], 4, 10, {}), ([2, 2], 5, 10, {}), ([7], 2, 3, {}), ([12, 12], 1, 4, {})], [([2, 2], 4, 64, {}), ([2, 3, 2], 3, 50, {})],
                                     [([2, 2, 2], 5, 200, {}), ([4, 4], 2, 7, {})], [([2, 2, 2, 2], 5, 1024, {}), ([4, 4], 5, 1024, {})],
                                     [([2, 4], 3, 5, dict(op_mask=2)), ([2, 4], 3, 5, {}), ([4, 4], 4, 3, dict(op_mask=0b10101))], [([2] * 5, 4, 9, {}), ([2, 2, 2], 7, 6, {})]])
def test_shortlists_selected_before_the_count(queries):
    """Calls whose queries all ask for shortlists: the cheapest of the lists that they have without, by (cost, index)."""
    from paper_2110_10548_amd import binding as B
    asked = [_query(c, m, i, topk=k, **more) for i, (c, m, k, more) in enumerate(queries)]
    for msg in (MSG, [1.0, 2.0 ** 22, 5e9]):
        for q, r in zip(asked, B.p2_synthesize_batch(asked, msg)):
            full = B.p2_synthesize_batch([dict(q, topk=0)], msg)[0]
            kk = min(q["topk"], len(full["programs"]))
            assert r["stats"]["valid"] == len(full["programs"]) and len(r["programs"]) == kk * len(msg)
            for m in range(len(msg)):
                best = np.lexsort((full["programs"]["index"], full["cost"][:, m]))[:kk]
                assert np.array_equal(r["programs"][m * kk:(m + 1) * kk], full["programs"][best]) and np.array_equal(r["cost"][m * kk:(m + 1) * kk], full["cost"][best])


# rows of one graph written once for its queries, 32 to a block: two blocks and three, step costs not fused (more than 2^30 candidates); beside queries with rows of their own
@pytest.mark.gpu
@pytest.mark.parametrize("large,n", [(False, 33), (True, 65)])
def test_rows_written_once_for_many_queries(large, n):
    from paper_2110_10548_amd import binding as B
    rng = random.Random(n)
    cards = [c for c in ([a, b, c, d] for a in (2, 3, 4) for b in (2, 4, 5) for c in (2, 3, 8) for d in (2, 4, 6, 8)) if (300 if large else 16) <= np.prod(c) <= (512 if large else 64)]
    queries = [_query(rng.choice(cards), 6, i, topk=rng.choice((1, 7, 40)), algo=i % 2) for i in range(n)]
    queries += [_query([3, 4, 6], 4, 99, topk=5), _query([2, 2], 5, 98, topk=5)]
    rng.shuffle(queries)
    for msg in (MSG[:1], MSG + [7.0]):
        full = B.p2_synthesize_batch([dict(q, topk=0) for q in queries], msg)
        for q, f, r in zip(queries, full, B.p2_synthesize_batch(queries, msg)):
            kk = q["topk"]
            assert r["stats"]["valid"] == len(f["programs"]) and len(r["programs"]) == kk * len(msg)
            for m in range(len(msg)):
                best = np.lexsort((f["programs"]["index"], f["cost"][:, m]))[:kk]
                assert np.array_equal(r["programs"][m * kk:(m + 1) * kk], f["programs"][best]) and np.array_equal(r["cost"][m * kk:(m + 1) * kk], f["cost"][best])


# the same with step costs that are fused (spaces of up to 2^30 candidates are costed as their walk is): three and four levels, small groups and large among them; one block more or less than full
@pytest.mark.gpu
@pytest.mark.parametrize("levels,max_len,n", [(4, 4, 32), (4, 4, 33), (3, 5, 70), (2, 5, 64)])
def test_rows_written_once_with_fused_costs(levels, max_len, n):
    from paper_2110_10548_amd import binding as B
    rng = random.Random(n)
    cards = [c for c in itertools.product((2, 3, 4, 5, 8, 11), repeat=levels) if 66 <= math.prod(c) <= 512] + [(2,) * levels, (2,) * (levels - 1) + (4,)]
    queries = [_query(list(rng.choice(cards)), max_len, i, topk=rng.choice((1, 7, 40)), algo=i % 2) for i in range(n)]
    for msg in (MSG[:1], MSG + [7.0]):
        full = B.p2_synthesize_batch([dict(q, topk=0) for q in queries], msg)
        for q, f, r in zip(queries, full, B.p2_synthesize_batch(queries, msg)):
            assert r["stats"]["candidates"] <= 1 << 30 and r["stats"]["route"] == B.ROUTE_GRAPH and r["stats"]["valid"] == len(f["programs"])
            for m in range(len(msg)):
                kk = min(q["topk"], len(f["programs"]))
                best = np.lexsort((f["programs"]["index"], f["cost"][:, m]))[:kk]
                assert np.array_equal(r["programs"][m * kk:(m + 1) * kk], f["programs"][best]) and np.array_equal(r["cost"][m * kk:(m + 1) * kk], f["cost"][best])


# selections by wavefronts, by blocks of 64, 256 and 1 024 threads; the first size or a later one; a query that has no program beside them
@pytest.mark.gpu
@pytest.mark.parametrize("k", [2, 9, 20, 200, 1024])
@pytest.mark.parametrize("msg", [[float("inf")], [1e6, float("inf"), 1e7]])
def test_shortlists_of_costs_that_are_no_numbers(k, msg):
    """Links that take no time and a size without end: every selection reports for itself, the call is refused, and the next one finds nothing of it."""
    from paper_2110_10548_amd import binding as B
    no_time = lambda n: [float("inf")] * n
    asked = [_query([2, 2], 3, 1, topk=k, bw=no_time(2)), _query([3, 4, 6], 4, 2, topk=k, bw=no_time(3)), _query([2, 4], 3, 3, topk=k, op_mask=2, bw=no_time(2))]
    with pytest.raises(Exception, match="NaN cost"):
        B.p2_synthesize_batch(asked, msg)
    for q, r in zip(asked, B.p2_synthesize_batch(asked, [1e6])):
        full = B.p2_synthesize_batch([dict(q, topk=0)], [1e6])[0]
        best = np.lexsort((full["programs"]["index"], full["cost"][:, 0]))[:k]
        assert np.array_equal(r["programs"], full["programs"][best])


@pytest.mark.gpu
def test_room_for_the_costs_of_many_queries():
    """What each query keeps beside a skeleton's graph: a cost for every edge of the states on the way to a goal that there can be (at most as many as states
    and 256 more), its rows' costs and its description."""
    import torch
    from paper_2110_10548_amd import binding as B
    n, max_len, states, rows = 4096, 3, 768, 138
    queries = [_query([2, 2, 2, 2], max_len, i, topk=1) for i in range(n)]
    B.p2_synthesize_batch(queries[:1], MSG[:1])          # (the runtime's own memory)
    B.p2_release_thread()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    results = B.p2_synthesize_batch(queries, MSG[:1])
    held = before - torch.cuda.mem_get_info()[0]
    assert {r["stats"]["route"] for r in results} == {B.ROUTE_GRAPH} and [r["stats"]["valid"] for r in results] == [rows] * n
    assert held < n * (8 * (states + 256) + 8 * rows + 4096) + (24 << 20)
    B.p2_release_thread()


@pytest.mark.gpu
def test_shortlists_beyond_the_bound_of_pinned_memory():
    """More rows to pick than are written to the host before they are counted: 400 queries of 86 programs, all of them asked for, 64 sizes."""
    from paper_2110_10548_amd import binding as B
    queries = [_query([2, 2 + i % 3], 4, i, topk=1024) for i in range(400)]
    msg = [2.0 ** (10 + 0.25 * m) for m in range(64)]
    for i, r in list(enumerate(B.p2_synthesize_batch(queries, msg)))[::57]:
        o = B.p2_synthesize_batch(queries[i:i + 1], msg)[0]
        assert r["stats"]["valid"] == 86 and len(o["programs"]) == 64 * 86
        assert np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"], o["cost"])


# a size without end over links that take no time, and no bytes over links that take for ever; the last one has numbers
@pytest.mark.gpu
@pytest.mark.parametrize("bytes_, bw, none", [(float("inf"), float("inf"), True), (0.0, 1e-310, True), (float("inf"), 1e9, False)])
def test_baselines_that_are_no_numbers(bytes_, bw, none):
    """A search whose own programs are none: the AllReduce beside them is reported whatever its cost."""
    from paper_2110_10548_amd import binding as B
    r = B.p2_search_placements([2, 4], [4, 2], [[0], [1]], 3, bytes_, bw=[bw] * 2, alpha=[1e-5, 1e-6], op_mask=2)
    for row in r["rows"].values():
        assert row["valid"] == 0 and row["best_cost"] == float("inf")
        assert np.isnan(row["allreduce_cost"]) if none else row["allreduce_cost"] == float("inf")


@pytest.mark.gpu
def test_who_was_evaluated_for_itself():
    """evaluated_with names the query that a graph was built for, whatever the sizes of its levels; what is -1 was evaluated."""
    from paper_2110_10548_amd import binding as B
    cards = [[2, 4, 8, 8], [4, 16], [2, 2, 2, 2], [3, 4, 6], [8, 9], [2, 4, 8, 8], [5, 2, 7], [3, 2, 4, 5]]
    queries = [_query(c, 4, i) for i, c in enumerate(cards)] + [_query([4, 4], 4, 9, n_chunks=6), _query([4, 4], 4, 8, n_chunks=6)]
    results = B.p2_synthesize_batch(queries, MSG)
    assert [r["stats"]["evaluated_with"] for r in results] == [-1, -1, 0, -1, 1, 0, 3, 0, -1, 8]
    for r in results:
        s = r["stats"]
        assert s["route"] == B.ROUTE_GRAPH and (s["steps_evaluated"] > 0) == (s["members_evaluated"] > 0) == (s["evaluated_with"] < 0)
        if s["evaluated_with"] >= 0:
            first = results[s["evaluated_with"]]
            assert np.array_equal(r["programs"], first["programs"]) and s["steps_executed"] == first["stats"]["steps_executed"]


# every list of so many levels with at most so many devices, every number of chunks up to one and a half times as many: those that are no multiple of the
# group's devices, where how often rows can be cut is the group's own, and the multiple
@pytest.mark.parametrize("levels,devices,max_len", [(1, 30, 7), (2, 20, 4), (2, 12, 7), (3, 12, 4), (3, 8, 6), (4, 24, 2), (4, 16, 3), (4, 16, 4)])
def test_rules_of_skeletons(oracle, levels, devices, max_len):
    """What the kernels of skeletons go by (tests/skeleton_rules.py) beside the oracle on the devices themselves: programs and prefixes."""
    for card in itertools.product(range(2, devices + 1), repeat=levels):
        R = math.prod(card)
        for k in range(1, R * 3 // 2 + 1) if R <= devices else ():
            split = k % R != 0
            if levels == 4 and max_len == 4 and k not in (2, 8, 16, 24):
                continue
            edges, _ = skeleton_rules.graph(levels, max_len, card[::-1] if split else None, k if split else 0)
            mine = sorted(skeleton_rules.programs(edges, max_len))
            o = oracle.Query(card, [R], [card], [0], n_chunks=k)
            r = o.synthesize(max_len)
            assert mine == sorted(tuple(i[:n]) for i, n in zip(r["instr"].tolist(), r["len"].tolist())), (card, k)
            # (the oracle tries the alphabet behind every prefix and every program that is not at the limit)
            tried = sum(skeleton_rules.prefixes(edges, max_len)) + sum(len(p) < max_len for p in mine)
            assert tried * o.alphabet == r["steps_tried"], (card, k)


# graphs of their own for many numbers of chunks: more than a launch has blocks for every state of, with and without one of four levels; two of four levels
@pytest.mark.gpu
@pytest.mark.parametrize("n,four", [(3, 1), (40, 0), (130, 2)])
def test_many_skeletons_in_one_launch(n, four):
    from paper_2110_10548_amd import binding as B
    cards = [[2, 4, 8], [4, 16], [3, 4, 5], [8, 2, 4], [80], [2, 8, 4]]
    queries = [_query(cards[i % 6], 4, i, n_chunks=3 + i // 6, topk=(0, 5)[i % 2]) for i in range(n)] + [_query([2, 2, 2, 2], 5, 900 + i, n_chunks=(16, 6)[i]) for i in range(four)]
    together = B.p2_synthesize_batch(queries, MSG)
    assert sum(r["stats"]["route"] == B.ROUTE_GRAPH and r["stats"]["evaluated_with"] < 0 for r in together) > n // 2
    for i in list(range(0, n, 7)) + list(range(n, n + four)):
        own = B.p2_synthesize_batch([dict(queries[i], flags=B.FLAG_EVALUATE_EVERY_QUERY)], MSG)[0]
        # (many groups of more than 64 devices may be walked, and say so; the results are the same)
        assert np.array_equal(together[i]["programs"], own["programs"]) and np.array_equal(together[i]["cost"], own["cost"]) and len(own["programs"]) > 0
        assert together[i]["stats"]["valid"] == own["stats"]["valid"]


# skeletons of five and six levels that are their queries' own graphs: up to eight queries costed from bandwidth rows, with one of other sizes among them not
@pytest.mark.gpu
@pytest.mark.parametrize("levels,max_len,n,other", [(5, 5, 8, []), (5, 5, 9, []), (6, 4, 3, []), (5, 5, 2, [[3, 2, 2, 2, 2]]), (6, 4, 1, [[2, 2, 2, 2, 2, 3]])])
def test_large_skeletons_of_few_queries(levels, max_len, n, other):
    from paper_2110_10548_amd import binding as B
    queries = [_query([2] * levels, max_len, i, algo=i % 2, topk=(0, 30)[i % 3 == 1], n_chunks=(0, 2 ** levels * 2)[i % 2]) for i in range(n)] + [_query(c, max_len, 50) for c in other]
    for q, r in zip(queries, B.p2_synthesize_batch(queries, MSG)):
        _same(r, B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY)], MSG)[0])
        assert r["stats"]["route"] == B.ROUTE_GRAPH


@pytest.mark.gpu
def test_room_for_shortlists_of_narrowed_alphabets():
    """Queries that have a handful of the programs that their levels can have take no room for all of them."""
    import torch
    from paper_2110_10548_amd import binding as B
    queries = [_query([2, 2, 2, 2], 6, i, topk=3, op_mask=1) for i in range(200)]
    B.p2_synthesize_batch(queries[:1], MSG[:1])
    B.p2_release_thread()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    results = B.p2_synthesize_batch(queries, MSG[:1])
    held = before - torch.cuda.mem_get_info()[0]
    B.p2_release_thread()
    assert {r["stats"]["route"] for r in results} == {B.ROUTE_GRAPH} and all(0 < r["stats"]["valid"] < 1000 for r in results)
    # (200 times 83 920 rows of 32 bytes would be 537 MB)
    assert held < 200 << 20
