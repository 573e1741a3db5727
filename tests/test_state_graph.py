"""The state graph that engine AUTO answers groups of up to 64 devices with power-of-two patterns from, beside the engines
whose place it takes: the walk of every candidate (compact) and the enumeration by size (frontier)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_10548_amd", "csrc")


def _compiled(tmp_path, code, *sources):
    """What a host program over the library's host sources prints."""
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text(code)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(tmp_path / "main.cpp"), *(os.path.join(CSRC, s) for s in sources), "-o", str(tmp_path / "main")], check=True)
    return subprocess.run([str(tmp_path / "main")], check=True, capture_output=True, text=True, timeout=60).stdout


def _query(card, max_len, **more):
    n = int(np.prod(card))
    L = len(card)
    return dict(dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len,
                     bw=[12.7e9, 30e9, 50.3e9, 151e9, 180e9, 307e9][:L], alpha=[2.3e-5, 1.5e-5, 1.1e-5, 5.7e-6, 3.1e-6, 1.9e-6][:L]), **more)


MSG = [2.0 ** 20, 3.0e8]
COUNTS = ("candidates", "steps_executed", "member_visits", "valid")

# teams of 2 to 64 lanes; one block alone (up to two levels) and launches per level; size limits from 1; rows that are
# blocks of chunks (a multiple of R), chunks that are not, a single one; alphabets that end inside a word and run over three
WALKED = [([2], 1, {}), ([2], 4, {}), ([64], 3, {}), ([2, 2], 5, {}), ([4, 16], 3, {}), ([32, 2], 3, dict(n_chunks=128)), ([8, 8], 2, dict(n_chunks=3)),
          ([2, 4], 4, dict(n_chunks=12)), ([2, 4], 3, dict(n_chunks=1)), ([4, 4], 4, dict(op_mask=0b10101)), ([4, 4], 4, dict(form_mask=3)),
          ([2, 2, 2], 4, {}), ([4, 2, 8], 2, dict(n_chunks=8)), ([2, 4, 8], 3, dict(algo=1)), ([2, 2, 4], 4, dict(op_mask=0b00111, n_chunks=48)),
          ([2, 2, 2, 2], 3, dict(form_mask=5)), ([2, 2, 2, 2, 2], 2, {}), ([2, 2, 2, 2, 2, 2], 2, dict(n_chunks=7)), ([4, 4, 4], 1, {})]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more", WALKED)
def test_graph_matches_the_walk(card, max_len, more):
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, **more)
    auto, short, shared = B.p2_synthesize_batch([q, dict(q, topk=5), dict(q, bw=q["bw"][::-1], algo=1)], MSG)
    walk, walk_b = B.p2_synthesize_batch([dict(q, engine=2), dict(q, engine=2, bw=q["bw"][::-1], algo=1)], MSG)
    alone = B.p2_synthesize_batch([q], MSG)[0]           # (rows written straight to the host)
    for a, w in ((auto, walk), (alone, walk), (shared, walk_b)):
        assert a["stats"]["engine"] == 5 and a["stats"]["route"] == B.ROUTE_GRAPH and np.array_equal(a["programs"], w["programs"])
        assert np.array_equal(a["cost"], w["cost"])      # (to the last bit: shortlists with ties stay as they were)
        for key in COUNTS:
            assert a["stats"][key] == w["stats"][key], key
        assert a["stats"]["steps_evaluated"] <= a["stats"]["steps_executed"]
    kk = min(5, len(walk["programs"]))
    for m in range(len(MSG)):
        want = np.lexsort((walk["programs"]["index"], walk["cost"][:, m]))[:kk]
        assert np.array_equal(short["programs"]["index"][m * kk:(m + 1) * kk], walk["programs"]["index"][want])
    nothing = B.p2_synthesize_batch([q], [])[0]          # (no message size: validity alone)
    assert np.array_equal(nothing["programs"], walk["programs"]) and {r["stats"]["route"] for r in (short, nothing)} == {B.ROUTE_GRAPH}
    assert {r["stats"]["route"] for r in (walk, walk_b)} == {0}


# too many candidates to walk; three and four pairs on a device; the most levels, states and rows
ENUMERATED = [([2, 2, 2], 7, {}), ([4, 4, 4], 6, {}), ([2, 2, 2, 2], 6, {}), ([2, 2, 2, 4], 5, dict(n_chunks=24)), ([2, 2, 2, 2, 2], 5, {}),
              ([2, 2, 2, 2, 2, 2], 4, {})]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more", ENUMERATED)
def test_graph_matches_the_enumeration(card, max_len, more):
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, **more)
    a = B.p2_synthesize_batch([q], MSG)[0]
    b = B.p2_synthesize_batch([dict(q, engine=3)], MSG)[0]
    assert (a["stats"]["route"], b["stats"]["route"]) == (B.ROUTE_GRAPH, 0)
    assert np.array_equal(a["programs"], b["programs"]) and len(a["programs"]) > 1000
    assert np.allclose(a["cost"], b["cost"], rtol=1e-14, atol=0.0)       # (a dozen additions in 64 bits)
    if a["stats"]["engine"] == 3:
        assert np.array_equal(a["cost"], b["cost"])
        # (one step per valid prefix and instruction; the enumeration also counts what it applies again to rebuild a prefix)
        assert a["stats"]["valid"] == b["stats"]["valid"] and 0 < a["stats"]["steps_executed"] <= b["stats"]["steps_executed"]


# Groups that the frontier's kernels build the graph of: more than 64 devices, levels that are no power of two; rows that are
# blocks of chunks; children that need a third pair judged at the size limit (six instructions); tree costs
LARGE = [([3, 4, 6], 4, {}), ([3, 4, 6], 5, dict(algo=1)), ([128], 4, {}), ([2, 8, 8], 4, dict(n_chunks=512)), ([2, 8, 8], 3, dict(n_chunks=96)),
         ([3, 5, 7], 4, dict(n_chunks=210, op_mask=0b11101)), ([5, 2, 2, 6], 4, dict(form_mask=3)), ([2, 2, 4, 8], 6, {}), ([3, 2, 12], 6, {}), ([3, 2, 12], 7, dict(op_mask=0b11011)), ([6, 6], 6, {})]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more", LARGE)
def test_large_graph_matches_the_enumeration(card, max_len, more):
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, **more)
    alone = B.p2_synthesize_batch([q], MSG)[0]
    listed, short = B.p2_synthesize_batch([dict(q, bw=q["bw"][::-1]), dict(q, topk=9)], MSG)
    want, want_b = B.p2_synthesize_batch([dict(q, engine=3), dict(q, engine=3, bw=q["bw"][::-1])], MSG)
    assert {r["stats"]["route"] for r in (alone, listed, short)} == {B.ROUTE_GRAPH} and want["stats"]["route"] == 0
    for a, w in ((alone, want), (listed, want_b)):
        assert np.array_equal(a["programs"], w["programs"])
        assert np.allclose(a["cost"], w["cost"], rtol=1e-14, atol=0.0)
        assert a["stats"]["valid"] == w["stats"]["valid"] and a["stats"]["candidates"] == w["stats"]["candidates"]
        assert a["stats"]["steps_executed"] > 0
    kk = min(9, len(want["programs"]))
    for m in range(len(MSG)):
        best = np.lexsort((alone["programs"]["index"], alone["cost"][:, m]))[:kk]
        assert np.array_equal(short["programs"]["index"][m * kk:(m + 1) * kk], alone["programs"]["index"][best])


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len", [([5, 10, 10], 3), ([2, 4, 8, 8], 3), ([3, 4, 6], 4), ([2, 9, 9], 4), ([130], 5), ([7, 11], 5)])
def test_large_graph_matches_the_walk(card, max_len):
    """Against the engine that walks every candidate: groups with few and many patterns' groups, odd sizes, up to 512 devices."""
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len)
    auto, want = (B.p2_synthesize_batch([dict(q, engine=e)], MSG)[0] for e in (0, 2))
    assert np.array_equal(auto["programs"], want["programs"]) and len(want["programs"]) > 0
    assert np.allclose(auto["cost"], want["cost"], rtol=1e-14, atol=0.0)
    assert auto["stats"]["valid"] == want["stats"]["valid"] and (auto["stats"]["route"], want["stats"]["route"]) == (B.ROUTE_GRAPH, 0)


@pytest.mark.gpu
def test_large_graphs_side_by_side():
    """Several large groups on streams of their own beside small ones, and one after the other: the same bytes."""
    from paper_2110_10548_amd import binding as B
    queries = [_query(c, m, topk=k) for c, m, k in (([3, 4, 6], 4, 0), ([9, 8], 4, 5), ([2, 4, 4], 4, 0), ([2, 8, 8], 4, 7), ([12, 12], 4, 0), ([80], 4, 0),
                                                    ([4, 4], 4, 3), ([5, 2, 2, 6], 3, 0))]
    side = B.p2_synthesize_batch(queries, MSG)
    one = B.p2_synthesize_batch([dict(q, flags=B.FLAG_ONE_ENUMERATION_AT_A_TIME) for q in queries], MSG)
    assert {r["stats"]["route"] for r in side + one} == {B.ROUTE_GRAPH}
    for q, a, b in zip(queries, side, one):
        alone = B.p2_synthesize_batch([q], MSG)[0]
        for r in (b, alone):
            assert np.array_equal(a["programs"], r["programs"]) and np.array_equal(a["cost"], r["cost"])
            for key in COUNTS:
                assert a["stats"][key] == r["stats"][key], key


@pytest.mark.gpu
def test_graphs_beside_other_engines():
    """Queries answered from graphs, walked and enumerated in one batch, each as alone."""
    from paper_2110_10548_amd import binding as B
    queries = [_query([2, 3], 3), _query([4, 4], 4), _query([80], 3, topk=4), _query([2, 4, 4], 3, topk=3), _query([4, 4], 4, engine=5),
               _query([2, 2], 3, hierarchy=1), _query([2, 4, 4], 3), _query([4, 4], 4, n_chunks=32)]
    single = dict(_query([4], 2), axes=[2, 2], placement=[[2], [2]], card=[4])
    queries += [dict(single, reduce_axes=[0]), dict(single, axes=[4, 1], placement=[[4], [1]], reduce_axes=[1])]      # (over one device: nothing)
    together = B.p2_synthesize_batch(queries, MSG)
    for q, r in zip(queries, together):
        o = B.p2_synthesize_batch([q], MSG)[0]
        assert np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"], o["cost"])
        for key in COUNTS:
            assert r["stats"][key] == o["stats"][key], key


@pytest.mark.gpu
def test_lists_too_large_for_the_graphs():
    """A batch whose graphs would take more room than they may is evaluated by the other engines."""
    from paper_2110_10548_amd import binding as B
    q = _query([2, 2, 4, 4], 6, op_mask=1, topk=3)
    one = B.p2_synthesize_batch([q], MSG)[0]
    many = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY)] * 900, MSG)
    for r in (many[0], many[450], many[-1]):
        assert np.array_equal(r["programs"], one["programs"]) and np.array_equal(r["cost"], one["cost"])
        for key in COUNTS:
            assert r["stats"][key] == one["stats"][key], key


@pytest.mark.gpu
def test_small_spaces_beside_walked_queries():
    """Spaces just within and beyond what is walked beside a query that no graph answers: the same rows as alone."""
    from paper_2110_10548_amd import binding as B
    odd = _query([3], 3)
    graph = B.ROUTE_GRAPH
    for small, routes in (([_query([2, 16], 3)], [0]), ([_query([4, 4], 4)], [0]), ([_query([4, 8], 4)], [graph]), ([_query([2, 2, 4, 4], 2)], [graph]),
                          ([_query([2, 16], 3), _query([4, 8], 4), _query([4], 2, topk=2)], [graph] * 3), ([_query([2, 16], 3), _query([4, 4], 4), _query([4], 2, topk=2)], [0] * 3)):
        together = B.p2_synthesize_batch([odd] + small, MSG)
        assert [r["stats"]["route"] for r in together] == [0] + routes
        for q, r in zip([odd] + small, together):
            o = B.p2_synthesize_batch([q], MSG)[0]
            assert np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"], o["cost"]) and len(o["programs"]) > 0
            for key in COUNTS:
                assert r["stats"][key] == o["stats"][key], key


SIX, FIVE, FEW = _query([2] * 6, 4), _query([2] * 5, 4), _query([2, 4], 5, n_chunks=1)


@pytest.mark.gpu
@pytest.mark.parametrize("queries", [[SIX] + [FEW] * 36, [FEW] * 36 + [SIX], [SIX] * 2 + [FIVE] * 9, [FEW] * 12 + [_query([64], 5)] + [SIX] + [FEW] * 30,
                                     [_query([2] * 6, 5, form_mask=2)] + [FEW] * 520])
def test_rows_beyond_one_querys_room(queries):
    """One query has more valid programs than the call makes room for, the others fewer: in all they fit, and every row is there."""
    from paper_2110_10548_amd import binding as B
    queries = [dict(q, bw=[b * (1.0 + 0.01 * i) for b in q["bw"]]) for i, q in enumerate(queries)]
    B.p2_synthesize_batch([dict(q, bw=q["bw"][::-1], algo=1) for q in queries[::-1]], MSG)       # (other rows where these go)
    together = B.p2_synthesize_batch(queries, MSG)
    for q, r in zip(queries, together):
        o = B.p2_synthesize_batch([q], MSG)[0]
        assert len(o["programs"]) > 0 and np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"], o["cost"])


@pytest.mark.gpu
def test_stats_say_which_way_was_taken():
    """What answered a query: a graph, or another engine since the graph was asked not to be used, or had to be given up."""
    from paper_2110_10548_amd import binding as B
    routes = [B.p2_synthesize_batch([q], MSG)[0]["stats"]["route"] for q in (_query([4, 4], 4), _query([3, 4, 6], 4), _query([4, 4], 4, engine=5),
                                                                             _query([3, 4, 6], 4, frontier_pairs=2), _query([3], 3), _query([2, 2], 3, hierarchy=1))]
    assert routes == [B.ROUTE_GRAPH, B.ROUTE_GRAPH, 0, 0, 0, 0]
    q = _query([2, 2, 4, 4], 6, op_mask=1, topk=3)
    many = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY)] * 900, MSG)        # (more lists than there is room for)
    assert {r["stats"]["route"] for r in many} == {B.ROUTE_GRAPH_LEFT}


ROOM = r"""
#include "p2_plan.h"
#include <cstdio>
int main() {
    using p2::rows_at_once;
    // 1 000 queries of four levels and six instructions, eleven sizes: 83.9 million rows at most
    std::printf("%zu %zu %zu %zu %zu %zu %zu\n", rows_at_once(83920000, 262144, 11), rows_at_once(83920000, 1 << 30, 11), rows_at_once(83920, 1 << 17, 1),
                rows_at_once(83920, 100, 64), rows_at_once(83920, 1 << 17, 64), rows_at_once(110, 0, 1), rows_at_once(110, 1 << 17, 0));
}
"""


def test_room_for_rows_not_yet_counted(tmp_path):
    """Pinned memory for rows whose number is not known: no more than the caller can take, and bounded."""
    out = _compiled(tmp_path, ROOM).split()
    assert out == ["262144", "0", "83920", "100", "83920", "0", "110"]


SHORT_ROOM = r"""
#include "p2_plan.h"
#include <cstdio>
int main() {
    using namespace p2;
    const int32_t card[2] = {2, 8}, axes[1] = {16}, reduce[1] = {0};
    const p2_hierarchy h = {2, card, nullptr, nullptr};
    Plan pl;
    std::string err;
    if (make_plan(&h, axes, 1, card, reduce, 1, 3, nullptr, false, pl, err) != P2_OK) return 1;
    const size_t one = shortlist_rows_of(pl, 1024, 64);
    std::printf("%zu %zu %zu %zu\n", shortlist_rows_of(pl, 10, 11), one, rows_at_once(50 * one, 1 << 30, 64), rows_at_once(200 * one, 1 << 30, 64));
}
"""


def test_room_for_shortlists_not_yet_counted(tmp_path):
    """Shortlists of more than there can be take room for what there can be (35 programs), and pinned memory for them is bounded too."""
    assert _compiled(tmp_path, SHORT_ROOM, "p2_plan.cpp").split() == ["110", "2240", "112000", "0"]


@pytest.mark.gpu
@pytest.mark.parametrize("cap", [34, 35, 36, 86, 200])
def test_rows_as_far_as_the_caller_has_room(cap):
    """The caller's room below, at and above the rows that come out (35 of at most 110, then all of 86)."""
    from paper_2110_10548_amd import binding as B
    for q, n in ((_query([4, 4], 3), 35), (_query([4, 4], 4), 86)):
        want = B.p2_synthesize_batch([q], MSG)[0]
        assert len(want["programs"]) == n
        if cap < n:
            with pytest.raises(B.P2Error) as e:
                B.p2_synthesize_batch([q], MSG, cap=cap)
            assert e.value.code == B.P2_ENOSPC
            continue
        got = B.p2_synthesize_batch([q], MSG, cap=cap)[0]
        assert np.array_equal(got["programs"], want["programs"]) and np.array_equal(got["cost"], want["cost"]) and got["stats"]["route"] == B.ROUTE_GRAPH


@pytest.mark.gpu
def test_more_rows_expected_than_are_pinned():
    """Lists that would take more pinned memory than is taken beforehand are counted first: the same rows."""
    from paper_2110_10548_amd import binding as B
    q = _query([2, 2, 4, 4], 6, op_mask=0b00111)
    sizes = [2.0 ** 20 * (i + 1) for i in range(64)]
    many = B.p2_synthesize_batch([dict(q, bw=[b * (1 + 0.1 * i) for b in q["bw"]]) for i in range(3)], sizes, cap=3 * 83920)
    for i, r in enumerate(many):
        o = B.p2_synthesize_batch([dict(q, bw=[b * (1 + 0.1 * i) for b in q["bw"]])], sizes[::9])[0]
        assert np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"][:, ::9], o["cost"]) and r["stats"]["route"] == B.ROUTE_GRAPH


@pytest.mark.gpu
def test_little_device_memory():
    """With most of the device taken by others, large groups go without their graphs, and what these had got is given back."""
    import torch
    from paper_2110_10548_amd import binding as B
    queries = [_query(card, 6, op_mask=1) for card in ([2, 4, 8, 8], [2, 4, 4, 8], [4, 4, 4, 4], [2, 2, 8, 8])] + [_query([2, 2, 4, 4], 6, op_mask=1)]
    want = B.p2_synthesize_batch(queries, MSG)
    assert {r["stats"]["route"] for r in want} == {B.ROUTE_GRAPH}
    B.p2_release_thread()
    torch.cuda.empty_cache()
    try:
        others = torch.empty(torch.cuda.mem_get_info()[0] - (5 << 30), dtype=torch.uint8, device="cuda")
    except torch.cuda.OutOfMemoryError:
        pytest.skip("the device's free memory is not to be had in one piece")
    before = torch.cuda.mem_get_info()[0]
    got = B.p2_synthesize_batch(queries, MSG)
    held = before - torch.cuda.mem_get_info()[0]
    del others
    torch.cuda.empty_cache()
    assert [r["stats"]["route"] for r in got] == [B.ROUTE_GRAPH_LEFT] * 4 + [B.ROUTE_GRAPH] and held < 1 << 30       # (the small group keeps its own)
    again = B.p2_synthesize_batch(queries, MSG)
    for w, g, a in zip(want, got, again):
        assert np.array_equal(w["programs"], g["programs"]) and np.array_equal(w["cost"], g["cost"])
        assert np.array_equal(w["programs"], a["programs"]) and a["stats"]["route"] == B.ROUTE_GRAPH
    B.p2_release_thread()


MOST = r"""
#include "p2_plan.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
    using namespace p2;
    for (int levels = 1; levels <= 6; ++levels)
        for (int len = 1; len <= P2_MAX_LEN; ++len) {
            std::vector<int32_t> card(levels, 2);
            const int32_t axes[1] = {1 << levels}, reduce[1] = {0};
            const p2_hierarchy h = {levels, card.data(), nullptr, nullptr};
            Plan pl;
            std::string err;
            if (make_plan(&h, axes, 1, card.data(), reduce, 1, len, nullptr, false, pl, err) != P2_OK) return 1;
            std::printf("%zu ", most_valid(pl));
        }
    return 0;
}
"""


def test_expected_rows_are_what_the_oracle_counts(tmp_path, oracle):
    most = np.array(list(map(int, _compiled(tmp_path, MOST, "p2_plan.cpp").split()))).reshape(6, 7)
    for levels, upto in enumerate((7, 6, 5, 4, 4, 3), start=1):
        o = oracle.Query([2] * levels, [2 ** levels], [[2] * levels], [0]).synthesize(upto)
        for n in range(1, upto + 1):
            assert most[levels - 1, n - 1] == int(np.count_nonzero(o["len"] <= n)), (levels, n)


# levels, size limits and the states behind them (of a skeleton, whatever the sizes, those of as many levels of two: 905, 16 798, 50 275 and 29 586,
# which the devices themselves have some more of; three levels and seven instructions have none): room for all at the first attempt, rows with the evaluation
STATES = [([2, 32], 7, 42), ([2, 4, 8], 7, 1008), ([2, 2, 4, 4], 6, 16798), ([4, 2, 2, 2, 2], 5, 50275), ([2] * 6, 3, 2513), ([2] * 6, 4, 29586),
          ([12, 12], 7, 42), ([3, 4, 6], 6, 905), ([2, 3, 2, 4], 6, 16798), ([2, 2, 2, 4, 4], 5, 50275), ([2, 2, 2, 2, 2, 3], 4, 29586)]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,states", STATES)
def test_room_for_every_state(card, max_len, states):
    from paper_2110_10548_amd import binding as B
    s = B.p2_synthesize_batch([_query(card, max_len)], MSG)[0]["stats"]
    assert s["route"] == B.ROUTE_GRAPH and s["steps_evaluated"] == states * s["alphabet"]


# the same on the devices themselves, which states of masks and forms that no skeleton serves are of, and those of queries each by itself
OWN_STATES = [([2, 32], 7, 42), ([2, 4, 8], 7, 1008), ([2, 2, 4, 4], 6, 17274), ([4, 2, 2, 2, 2], 5, 50567), ([2] * 6, 3, 2513), ([2] * 6, 4, 29586),
              ([12, 12], 7, 42), ([3, 4, 6], 6, 938), ([2, 3, 2, 4], 6, 17427), ([2, 2, 2, 4, 4], 5, 50647), ([2, 2, 2, 2, 2, 3], 4, 29599)]


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,states", OWN_STATES)
def test_room_for_every_state_of_the_devices(card, max_len, states):
    from paper_2110_10548_amd import binding as B
    s = B.p2_synthesize_batch([_query(card, max_len, flags=B.FLAG_EVALUATE_EVERY_QUERY)], MSG)[0]["stats"]
    assert s["route"] == B.ROUTE_GRAPH and s["steps_evaluated"] == states * s["alphabet"]


@pytest.mark.gpu
def test_few_forms_have_no_more_rows():
    """Patterns of one form are as few as those of fewer levels, their programs are not."""
    from paper_2110_10548_amd import binding as B
    for q in (_query([2] * 5, 4, form_mask=2), _query([2, 2, 2, 4, 4], 3, form_mask=3, n_chunks=256), _query([2, 2, 2, 2, 3], 5, form_mask=3, n_chunks=48)):
        assert B.p2_synthesize_batch([q], MSG)[0]["stats"]["route"] == B.ROUTE_GRAPH


@pytest.mark.gpu
def test_no_graph_is_begun_in_vain():
    """Seven instructions of three levels are enumerated from the start, unless no AllGather can lead to a third pair."""
    from paper_2110_10548_amd import binding as B
    for card, more, route in (([3, 4, 6], {}, 0), ([2, 8, 8], dict(n_chunks=256), 0), ([3, 4, 6], dict(op_mask=0b11011), B.ROUTE_GRAPH), ([6, 12], {}, B.ROUTE_GRAPH)):
        assert B.p2_synthesize_batch([_query(card, 7, **more)], MSG)[0]["stats"]["route"] == route


@pytest.mark.gpu
@pytest.mark.parametrize("n", [40, 300, 900])
def test_rows_of_other_hierarchies_built_by_several_threads(n):
    """Batches whose queries each have bandwidth rows of their own beside some that share theirs."""
    from paper_2110_10548_amd import binding as B
    queries = []
    for i in range(n):
        q = _query([2, 2, 2], 1 + i % 2, axes=[2, 4], placement=[[2, 1, 1], [1, 2, 2]] if i % 3 else [[1, 2, 1], [2, 1, 2]], reduce_axes=[i % 2], hierarchy=(0, 1, 2, 3, 4)[i % 5])
        queries.append(dict(q, bw=[b * (1 + 0.001 * i) for b in q["bw"]]))
    together = B.p2_synthesize_batch(queries, MSG)
    for i in range(0, n, 7):
        o = B.p2_synthesize_batch([queries[i]], MSG)[0]
        assert np.array_equal(together[i]["programs"], o["programs"]) and np.array_equal(together[i]["cost"], o["cost"]) and len(o["programs"]) > 0


@pytest.mark.gpu
def test_large_groups_beside_enumerations():
    """Groups enumerated beside others that are in any case, or from graphs after them where that is less: as each by itself."""
    from paper_2110_10548_amd import binding as B
    seven = _query([3, 4, 6], 7)
    few, many = [_query([2, 8, 8], 4), _query([9, 8], 4, topk=6)], [_query([2, 4, 8, 8], 5, topk=3)]
    for queries, routes in (([seven] + few, [0] * 3), (few + [_query([3, 5, 7], 4, engine=3)], [0] * 3), ([seven] + many, [0, B.ROUTE_GRAPH])):
        together = B.p2_synthesize_batch(queries, MSG)
        assert [r["stats"]["route"] for r in together] == routes
        for q, r in zip(queries, together):
            o = B.p2_synthesize_batch([q], MSG)[0]
            assert np.array_equal(r["programs"], o["programs"]) and np.array_equal(r["cost"], o["cost"]) and len(o["programs"]) > 0
            for key in COUNTS:
                assert r["stats"][key] == o["stats"][key], key


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more", [([3, 4, 6], 5, {}), ([3, 4, 6], 6, dict(algo=1)), ([2, 2, 4, 8], 6, {}), ([2, 4, 8, 8], 5, {}), ([2, 2, 2], 7, {}), ([2, 2, 2, 2], 6, {}),
                                               ([2, 2, 2, 2, 2], 5, {})])
def test_costs_to_the_bit_whichever_way(card, max_len, more):
    """From a graph or enumerated, what AUTO hands out is the same: a query's shortlist does not depend on its batch."""
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, **more)
    a, b = (B.p2_synthesize_batch([x], MSG)[0] for x in (q, dict(q, frontier_pairs=2)))
    assert (a["stats"]["route"], b["stats"]["route"]) == (B.ROUTE_GRAPH, 0)
    assert np.array_equal(a["programs"], b["programs"]) and np.array_equal(a["cost"], b["cost"])


@pytest.mark.gpu
@pytest.mark.parametrize("card,max_len,more,route", [([2] * 5, 6, dict(form_mask=4), 5), ([2] * 6, 5, dict(form_mask=2), 9)])
def test_lists_that_were_too_short(card, max_len, more, route):
    """More states, or more rows, than was expected of so few forms: evaluated or written again with room."""
    from paper_2110_10548_amd import binding as B
    q = _query(card, max_len, **more)
    a, b = (B.p2_synthesize_batch([x], MSG)[0] for x in (q, dict(q, frontier_pairs=2)))
    assert a["stats"]["route"] == route and len(a["programs"]) > 10000          # (a graph, with its lists enlarged; with its rows written later)
    assert np.array_equal(a["programs"], b["programs"]) and np.array_equal(a["cost"], b["cost"])
