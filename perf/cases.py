"""What the speed of this framework is judged by: calls that its users make, from the smallest to the largest.

A case describes one call by plain values; lists are written as text ("4x8x8" a hierarchy, outermost level first;
"0,1 2" the reduce sets {0,1} and {2}).  Four kinds, one per public entry point:

  query   one placement, one reduction: p2_synthesize
  batch   many placements / reductions / chunk counts in one call, marshalled beforehand as a planner keeps them: Batch
  search  every placement x every requested reduction with its ranking: p2_search_placements
  topk    the shortlist of a cost column that is on the device already: p2_topk_device

What a call asks about (system, axes, placements, size limit) is fixed by the case; what it is asked with (link
bandwidths and latencies, message sizes, cost columns) comes from the seed.
"""
import math
import random

import numpy as np
import torch

from paper_2110_10548_amd import binding as B

# Valid programs of at most 1, 2, ... instructions by the number of levels that the reduction spans (every form and
# collective, one chunk per device): a fact of the grammar, the same for all level sizes.
VALID = {1: (1, 3, 3, 3, 3, 3), 2: (1, 5, 35, 86, 110, 110), 3: (1, 7, 80, 571, 2549, 6794), 4: (1, 9, 138, 1646, 16000, 83920)}


def _ints(text, sep="x"):
    return [int(v) for v in text.split(sep)]


def _sets(text):
    return [_ints(s, ",") for s in text.split()]


def _subsets(n):
    return [[a for a in range(n) if m >> a & 1] for m in range(1, 1 << n)]


def listed():
    return [
        # one reduction of one matrix on two nodes of four GPUs, every program listed: the smallest question there is
        dict(name="query 2x4", kind="query", card="2x4", axes="2x4", place=0, reduce="1", max_len=3, chunks=0, n_msg=1, topk=0, algo=0),
        # all 64 GPUs of four nodes of sixteen (the paper's largest system, its size limit), full list, three sizes, tree AllReduce
        dict(name="query 4x16", kind="query", card="4x16", axes="64", place=0, reduce="0", max_len=5, chunks=0, n_msg=3, topk=0, algo=1),
        # a system that is no power of two: three racks of four nodes of six GPUs, all 72 of them reduced together
        dict(name="query 3x4x6", kind="query", card="3x4x6", axes="72", place=0, reduce="0", max_len=4, chunks=0, n_msg=1, topk=10, algo=0),
        # one reduction over all of 512 GPUs, four levels, size limit 6, every valid program listed
        dict(name="query 2x4x8x8", kind="query", card="2x4x8x8", axes="512", place=0, reduce="0", max_len=6, chunks=0, n_msg=1, topk=0, algo=0),
        # every placement of two axes on 32 GPUs, two reductions, a sweep of eleven message sizes, full lists
        dict(name="batch 4x2x4", kind="batch", card="4x2x4", axes="4x8", draws=0, pick=0, reduce="0 0,1", max_len=4, chunks="0", n_msg=11, topk=0, algo=0),
        # every placement and every reduction of three axes on 64 GPUs, full lists
        dict(name="batch 2x4x8", kind="batch", card="2x4x8", axes="2x4x8", draws=0, pick=0, reduce="all", max_len=5, chunks="0", n_msg=1, topk=0, algo=0),
        # every placement of three axes on 256 GPUs, four chunk granularities, shortlists
        dict(name="batch 4x8x8", kind="batch", card="4x8x8", axes="4x8x8", draws=0, pick=0, reduce="1,2", max_len=5, chunks="1 8 64 256", n_msg=1, topk=10, algo=0),
        # 512 questions about 512 GPUs, four levels, size limit 6, shortlists: the largest
        dict(name="batch 2x4x8x8", kind="batch", card="2x4x8x8", axes="2x4x8x8", draws=512, pick=5, reduce="all", max_len=6, chunks="0", n_msg=1, topk=10, algo=0),
        # which matrix of data and model parallelism is best on four nodes of sixteen, both reductions in view
        dict(name="search 4x16", kind="search", card="4x16", axes="8x8", reduce="0 1", max_len=5),
        # the shortlist of one query's programs
        dict(name="topk 10k", kind="topk", n=10_007, k=10, cols=1),
        # one message size of three, a large query's programs
        dict(name="topk 1.3M", kind="topk", n=1_300_003, k=64, cols=3),
        # many queries' programs in one column
        dict(name="topk 50M", kind="topk", n=50_000_017, k=100, cols=1),
    ]


def draw(rng):
    kind = rng.choice(("query", "query", "query", "batch", "batch", "batch", "search", "topk", "topk"))
    if kind == "topk":
        n = int(math.exp(rng.uniform(math.log(1000), math.log(50_000_000))))
        cols = rng.choice((1, 1, 2, 3, 5))
        return dict(kind=kind, n=min(n, 50_000_000 // cols), k=int(math.exp(rng.uniform(0.0, math.log(1024)))), cols=cols)
    n_msg, algo = rng.choice((1, 1, 2, 3, 5, 11)), rng.randrange(2)
    if kind == "query":
        while True:                                         # 4 to 512 devices on two to four levels
            card = [rng.choice((2, 3, 4, 5, 6, 8, 12, 16)) for _ in range(rng.choice((2, 2, 3, 3, 4)))]
            devices = math.prod(card)
            if devices > 512:
                continue
            levels, plain = len(card), all(c & (c - 1) == 0 for c in card)
            if plain and devices <= 64:
                max_len = rng.choice((3, 4, 5) if levels <= 3 else (3, 4))
            elif levels == 4 and plain:
                max_len = 6
            else:                                           # (candidates of one query x state words: no more than "query 3x4x6")
                fits = [m for m in (3, 4, 5) if devices <= (128 if levels == 4 else 224) and (5 * levels * levels) ** m * devices * devices <= 21_740_000_000]
                if not fits:
                    continue
                max_len = rng.choice(fits)
            break
        return dict(kind=kind, card="x".join(map(str, card)), axes=str(devices), place=0, reduce="0", max_len=max_len, chunks=rng.choice((0, 0, 0, devices * 2 if devices <= 128 else 0)),
                    n_msg=n_msg, topk=rng.choice((0, 0, 1, 10, 50)), algo=algo)
    if kind == "search":
        card = [rng.choice((2, 3, 4, 6, 8)), rng.choice((4, 8, 16))]
        first = rng.choice([d for d in range(2, card[0] * card[1]) if card[0] * card[1] % d == 0])
        return dict(kind=kind, card="x".join(map(str, card)), axes="%dx%d" % (first, card[0] * card[1] // first), reduce=rng.choice(("0", "0 1", "0 1 0,1")),
                    max_len=rng.choice((3, 4)))
    shape = rng.choice(("small", "wide", "deep"))
    if shape == "deep":                                     # four levels, pruned enumeration
        card, max_len, n = rng.choice(("2x4x8x8", "4x4x4x8", "2x4x4x8", "8x4x2x4")), 6, int(math.exp(rng.uniform(math.log(4), math.log(120))))
        axes = "2x%d" % (math.prod(_ints(card)) // 2) if rng.random() < 0.3 else card
        return dict(kind=kind, card=card, axes=axes, draws=n, pick=rng.randrange(1000), reduce="all", max_len=max_len, chunks="0", n_msg=min(n_msg, 3), topk=rng.choice((1, 5, 10, 20)), algo=algo)
    if shape == "wide":                                     # several nodes, sizes of any kind
        card = [rng.choice((2, 3, 4, 5, 6)), rng.choice((2, 3, 4)), rng.choice((4, 6, 8))]
    else:
        card = [rng.choice((2, 4)), rng.choice((2, 4)), rng.choice((2, 4))]
    plain = all(c & (c - 1) == 0 for c in card) and math.prod(card) <= 64
    return dict(kind=kind, card="x".join(map(str, card)), axes="%dx%dx%d" % tuple(card), draws=rng.choice((0, rng.randrange(5, 100))), pick=rng.randrange(1000), reduce=rng.choice(("all", "0 1,2", "0,1,2 1")),
                max_len=rng.choice((3, 4, 5) if plain else (3,)), chunks=rng.choice(("0", "0", "1 0")), n_msg=n_msg, topk=rng.choice((0, 0, 10)), algo=algo)


def _links(levels, rng):
    """Bandwidth and latency of every level from the seed: inner links are the faster ones, as in real systems."""
    bw = sorted(rng.uniform(10e9, 400e9) for _ in range(levels))
    alpha = sorted((rng.uniform(1e-6, 30e-6) for _ in range(levels)), reverse=True)
    return bw, alpha


def _sizes(n_msg, rng):
    """Message sizes in bytes: powers of two from 1 MiB on, shifted by the seed (tensors are not round)."""
    return [float(int(2.0 ** (20 + i) * rng.uniform(1.0, 2.0))) for i in range(n_msg)]


def _asked(case):
    """(placement, reduce axes, chunks) of every query of a batch."""
    card, axes = _ints(case["card"]), _ints(case["axes"])
    places = B.p2_enumerate_placements(card, axes).tolist()
    sets = _subsets(len(axes)) if case["reduce"] == "all" else _sets(case["reduce"])
    chunks = _ints(case["chunks"], " ")
    if case["draws"]:
        rng = random.Random(case["pick"])
        return [(rng.choice(places), rng.choice(sets), rng.choice(chunks)) for _ in range(case["draws"])]
    return [(p, s, c) for p in places for s in sets for c in chunks]


def prepare(case, seed):
    rng = random.Random(seed)
    kind = case["kind"]
    if kind == "topk":
        g = torch.Generator(device="cuda").manual_seed(seed)
        n, cols = case["n"], case["cols"]
        # simulated times: a broad positive distribution in which many programs share a value exactly
        cost = torch.exp(torch.randn(n * cols, generator=g, device="cuda", dtype=torch.float64))
        cost = (cost * 65536.0).round() / 65536.0e3
        # candidate indices in ascending order, with gaps
        index = torch.cumsum(torch.randint(1, 4000, (n,), generator=g, device="cuda", dtype=torch.int64), 0)
        torch.cuda.synchronize()
        return dict(kind=kind, n=n, k=case["k"], cols=cols, cost=cost, index=index, pos=torch.zeros(min(case["k"], n), dtype=torch.int64, device="cuda"))
    card, axes = _ints(case["card"]), _ints(case["axes"])
    bw, alpha = _links(len(card), rng)
    if kind == "search":
        return dict(kind=kind, args=(card, axes, _sets(case["reduce"]), case["max_len"], _sizes(1, rng)[0]), more=dict(bw=bw, alpha=alpha))
    msg = _sizes(case["n_msg"], rng)
    if kind == "query":
        place = B.p2_enumerate_placements(card, axes)[case["place"]].tolist()
        return dict(kind=kind, args=(card, axes, place, _ints(case["reduce"], ","), case["max_len"], msg),
                    more=dict(bw=bw, alpha=alpha, n_chunks=case["chunks"], topk=case["topk"], algo=case["algo"]))
    queries = [dict(card=card, bw=bw, alpha=alpha, axes=axes, placement=p, reduce_axes=s, max_len=case["max_len"], n_chunks=c, topk=case["topk"], algo=case["algo"])
               for p, s, c in _asked(case)]
    return dict(kind=kind, batch=B.Batch(queries, msg))


def run(state):
    kind = state["kind"]
    if kind == "topk":
        cost, cols = state["cost"], state["cols"]
        B.p2_topk_device(cost.data_ptr() + 8 * (cols - 1), cols, state["index"].data_ptr(), state["n"], state["k"], state["pos"].data_ptr())
        return state["pos"]
    if kind == "query":
        r = B.p2_synthesize(*state["args"], **state["more"])
        return {"index": r["programs"]["index"], "instr": r["programs"]["instr"], "len": r["programs"]["len"], "cost": r["cost"], "valid": r["stats"]["valid"],
                "candidates": r["candidates"]}
    if kind == "batch":
        results = state["batch"].run()
        programs = np.concatenate([r["programs"] for r in results])
        return {"index": programs["index"], "instr": programs["instr"], "len": programs["len"], "cost": np.concatenate([r["cost"] for r in results]),
                "valid": np.array([r["stats"]["valid"] for r in results])}
    r = B.p2_search_placements(*state["args"], **state["more"])
    rows = [r["rows"][key] for key in sorted(r["rows"])]
    return {"order": np.array(r["order"]), "total": np.array(r["total"]), "best": np.array([row["best_cost"] for row in rows]),
            "program": np.array([-1 if row["best_index"] is None else row["best_index"] for row in rows]),
            "allreduce": np.array([row["allreduce_cost"] for row in rows]), "valid": np.array([row["valid"] for row in rows])}


def _of_queries(card, asked, max_len, n_msg, topk):
    """Bytes and operations that a list of (placement, reduce axes, chunks) cannot do without.  Bytes: each query's
    description in, the rows it asks for out (a program is 16 bytes, a cost 8).  Operations: per distinct reduction
    structure every valid program's last instruction applied once to the state it meets (the chunk set and the mask of
    each device, a word at a time: read, combine, test, write), and per query two per cost (alpha and beta term)."""
    nbytes, ops, seen = 0.0, 0.0, set()
    for place, axes, chunks in asked:
        sizes = tuple(s for s in (math.prod(place[a][j] for a in axes) for j in range(len(card))) if s > 1)
        nbytes += 16.0 * len(card) + 4.0 * sum(len(row) for row in place) + 64.0
        if not sizes:
            continue
        valid = VALID[len(sizes)][min(max_len, 6) - 1]
        group = math.prod(sizes)
        k = chunks or math.prod(card)
        nbytes += (16.0 + 8.0 * n_msg) * (min(topk, valid) * n_msg if topk else valid)
        ops += 2.0 * valid * n_msg
        if (sizes, k) not in seen:
            seen.add((sizes, k))
            ops += 4.0 * valid * group * (-(-k // 32) + -(-group // 32))
    return {"bytes": nbytes, "flops": ops}


def work(case):
    if case["kind"] == "topk":
        # every cost once (a strided column is fetched with its neighbours), the indices of what is picked; a comparison each
        return {"bytes": 8.0 * case["n"] * case["cols"] + 16.0 * min(case["k"], case["n"]), "flops": float(case["n"])}
    card, axes = _ints(case["card"]), _ints(case["axes"])
    if case["kind"] == "query":
        place = B.p2_enumerate_placements(card, axes)[case["place"]].tolist()
        return _of_queries(card, [(place, _ints(case["reduce"], ","), case["chunks"])], case["max_len"], case["n_msg"], case["topk"])
    if case["kind"] == "batch":
        return _of_queries(card, _asked(case), case["max_len"], case["n_msg"], case["topk"])
    asked = [(p, s, 0) for p in B.p2_enumerate_placements(card, axes).tolist() for s in _sets(case["reduce"])]
    return _of_queries(card, asked, case["max_len"], 1, 1)


def tolerance(case):
    """Positions and programs are whole numbers and costs are sums of a few dozen positive terms in 64 bits: engines that
    add them in another order differ in the last bits, and then programs of equal cost may swap places in a shortlist."""
    if case["kind"] == "topk":
        return "exact"
    return {"rel": 1e-14, "max": 1e-13, "differ": 0.005}
