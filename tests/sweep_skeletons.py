"""Every list of levels that is answered from a skeleton's graph, beside the graphs of the devices themselves (or, where these cannot hold it,
the enumeration): programs, counts and costs to the bit.  Not collected with the tests, for it takes minutes of a GPU:

    python tests/sweep_skeletons.py whole [part of parts]      15 407 lists, one chunk for every device, at the largest size limit and at a smaller one
    python tests/sweep_skeletons.py split [part of parts]      lists of up to four levels, every number of chunks that divides the devices and one that does not
"""
import math
import os
import random
import sys
import time

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
from paper_2110_10548_amd import binding as B  # noqa: E402

MOST = {1: 7, 2: 7, 3: 6, 4: 6, 5: 5, 6: 4}              # the size limits up to which skeletons are used, by levels
ROWS = {1: 3, 2: 110, 3: 6794, 4: 83920, 5: 44182, 6: 6423}      # valid programs at these
MSG = [2.0 ** 20, 3.0e8]
COUNTS = ("candidates", "valid", "group_size", "alphabet")
STEPS = ("steps_executed", "member_visits")              # (an enumeration adds what it applies again to rebuild a prefix)


def lists(levels, devices=512):
    if levels == 0:
        return [[]]
    return [[first] + rest for first in range(2, devices + 1) for rest in lists(levels - 1, devices // first)]


def query(card, max_len, chunks, rng):
    n, L = math.prod(card), len(card)
    return dict(card=card, axes=[n], placement=[card], reduce_axes=[0], max_len=max_len, n_chunks=chunks, algo=rng.randrange(2),
                bw=[rng.uniform(1e9, 4e11) for _ in range(L)], alpha=[rng.uniform(1e-6, 3e-5) for _ in range(L)])


def compare(queries, cap):
    """How many were answered from a skeleton's graph."""
    together = B.p2_synthesize_batch(queries, MSG, cap=cap)
    # (a call of which some queries are walked has others walked beside them: those by themselves)
    for i, r in enumerate(together):
        if not r["stats"]["route"] & B.ROUTE_GRAPH:
            together[i] = B.p2_synthesize_batch(queries[i:i + 1], MSG, cap=cap)[0]
    apart = B.p2_synthesize_batch([dict(q, flags=B.FLAG_EVALUATE_EVERY_QUERY) for q in queries], MSG, cap=cap)
    for q, a, b in zip(queries, together, apart):
        keys = COUNTS + (STEPS if b["stats"]["route"] & B.ROUTE_GRAPH or not a["stats"]["route"] & B.ROUTE_GRAPH else ())
        if not (np.array_equal(a["programs"], b["programs"]) and np.array_equal(a["cost"], b["cost"])) or any(a["stats"][k] != b["stats"][k] for k in keys):
            raise SystemExit("differs: %r\n%r\n%r" % (q, a["stats"], b["stats"]))
    return sum(1 for r in together if r["stats"]["route"] & B.ROUTE_GRAPH)


def main(what, part, parts):
    rng, t0, said, n, graphs, at = random.Random(part), time.time(), time.time(), 0, 0, 0
    for levels in range(1, 7 if what == "whole" else 5):
        # (a batch: groups of one skeleton; not more of four levels than their own devices' graphs have memory for)
        size = {1: 64, 2: 48, 3: 24, 4: 6, 5: 3, 6: 6}[levels]
        asked = []
        for card in lists(levels):
            R = math.prod(card)
            chunks = [R] if what == "whole" else [k for k in range(1, R) if R % k == 0] + [rng.choice([k for k in range(1, 513) if k % R != 0 and math.gcd(k, R) > 1] or [1])]
            for k in chunks:
                asked.append((card, k))
        rng2 = random.Random(levels)
        rng2.shuffle(asked)
        asked = asked[part::parts]
        for limits in ("largest", "smaller"):
            for i in range(0, len(asked), size):
                queries, limit = asked[i:i + size], MOST[levels] if limits == "largest" else rng.randrange(1, MOST[levels])
                graphs += compare([query(c, limit, k, rng) for c, k in queries], ROWS[levels] * len(queries))
                n += len(queries)
                if time.time() - said > 20:
                    said = time.time()
                    print("%s %d/%d: %d levels, %s limit, %d of %d; %d queries, %d from graphs, %.0f s" % (what, part, parts, levels, limits, i, len(asked), n, graphs, said - t0), flush=True)
    print("%s %d/%d: %d queries, %d from graphs, all the same, %.0f s" % (what, part, parts, n, graphs, time.time() - t0), flush=True)


if __name__ == "__main__":
    main(sys.argv[1], *(map(int, sys.argv[2:4]) if len(sys.argv) > 3 else (0, 1)))
