"""The graph of a skeleton (as many levels, two devices each) as p2_skeleton.hip builds it, on the CPU: what its kernels' rules say,
restated plainly, for tests to set beside the oracle.  Test infrastructure; nothing of the library is used."""
import functools
import math

AR, RS, AG, RD, BC = range(5)


@functools.lru_cache(maxsize=None)
def patterns(levels):
    """(outermost varied level, innermost one, Master) of the canonical patterns of Sec. 3.3 where every level has devices."""
    out = []
    for i in range(levels + 1):
        for lo, hi, master in [(i, levels - 1, False)] + [(j, i - 1, False) for j in range(i)] + [(j, i - 1, True) for j in range(i)]:
            p = (lo, hi, master and hi < levels - 1)
            if lo <= hi and p not in out:
                out.append(p)
    return tuple(out)


@functools.lru_cache(maxsize=None)
def groups(levels, pattern):
    """Members of the groups that take part, in ascending order: devices by number, the innermost level in the lowest bit."""
    lo, hi, master = patterns(levels)[pattern]
    inner = levels - 1 - hi
    by_group = {}
    for d in range(1 << levels):
        if not master or d & ((1 << inner) - 1) == 0:
            by_group.setdefault(d & ~(((1 << (hi - lo + 1)) - 1) << inner), []).append(d)
    return tuple(map(tuple, by_group.values()))


@functools.lru_cache(maxsize=None)
def words(levels, rows):
    """All columns of the given rows."""
    n = 1 << levels
    return sum(((1 << n) - 1) << (r * n) for r in range(n) if rows >> r & 1)


def apply(levels, state, pattern, op, sizes=None):
    """The child of a state, None where a rule fails, "goal" at the goal.  A device of a state is (masks of its rows, its rows, its chunks);
    sizes: the levels' devices, innermost first, where chunks are counted because rows do not stand for as many each."""
    n, out = 1 << levels, list(state)
    lo, hi, _ = patterns(levels)[pattern]
    g = math.prod(sizes[l] for l in range(levels - 1 - hi, levels - lo)) if sizes else 1
    changed, held_any = True, False
    for ms in groups(levels, pattern):
        own = [state[d] for d in ms]
        together, rows_all = 0, 0
        for w, r, c in own:
            if op in (AR, RS, RD) and (r != own[0][1] or together & w):
                return None                              # (equal rows, no contribution twice)
            if op == AG and (r == 0 or rows_all & r):
                return None                              # (rows of their own)
            if op == BC and w & ~own[0][0]:
                return None                              # (nothing that the root lacks)
            if op == RS and (bin(r).count("1") % len(ms) or c % g):
                return None
            together |= w
            rows_all |= r
            held_any |= r != 0
        if op == BC:
            changed &= any(w != own[0][0] for w, _, _ in own)
        held = sum(c for _, _, c in own)
        if sizes and op == AG:                           # (a digit other than zero stands for all of its level's others)
            held = [c for _, _, c in own]
            for l in range(levels - 1 - hi, levels - lo):
                held = [held[x] + held[x + 1] * (sizes[l] - 1) for x in range(0, len(held), 2)]
            held = held[0]
        for t, d in enumerate(ms):
            w, r, c = own[t]
            if op == AR:
                w = together
            elif op == RD:
                w, r, c = (together, r, c) if t == 0 else (0, 0, 0)
            elif op == AG:
                w, r, c = together, rows_all, held
            elif op == BC:
                w, r, c = own[0]
            else:
                mine = [x for x in range(n) if r >> x & 1]
                per = len(mine) // len(ms)
                r = sum(1 << x for x in mine[t * per:(t + 1) * per])
                w, c = together & words(levels, r), c // g
            out[d] = (w, r, c)
    if not changed or (op in (AR, RS, RD) and not held_any):
        return None
    full = words(levels, (1 << n) - 1)
    return "goal" if op in (AR, AG, BC) and all(w == full for w, _, _ in out) else tuple(out)


def graph(levels, max_len, sizes=None, chunks=0):
    """Nodes in the order of their distance from the start, [(digit, node, or -1 for the goal)] of each, and how many nodes each distance
    has; nothing but goals from nodes that are max_len - 1 instructions away."""
    n = 1 << levels
    start = tuple((sum(1 << (r * n + d) for r in range(n)), (1 << n) - 1, chunks) for d in range(n))
    number, edges, layer, layers = {start: 0}, [], [start], []
    for depth in range(max_len):
        layers.append(len(layer))
        found = []
        for state in layer:
            own = []
            for digit in range(5 * len(patterns(levels))):
                child = apply(levels, state, digit // 5, digit % 5, sizes)
                if child == "goal":
                    own.append((digit, -1))
                elif child is not None and depth + 1 < max_len:
                    if child not in number:
                        number[child] = len(number)
                        found.append(child)
                    own.append((digit, number[child]))
            edges.append(own)
        layer = found
    return edges, layers


def programs(edges, max_len):
    """The valid programs: tuples of pattern * 5 + operation, the digits of the whole alphabet."""
    out = []

    def walk(node, before):
        for digit, to in edges[node]:
            if to < 0:
                out.append(before + (digit,))
            elif len(before) + 2 <= max_len:
                walk(to, before + (digit,))
    walk(0, ())
    return out


def prefixes(edges, max_len):
    """How many programs of 0, 1, .. max_len - 1 instructions have all their rules hold, short of the goal."""
    out, at = [], {0: 1}
    for _ in range(max_len):
        out.append(sum(at.values()))
        behind = {}
        for node, n in at.items():
            for _, to in edges[node]:
                if to >= 0:
                    behind[to] = behind.get(to, 0) + n
        at = behind
    return out
