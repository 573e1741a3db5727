// State-graph engine: reduction groups of at most 64 devices with power-of-two patterns, every candidate space.
//
// What the rules of Sec. 3.2 say about the next instruction depends on the state alone, and the programs of a
// query pass through very few distinct states (64 devices, instructions of three levels, size limit 5: 739 states
// behind 1.9 * 10^8 candidates; four levels, size limit 6: 17 274 behind 2.7 * 10^11).  The engine therefore builds the
// graph of the states once per reduction structure and answers everything from it:
//
//   nodes   the distinct states that are not the goal, each found once over all lengths (a hash proposes an equal
//           state, a comparison of every device decides; were two states to share a 64-bit hash, the call would say so
//           and be evaluated by the other engines);
//   edges   (state, instruction) pairs that satisfy the instruction's rule, to another state or to the goal;
//   counts  per node the programs of exactly r more instructions that end at the goal, and that are valid without
//           ending there: every number of a query's list and stats follows from the counts of the first node;
//   rows    the t-th valid program in ascending candidate index is read off the counts (a walk along the edges in the
//           order of the digits), so the list comes out in order, each row by a thread of its own;
//   costs   what a step adds to the two sums of the cost model depends on its edge and on the query's links: worked
//           out once per (edge on the way to a goal, query), then added up along each program in program order.
//
// A device holds (chunk set, mask) pairs, one to start with, more where an AllGather joins chunks with different
// contributions; up to two are kept, four from a size limit of six on (no structure that was enumerated needs more), and a
// device that would need more is reported.  Chunks that every rule treats alike are held as one: with a multiple of R chunks a row stands
// for a block of k / R consecutive ones.  A ReduceScatter deals blocks out, so this is exact unless it had to cut one
// in two; that is checked at every ReduceScatter and reported as well.  What is reported is evaluated by the other
// engines.
//
// What follows a state depends on the levels and not on how many devices each has (has_skeleton in p2_api.hip says how far
// and how that was checked), so the graph is that of the skeleton, two devices a level: two to 64 devices, whatever the sizes,
// and one graph for all structures of as many levels in a call.  [2 4 8 8], 512 devices, six instructions: 3 740 us with its
// own devices, 1 300 so; 512 queries of it, 48 structures: 15.5 ms and 3.5.  Groups that no skeleton is used for are evaluated
// on their own devices, and those among them that are larger or have other patterns bring their edges from the frontier's
// kernels (p2_frontier.hip) and are counted, costed and listed here.
#include "p2_graph_dev.h"

namespace p2 {

namespace {

constexpr int kMostPairs = 4;
constexpr uint32_t kChunk = 8;          // planes a wavefront reserves at a time (a returning addition to one address takes some 10 ns)
constexpr uint32_t kPlaneMask = 0x0fffffffu;
// a structure of one or two levels has at most 42 states and 93 edges
constexpr uint32_t kAloneSlots = 256, kAloneNodes = 96, kAlonePlanes = 112, kAloneFound = 160, kAloneScratch = 512;

// The edges a wavefront has found and not yet written to the lists.
struct Found {
    u64 hash[kWave];                    // of the child's state; 0: the goal
    u64 path[kWave];                    // instructions that lead to the child
    uint32_t state[kWave], from[kWave]; // child: plane | pairs << 28; node | digit << 23
};
// What a block that works on a graph alone keeps with it instead of in device memory.
struct AloneShared {
    u64 table[kAloneSlots];
    uint32_t table_node[kAloneSlots];
    u64 found[P2_MAX_LEN + 1];
    uint32_t n_planes, flags;
    uint32_t node_state[kAloneNodes], use_id[kAloneNodes];
    u64 node_path[kAloneNodes];
    uint4 edges[kAloneFound];
    uint2 links[kAloneFound];
};

// A description of a graph for a kernel to work with: a copy, so that the kernel's stores do not make it read again, with
// pointers to the global address space.
// The lists that a graph is worked out in: device memory, or the LDS of the one block that does it.
struct InDevice {
    using planes = P2_GLOBAL u64x2*; using words = P2_GLOBAL uint32_t*; using found = P2_GLOBAL u32x4*; using links = P2_GLOBAL u32x2*; using paths = P2_GLOBAL u64*;
};
struct InBlock {
    using planes = P2_LOCAL u64x2*; using words = P2_LOCAL uint32_t*; using found = P2_LOCAL u32x4*; using links = P2_LOCAL u32x2*; using paths = P2_LOCAL u64*;
};
template <class Where>
struct Graph {
    uint32_t query;
    int R, rows_kept, n_pat, n_ops, alphabet, max_len, W, n_members;
    uint32_t op_mask, op_ranks, split_check;
    bool links_ready, skeleton;
    P2_GLOBAL const u32x4* large[2];
    int wq, qk;
    uint32_t cap_nodes, cap_planes, cap_found, cap_edges, table_mask;
    u64 all_rows, all_cols;
    P2_GLOBAL GraphCounters* ctr;
    P2_GLOBAL u64* table;
    typename Where::words table_node, node_state, use_id;
    typename Where::planes planes;
    typename Where::found found;
    typename Where::links links;
    typename Where::paths node_path;
    P2_GLOBAL u64* edge_path;
    P2_GLOBAL u64x2* planes_out;
    P2_GLOBAL u32x2* first_edge;
    P2_GLOBAL uint32_t *use_ends, *edges, *edge_state;
    P2_GLOBAL double* best;
    P2_GLOBAL const int32_t* members;
};
template <class Where>
__device__ __forceinline__ void open_graph(Graph<Where>& G, const DevGraph& D) {
    G.query = D.query; G.R = D.R; G.rows_kept = D.rows_kept; G.n_pat = D.n_pat; G.n_ops = D.n_ops; G.alphabet = D.alphabet;
    G.max_len = D.max_len; G.W = D.digit_words; G.n_members = D.n_members;
    G.op_mask = D.op_mask; G.op_ranks = D.op_ranks; G.split_check = D.split_check;
    G.cap_nodes = D.cap_nodes; G.cap_planes = D.cap_planes; G.cap_found = D.cap_found; G.cap_edges = D.cap_edges; G.table_mask = D.table_mask;
    G.all_rows = D.all_rows; G.all_cols = D.all_cols;
    G.links_ready = D.large[0] != nullptr; G.skeleton = D.sizes != nullptr; G.wq = D.wq; G.qk = D.qk;
    G.large[0] = in_global<const u32x4>(D.large[0]); G.large[1] = in_global<const u32x4>(D.large[1]);
    G.ctr = in_global<GraphCounters>(D.ctr); G.table = in_global<u64>(D.table);
    G.planes_out = in_global<u64x2>(D.planes); G.edge_path = in_global<u64>(D.edge_path);
    G.first_edge = in_global<u32x2>(D.first_edge); G.use_ends = in_global<uint32_t>(D.use_ends);
    G.edges = in_global<uint32_t>(D.edges); G.edge_state = in_global<uint32_t>(D.edge_state);
    G.best = in_global<double>(D.best); G.members = in_global<const int32_t>(D.members);
}
__device__ __forceinline__ Graph<InDevice> open_in_device(const DevGraph& D) {
    Graph<InDevice> G;
    open_graph(G, D);
    G.table_node = in_global<uint32_t>(D.table_node); G.node_state = in_global<uint32_t>(D.node_state); G.use_id = in_global<uint32_t>(D.use_id);
    G.planes = in_global<u64x2>(D.planes); G.found = in_global<u32x4>(D.found); G.links = in_global<u32x2>(D.links);
    G.node_path = in_global<u64>(D.node_path);
    return G;
}
__device__ __forceinline__ Graph<InBlock> open_in_block(const DevGraph& D, AloneShared& A, u64x2* planes) {
    Graph<InBlock> G;
    open_graph(G, D);
    G.table_node = (P2_LOCAL uint32_t*)A.table_node; G.node_state = (P2_LOCAL uint32_t*)A.node_state; G.use_id = (P2_LOCAL uint32_t*)A.use_id;
    G.planes = (P2_LOCAL u64x2*)planes; G.found = (P2_LOCAL u32x4*)A.edges; G.links = (P2_LOCAL u32x2*)A.links;
    G.node_path = (P2_LOCAL u64*)A.node_path;
    if (G.cap_nodes > kAloneNodes) G.cap_nodes = kAloneNodes;
    if (G.cap_planes > kAlonePlanes) G.cap_planes = kAlonePlanes;
    if (G.cap_found > kAloneFound) G.cap_found = kAloneFound;
    return G;
}
__device__ __forceinline__ uint32_t add_global(P2_GLOBAL uint32_t* p, uint32_t v) { return atomicAdd((uint32_t*)p, v); }
__device__ __forceinline__ u64 add_global(P2_GLOBAL u64* p, u64 v) { return atomicAdd((u64*)p, v); }
__device__ __forceinline__ u64 shfl64(u64 v, int src) { return __shfl(v, src, kWave); }

__device__ __forceinline__ u64 lowest64(u64 x, int n) {
    const Words<2> w{{(uint32_t)x, (uint32_t)(x >> 32)}};
    const Words<2> o = lowest_n(w, n);
    return (u64)o.w[0] | ((u64)o.w[1] << 32);
}

// One device's pairs: disjoint chunk sets, distinct masks, empty pairs (0, 0) last, the pair with the lowest chunk first.
template <int kPairs>
struct Pairs {
    u64 r[kPairs], m[kPairs];
};
template <int kPairs>
__device__ __forceinline__ u64 rows_of(const Pairs<kPairs>& a) {
    u64 o = 0;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) o |= a.r[i];
    return o;
}
// rows x with mask m to `a`; true if there is no room for another mask
template <int kPairs>
__device__ __forceinline__ bool add_pair(Pairs<kPairs>& a, u64 x, u64 m) {
    bool left = x != 0ull;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
        const bool here = left && (a.r[i] == 0ull || a.m[i] == m);
        if (here) { a.r[i] |= x; a.m[i] = m; }
        left = left && !here;
    }
    return left;
}
template <int kPairs>
__device__ __forceinline__ void order_pairs(Pairs<kPairs>& a) {
    static_assert(kPairs == 2 || kPairs == 4, "sorts two or four");
    auto key = [](u64 r) { return r == 0ull ? 64 : __ffsll((long long)r) - 1; };
    auto swap_if = [&](int i, int j) {
        const bool sw = key(a.r[j]) < key(a.r[i]);
        const u64 r = a.r[i], m = a.m[i];
        a.r[i] = sw ? a.r[j] : r; a.m[i] = sw ? a.m[j] : m;
        a.r[j] = sw ? r : a.r[j]; a.m[j] = sw ? m : a.m[j];
    };
    swap_if(0, 1);
    if constexpr (kPairs == 4) { swap_if(2, 3); swap_if(0, 2); swap_if(1, 3); swap_if(1, 2); }
}

// The lanes that hold one state: lane `base + d` plays device d.
struct Team {
    int lane, dev, base;
    u64 mask;
    __device__ __forceinline__ bool any(bool x) const { return (__ballot(x) & mask) != 0ull; }
};

// AllReduce's union on states with several pairs: per row the masks of the group's members, which must be disjoint.
// bad: rows held twice with a contribution in common, or chunk sets that differ; full: a device needs too many pairs.
template <int kPairs>
__device__ __forceinline__ void unite_pairs(Pairs<kPairs>& acc, const Team& t, bool in, int lg, int ls, bool& bad, bool& full) {
    for (int s = 0; __any(s < lg); ++s) {
        const bool act = in && s < lg;
        const int src = s < lg ? (t.lane ^ (1 << (ls + s))) : t.lane;
        Pairs<kPairs> other, to;
#pragma unroll
        for (int i = 0; i < kPairs; ++i) { other.r[i] = shfl64(acc.r[i], src); other.m[i] = shfl64(acc.m[i], src); to.r[i] = 0ull; to.m[i] = 0ull; }
        if (act) {
            bad |= rows_of(acc) != rows_of(other);
#pragma unroll
            for (int i = 0; i < kPairs; ++i)
#pragma unroll
                for (int j = 0; j < kPairs; ++j) {
                    const u64 x = acc.r[i] & other.r[j];
                    bad |= x != 0ull && (acc.m[i] & other.m[j]) != 0ull;
                    full |= add_pair(to, x, acc.m[i] | other.m[j]);
                }
            acc = to;
        }
    }
}

// What the rules say about one pattern on one state, and what the children are made of.
struct Verdict {
    uint32_t kids, goals;               // by op: the rule holds and the child is not the goal; it is the goal
    u64 ru, mu, rr, rm;                 // union of the group's rows and masks, the root's rows and mask (of a state with one pair)
    bool m_differs;                     // some member's mask differs (AllGather then leaves several pairs)
};

// A state and a pattern are judged by the R lanes of a team together; one walk over the bits of the group number serves
// the AllReduce-like rules and AllGather (`union == both sides` at every bit iff all members are equal, `no overlap` at every
// bit iff they are pairwise disjoint), and ends as soon as both have failed, as for nine in ten pairs at the first or second
// bit; Broadcast takes one exchange with the root.
template <int kPairs, class Where>
__device__ __forceinline__ void judge(Verdict& V, const Graph<Where>& G, const Team& t, const Pairs<kPairs>& st, int np, bool active, uint32_t shape, u64 part,
                                      bool last, uint32_t& flags) {
    const int lg = (int)(shape & 15u), ls = (int)((shape >> 4) & 15u);
    const int gm1 = (1 << lg) - 1, gmask = gm1 << ls;
    const bool in = ((part >> t.dev) & 1ull) != 0ull;
    const u64 all_r = G.all_rows, all_m = G.all_cols;
    const int root = t.base | (t.dev & ~gmask);
    const u64 r = rows_of(st), m = st.m[0];
    u64 ru = r, mu = m;
    const bool some = t.any(in && r != 0ull);
    // (lane flags; a rule has failed when any lane of the team says so)
    bool ar_bad = !some || !active, ag_bad = (in && r == 0ull) || !active, m_differs = false;
    bool ar = true, ag = true;
    for (int s = 0; __any(s < lg); ++s) {
        const bool act = in && s < lg;
        const int src = s < lg ? (t.lane ^ (1 << (ls + s))) : t.lane;
        const u64 pr = shfl64(ru, src), pm = shfl64(mu, src);
        if (act) {
            ar_bad |= pr != ru || (np == 1 && (pm & mu) != 0ull);
            ag_bad |= (pr & ru) != 0ull;
            m_differs |= pm != mu;
            ru |= pr; mu |= pm;
        }
        ar = !t.any(ar_bad); ag = !t.any(ag_bad);
        if (!__any(ar || ag)) break;
    }
    V.ru = ru; V.mu = mu; V.rr = 0ull; V.rm = 0ull; V.m_differs = false; V.kids = V.goals = 0u;
    V.rr = shfl64(r, root); V.rm = shfl64(m, root);
    bool bc_bad = !active || (in && ((r & ~V.rr) != 0ull || (np == 1 && (m & ~V.rm) != 0ull)));
    bool bc = !t.any(bc_bad);
    if (!__any(ar || ag || bc)) return;
    const bool r_short = t.any(r != all_r);
    uint32_t kids = 0u, goals = 0u;
    bool several_short = true;
    if (np > 1 && ar) {
        ar = !(last && r_short);                         // (only a goal counts then, and an AllReduce leaves the rows as they are)
        if (ar) {
            bool bad = false, full = false;
            Pairs<kPairs> acc = st;
            unite_pairs(acc, t, in, lg, ls, bad, full);
            ar = !t.any(bad);
            if (ar && t.any(full)) flags |= kGraphPairs;
            several_short = acc.r[1] != 0ull || acc.m[0] != all_m;
        }
    }
    if (ar) {
        const bool short_m = np == 1 ? (in ? mu : m) != all_m : several_short;
        const bool uneven = in && (__popcll(r) & gm1) != 0;
        const bool rs = !t.any(uneven);
        if (G.split_check && !rs) flags |= kGraphSplit;
        if (!r_short && !t.any(short_m)) goals |= 1u << OP_AR;
        kids |= (1u << OP_AR) | (1u << OP_RD) | (rs ? 1u << OP_RS : 0u);
    }
    if (ag) {
        V.m_differs = t.any(m_differs) || np > 1;
        if (!V.m_differs && !t.any(m != all_m) && !t.any((in ? ru : r) != all_r)) goals |= 1u << OP_AG;
        kids |= 1u << OP_AG;
    }
    if (bc) {
        bool diff = in && (r != V.rr || m != V.rm), own_short = r != all_r || m != all_m || st.r[1] != 0ull;
        bool root_short = V.rm != all_m;
        if (np > 1) {
            Pairs<kPairs> q;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) { q.r[i] = shfl64(st.r[i], root); q.m[i] = shfl64(st.m[i], root); }
            bool bad = false;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                diff = diff || (in && (st.r[i] != q.r[i] || st.m[i] != q.m[i]));
#pragma unroll
                for (int j = 0; j < kPairs; ++j) bad = bad || (in && (st.r[i] & q.r[j]) != 0ull && (st.m[i] & ~q.m[j]) != 0ull);
            }
            bc = !t.any(bad);
            root_short = q.r[1] != 0ull || q.m[0] != all_m;
        }
        // in every group some member must differ from the root
        u64 told = __ballot(diff) & t.mask;
        for (int s = 0; s < lg; ++s) told |= told >> (1u << (ls + s));
        const bool idle = in && (t.dev & gmask) == 0 && ((told >> t.lane) & 1ull) == 0ull;
        bc = bc && !t.any(idle);
        if (bc) {
            kids |= 1u << OP_BC;
            if (!t.any(in ? (V.rr != all_r || root_short) : own_short)) goals |= 1u << OP_BC;
        }
    }
    V.goals = goals & G.op_mask;
    V.kids = last ? 0u : kids & ~goals & G.op_mask;
}

// The child of a state under an instruction whose rule holds.
template <int kPairs>
__device__ __forceinline__ bool make_child(Pairs<kPairs>& st, const Verdict& V, const Team& t, int np, uint32_t shape, u64 part, int op) {
    const int lg = (int)(shape & 15u), ls = (int)((shape >> 4) & 15u);
    const int gm1 = (1 << lg) - 1, gmask = gm1 << ls;
    const bool in = ((part >> t.dev) & 1ull) != 0ull;
    bool full = false;
    if (op == OP_BC) {
        if (np == 1) {
            if (in) { st.r[0] = V.rr; st.m[0] = V.rm; }
            return false;
        }
        const int root = t.base | (t.dev & ~gmask);
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const u64 rr = shfl64(st.r[i], root), rm = shfl64(st.m[i], root);
            if (in) { st.r[i] = rr; st.m[i] = rm; }
        }
        return false;
    }
    if (op == OP_AG) {
        if (!V.m_differs) {
            if (in) st.r[0] = V.ru;
            return false;
        }
        for (int s = 0; __any(s < lg); ++s) {
            const int src = s < lg ? (t.lane ^ (1 << (ls + s))) : t.lane;
            Pairs<kPairs> other;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) { other.r[i] = shfl64(st.r[i], src); other.m[i] = shfl64(st.m[i], src); }
            if (in && s < lg) {
#pragma unroll
                for (int i = 0; i < kPairs; ++i) full |= add_pair(st, other.r[i], other.m[i]);
            }
        }
        order_pairs(st);
        return full;
    }
    if (np == 1) {
        if (in) st.m[0] = V.mu;
    } else {
        bool bad = false;
        unite_pairs(st, t, in, lg, ls, bad, full);
    }
    if (in && op == OP_RS) {
        // the member of rank p keeps the p-th block of the rows in ascending order
        const u64 all = rows_of(st);
        const int per = __popcll(all) >> lg, p = (t.dev >> ls) & gm1;
        const u64 mine = lowest64(all, (p + 1) * per) & ~lowest64(all, p * per);
        if (np == 1) {
            st.r[0] = mine;
        } else {
            const Pairs<kPairs> from = st;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) { st.r[i] = 0ull; st.m[i] = 0ull; }
#pragma unroll
            for (int i = 0; i < kPairs; ++i) full |= add_pair(st, from.r[i] & mine, from.m[i]);
        }
    } else if (in && op == OP_RD && (t.dev & gmask) != 0) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) { st.r[i] = 0ull; st.m[i] = 0ull; }
    }
    // (pairs in the order of their lowest rows)
    if (np > 1) order_pairs(st);
    return full;
}

__device__ __forceinline__ u64 mix(u64 r, u64 m, uint32_t where) {
    u64 x = (r + 0x5851f42d4c957f2dull * (where + 1u)) * 0xd1342543de82ef95ull;
    x ^= x >> 31;
    x = (x ^ (m + (m << 21) + (m >> 35))) * 0xaf251af3b0f025b5ull;
    x ^= x >> 28;
    x *= 0xb564ef22ec7aece5ull;
    return x ^ (x >> 32);
}

// One level of one graph by wavefront w of nw: the states first reached by `level` instructions are judged against every
// pattern, a team of R lanes per (state, pattern), and the children of what holds are built and looked up.  The wavefronts
// do not meet: each collects the edges it finds and writes them to the lists some dozens at a time, so that a level is one
// chain of a few round trips however few its states are (a look at the hash table, a place in the lists).  The wavefronts
// at the other end compare the children that the level before found to have the hash of an earlier state with that state.
template <int kPairs, class Where>
__device__ void graph_level(const Graph<Where>& G, const uint32_t* shape, const u64* part, int level, uint32_t w, uint32_t nw, Found& F, AloneShared* A) {
    constexpr bool ALONE = std::is_same<Where, InBlock>::value;
    const int R = G.R, n_pat = G.n_pat;
    Team t;
    t.lane = (int)threadIdx.x & (kWave - 1);
    t.dev = t.lane & (R - 1);
    t.base = t.lane & ~(R - 1);
    t.mask = R >= 64 ? ~0ull : ((1ull << R) - 1ull) << t.base;
    const uint32_t teams = (uint32_t)(kWave / R), team = (uint32_t)(t.base / R);
    u64 leaders = 1ull;                                  // lanes that speak for their teams
    for (int x = R; x < kWave; x <<= 1) leaders |= leaders << x;
    P2_GLOBAL GraphCounters* const ctr = G.ctr;
    const bool last = level + 1 >= G.max_len;
    // (the counts of this level do not change while it is worked on; a list that has outgrown its room, which the call
    //  will say and repeat, is read as far as it was written)
    uint32_t first = 0, count = 1, edge0 = 0, edges = 0;   // the level's nodes; the edges that led to them
    if (level > 0) {
        first = 1;
        for (int l = 1; l <= level; ++l) {
            const u64 f = ALONE ? A->found[l] : ctr->found[l];
            if (l < level) first += (uint32_t)f; else count = (uint32_t)f;
            edge0 += edges;
            edges = (uint32_t)(f >> 32);
        }
    }
    const uint32_t next_first = first + count, next_edge = edge0 + edges;
    if (first > G.cap_nodes) first = G.cap_nodes;
    if (count > G.cap_nodes - first) count = G.cap_nodes - first;
    if (edge0 > G.cap_found) edge0 = G.cap_found;
    if (edges > G.cap_found - edge0) edges = G.cap_found - edge0;
    // at the size limit only goals count: a team takes a state, and several patterns of the few from which one can end there
    // (as many patterns at a time as leave every team a turn or two: they are judged one after the other)
    uint32_t pats = 1u;
    if (last) {
        pats = (count * (uint32_t)n_pat + 2u * nw * teams - 1u) / (2u * nw * teams);
        pats = pats < 1u ? 1u : pats > (uint32_t)n_pat ? (uint32_t)n_pat : pats;
    }
    const uint32_t per_node = ((uint32_t)n_pat + pats - 1u) / pats, items = count * per_node;
    uint32_t flags = 0u;
    for (uint32_t e = (nw - 1u - w) * teams + team; e < edges; e += nw * teams) {
        const u32x4 mine = G.found[edge0 + e];           // (node | digit << 23, slot, state, 1: the first with its hash)
        if (mine.w != 0u) continue;
        const uint32_t node = G.table_node[mine.y];
        if (node == 0u || node > G.cap_nodes) { flags |= kGraphFull; continue; }
        const uint32_t other = G.node_state[node - 1u];
        bool differ = (mine.z >> 28) != (other >> 28);
        if (!differ) {
            const typename Where::planes a = G.planes + (size_t)(mine.z & kPlaneMask) * R;
            const typename Where::planes b = G.planes + (size_t)(other & kPlaneMask) * R;
            for (uint32_t p = 0; p < (mine.z >> 28); ++p) {
                const u64x2 x = a[(size_t)p * R + t.dev], y = b[(size_t)p * R + t.dev];
                differ |= x.x != y.x || x.y != y.y;
            }
        }
        if (differ) flags |= kGraphCollision;
    }
    uint32_t n_found = 0;                                // (wave-uniform)
    uint32_t chunk = 0, chunk_left = 0;
    auto more_planes = [&](uint32_t n) {                 // places of n planes, by one lane
        return (ALONE ? atomicAdd(&A->n_planes, n) : add_global(&ctr->n_planes, n)) + 1u;      // (plane 0 is the first state's)
    };
    // the edges found so far to the lists, a lane each
    auto put_found = [&]() {
        if (n_found == 0u) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const bool mine = (uint32_t)t.lane < n_found;
        const u64 h = mine ? F.hash[t.lane] : 0ull;
        const uint32_t state = mine ? F.state[t.lane] : 0u, from = mine ? F.from[t.lane] : 0u;
        const u64 path = mine ? F.path[t.lane] : 0ull;
        const uint32_t slots = ALONE ? kAloneSlots - 1u : G.table_mask;
        uint32_t slot = kGoalEdge;
        bool fresh = false;
        if (h != 0ull) {
            slot = (uint32_t)h & slots;
            uint32_t tries = 0u;
            for (; tries < kMostTries; ++tries) {          // (the table is at most half full while the nodes have room)
                const u64 old = ALONE ? atomicCAS(&A->table[slot], 0ull, h) : atomicCAS((u64*)&G.table[slot], 0ull, h);
                fresh = old == 0ull;
                if (fresh || old == h) break;
                slot = (slot + 1u) & slots;
            }
            if (tries >= kMostTries) { flags |= kGraphFull; fresh = false; slot = 0u; }
        }
        const u64 firsts = __ballot(fresh);
        const u64 below = t.lane == 0 ? 0ull : ~0ull >> (kWave - t.lane);
        u64 at = 0ull;
        if (t.lane == 0) {
            const u64 n = ((u64)n_found << 32) | (u64)__popcll(firsts);
            at = ALONE ? atomicAdd(&A->found[level + 1], n) : add_global((P2_GLOBAL u64*)&ctr->found[level + 1], n);
        }
        at = shfl64(at, 0);
        if (fresh) {
            const uint32_t node = next_first + (uint32_t)at + (uint32_t)__popcll(firsts & below);
            if (node < G.cap_nodes) {
                G.node_state[node] = state;
                G.node_path[node] = path;
                G.table_node[slot] = node + 1u;
            } else flags |= kGraphFull;
        }
        if (mine) {
            const uint32_t e = next_edge + (uint32_t)(at >> 32) + (uint32_t)t.lane;
            if (e < G.cap_found) G.found[e] = u32x4{from, slot, state, fresh || h == 0ull ? 1u : 0u};
            else flags |= kGraphFull;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        n_found = 0u;
    };
    for (uint32_t i0 = w * teams; i0 < items; i0 += nw * teams) {
        const uint32_t it = i0 + team;
        const bool active = it < items;
        const uint32_t use = active ? it : i0;
        const uint32_t i = use / per_node, node = first + i;
        const int pat0 = (int)((use - i * per_node) * pats), pat1 = pat0 + (int)pats < n_pat ? pat0 + (int)pats : n_pat;
        Pairs<kPairs> st;
        int np = 1;
        u64 path = 0ull;
        st.r[0] = G.all_rows; st.m[0] = 1ull << t.dev;   // Sec. 3.5: device i holds column i in every row
#pragma unroll
        for (int p = 1; p < kPairs; ++p) { st.r[p] = 0ull; st.m[p] = 0ull; }
        if (!ALONE && !last && chunk_left == 0u && t.lane == 0) chunk = more_planes(kChunk);      // (asked for before it is needed)
        if (level > 0) {
            const uint32_t state = G.node_state[node];
            path = G.node_path[node];
            np = (int)(state >> 28);
            const typename Where::planes plane = G.planes + (size_t)(state & kPlaneMask) * R;
            const u64x2 v = plane[t.dev];
            st.r[0] = v.x; st.m[0] = v.y;
#pragma unroll
            for (int p = 1; p < kPairs; ++p)
                if (p < np) { const u64x2 u = plane[(size_t)p * R + t.dev]; st.r[p] = u.x; st.m[p] = u.y; }
        } else if (i0 == 0u && team == 0u) {
            G.planes[t.dev] = u64x2{st.r[0], st.m[0]};
            if (t.dev == 0) { G.node_state[0] = 1u << 28; G.node_path[0] = 0ull; }
        }
        if (!ALONE && !last && chunk_left == 0u) { chunk = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk); chunk_left = kChunk; }
        // The goal can only come from an AllReduce on devices that all hold every row, an AllGather on devices whose rows all
        // carry every column, or a Broadcast whose roots, device 0 among them, are at the goal.
        bool go = active;
        if (last) {
            const bool r_off = rows_of(st) != G.all_rows, m_off = st.m[0] != G.all_cols || st.r[1] != 0ull;
            go = active && (!t.any(r_off) || !t.any(m_off) || !t.any(t.dev == 0 && (r_off || m_off)));
            if (!__any(go)) continue;
        }
        for (int pp = 0; pp < (int)pats; ++pp) {
        const int pat = pat0 + pp < pat1 ? pat0 + pp : pat0;
        Verdict V;
        judge(V, G, t, st, np, go && pat0 + pp < pat1, shape[pat], part[pat], last, flags);
        // goals, then children: one of each team at a time
        uint32_t left = V.kids | (V.goals << 5);
        while (__any(left != 0u)) {
            const bool has = left != 0u;
            const int bit = has ? __ffs((int)left) - 1 : 0;
            left &= left - 1u;
            const bool child = has && bit < 5;
            const int op = bit >= 5 ? bit - 5 : bit;
            u64 h = 0ull;
            uint32_t place = 0u, cp = 0u;
            Pairs<kPairs> ch = st;
            if (child) {
                const bool full = make_child(ch, V, t, np, shape[pat], part[pat], op);
                if (t.any(full)) flags |= kGraphPairs;
                cp = 1u;
#pragma unroll
                for (int p = 1; p < kPairs; ++p) cp += t.any(ch.r[p] != 0ull) ? 1u : 0u;
#pragma unroll
                for (int p = 0; p < kPairs; ++p)
                    if ((uint32_t)p < cp) h += mix(ch.r[p], ch.m[p], (uint32_t)(t.dev + 64 * p));
                for (int off = R >> 1; off > 0; off >>= 1) h += shfl64(h, t.lane ^ off);
                if (h == 0ull) h = 1ull;
            }
            // planes for the children of all teams: consecutive ones of the wavefront's chunk, or fresh ones
            const u64 kids = __ballot(child) & leaders, lower = t.base == 0 ? 0ull : ~0ull >> (kWave - t.base);
            uint32_t before = (uint32_t)__popcll(kids & lower), need = (uint32_t)__popcll(kids);
            if (__any(cp > 1u))
#pragma unroll
                for (int p = 1; p < kPairs; ++p) {
                    const u64 more = __ballot(cp > (uint32_t)p) & leaders;
                    before += (uint32_t)__popcll(more & lower); need += (uint32_t)__popcll(more);
                }
            if (need > 0u) {
                if (need <= chunk_left) {
                    place = chunk + (kChunk - chunk_left) + before;
                    chunk_left -= need;
                } else {
                    uint32_t p0 = 0u;
                    if (t.lane == 0) p0 = more_planes(need);
                    place = (uint32_t)__builtin_amdgcn_readfirstlane((int)p0) + before;
                }
            }
            if (child && place + cp <= G.cap_planes) {
                const typename Where::planes out = G.planes + (size_t)place * R;
#pragma unroll
                for (int p = 0; p < kPairs; ++p)
                    if ((uint32_t)p < cp) out[(size_t)p * R + t.dev] = u64x2{ch.r[p], ch.m[p]};
            } else if (child) flags |= kGraphFull;
            const bool add = has && (!child || place + cp <= G.cap_planes);
            const u64 adders = __ballot(add) & leaders;
            if (n_found + (uint32_t)__popcll(adders) > (uint32_t)kWave) put_found();
            if (add && t.dev == 0) {
                const uint32_t at = n_found + (uint32_t)__popcll(adders & (t.lane == 0 ? 0ull : ~0ull >> (kWave - t.lane)));
                F.hash[at] = h;
                F.state[at] = place | (cp << 28);
                const uint32_t digit = (uint32_t)pat * (uint32_t)G.n_ops + ((G.op_ranks >> (4 * op)) & 15u);
                F.from[at] = node | (digit << kDigitShift);
                F.path[at] = path << 8 | (digit + 1u);
            }
            n_found += (uint32_t)__popcll(adders);
        }
        }
    }
    put_found();
    if (flags != 0u) {
        if (ALONE) atomicOr(&A->flags, flags); else atomicOr((uint32_t*)&ctr->flags, flags);
    }
}

// What graph_finish shares: sums of the wavefronts; nodes first reached by at most d instructions; how many nodes count r
// is kept for, and where in the scratch.
struct FinishShared {
    u64 wave_sums[kFinishThreads / kWave];
    uint32_t end[P2_MAX_LEN + 1], lim[P2_MAX_LEN + 1], at[P2_MAX_LEN + 1];
    uint32_t n_found, n_words;
};

// Exclusive sums over the block of two counts at once (each below 2^31 in total).
template <int T>
__device__ u64 block_scan(u64 v, u64& total, u64* wave_sums) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    u64 s = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const u64 o = __shfl_up(s, off, kWave);
        if (lane >= off) s += o;
    }
    if (lane == kWave - 1) wave_sums[wave] = s;
    __syncthreads();
    u64 before = 0ull, all = 0ull;
    for (int w = 0; w < T / kWave; ++w) { const u64 x = wave_sums[w]; if (w < wave) before += x; all += x; }
    __syncthreads();
    total = all;
    return before + s - v;
}

// The counts of every node, from one instruction left to the size limit, and the edges that lie on the way to a goal, by
// one block with a thread per edge.  Count r of a node that `d` instructions reach first is asked for up to r = max_len - d,
// so the lists of counts get short quickly (17 274 nodes: 7 976 counts for r = 2, then 2 519, 495, 48 and 1) and stay in LDS,
// the first one (edges to the goal, at most 180) as bytes.  scratch: `words` words of LDS.
template <int T, class Where, typename Found>
__device__ void graph_finish(const Graph<Where>& G, const Found found, uint32_t trouble, FinishShared& S,
                             uint32_t* scratch, uint32_t words) {
    const uint32_t tid = threadIdx.x;
    P2_GLOBAL GraphCounters* const ctr = G.ctr;
    const int M = G.max_len, W = G.W;
    if (trouble != 0u) return;                           // (the same for every thread)
    if (tid == 0) {
        uint32_t edges = 0u;
        S.end[0] = 1u;
        for (int d = 1; d <= P2_MAX_LEN; ++d) {
            const u64 f = d <= M ? found[d] : 0ull;
            S.end[d] = S.end[d - 1] + (d < M ? (uint32_t)f : 0u);
            edges += (uint32_t)(f >> 32);
        }
        uint32_t at = (S.end[P2_MAX_LEN] + 3u) / 4u;
        for (int r = 0; r <= P2_MAX_LEN; ++r) {
            S.at[r] = at;
            S.lim[r] = r >= 2 && r <= M ? S.end[M - r] : 0u;
            at += S.lim[r];
        }
        S.n_found = edges; S.n_words = at;
    }
    __syncthreads();
    const uint32_t* const end = S.end; const uint32_t* const lim = S.lim; const uint32_t* const at = S.at;
    u64* const wave_sums = S.wave_sums;
    const uint32_t n_nodes = end[P2_MAX_LEN], n_found = S.n_found, total_words = S.n_words;
    if (total_words > words) {
        if (tid == 0) ctr->flags = kGraphPairs;          // (no structure that graph_applies lets through has as many states)
        return;
    }
    uint8_t* const bytes = reinterpret_cast<uint8_t*>(scratch);
    // (the children by their nodes instead of their slots)
    if (!G.links_ready)
    for (uint32_t e = tid; e < n_found; e += T) {
        const u32x4 f = G.found[e];
        G.links[e] = u32x2{f.x, f.y == kGoalEdge ? kGoalEdge : G.table_node[f.y] - 1u};
    }
    // first the prefixes (programs whose rules all hold, short of the goal), then the programs that end at the goal
    for (int kind = 0; kind < 2; ++kind) {
        for (uint32_t x = tid; x < total_words; x += T) scratch[x] = 0u;
        __syncthreads();
        for (uint32_t e = tid; e < n_found; e += T) {
            const u32x2 l = G.links[e];
            const uint32_t from = l.x & kGoalEdge;
            if ((l.y == kGoalEdge) == (kind == 1)) atomicAdd(&scratch[from >> 2], 1u << (8u * (from & 3u)));
        }
        __syncthreads();
        for (int r = 2; r <= M; ++r) {
            const uint32_t lim_r = lim[r], at_r = at[r], at_before = at[r - 1];
            for (uint32_t e = tid; e < n_found; e += T) {
                const u32x2 l = G.links[e];
                const uint32_t from = l.x & kGoalEdge;
                if (l.y == kGoalEdge || from >= lim_r) continue;
                const uint32_t n = r == 2 ? (uint32_t)bytes[l.y] : scratch[at_before + l.y];
                if (n != 0u) atomicAdd(&scratch[at_r + from], n);
            }
            __syncthreads();
        }
        if (tid == 0)
            for (int r = 1; r <= M; ++r) {
                const uint32_t n = r == 1 ? (uint32_t)bytes[0] : scratch[at[r]];
                if (kind == 1) ctr->n_valid[r] = n;
                else if (r < M) ctr->n_prefixes[r] = n;
            }
        __syncthreads();
    }
    // a goal can be reached from node n with at most `left` instructions
    auto reaches = [&](uint32_t n, int left) {
        bool any = left >= 1 && bytes[n] != 0;
        for (int r = 2; r <= left && r <= M; ++r)
            if (n < lim[r]) any |= scratch[at[r] + n] != 0u;
        return any;
    };
    auto depth_of = [&](uint32_t n) {
        int d = 0;
        for (int x = 0; x < M; ++x) d += n >= end[x] ? 1 : 0;
        return d;
    };
    // the nodes on the way to a goal, renumbered, and their counts
    uint32_t n_use = 0u;
    for (uint32_t n0 = 0; n0 < n_nodes; n0 += T) {
        const uint32_t n = n0 + tid;
        const bool use = n < n_nodes && reaches(n, M);   // (counts beyond what is left there are not kept)
        u64 total;
        const uint32_t id = n_use + (uint32_t)block_scan<T>(use ? 1ull : 0ull, total, wave_sums);
        if (n < n_nodes) G.use_id[n] = use ? id : ~0u;
        if (use) {
            P2_GLOBAL uint32_t* const out = G.use_ends + (size_t)id * 8;
            out[1] = bytes[n];
            for (int r = 2; r <= P2_MAX_LEN; ++r) out[r] = n < lim[r] ? scratch[at[r] + n] : 0u;
        }
        n_use += (uint32_t)total;
    }
    // Their edges in the order of the digits: a set of digits per node says how many edges come before one of them.
    const uint32_t sets_at = (total_words + 1u) & ~1u, set_words = 2u * (uint32_t)W * n_use;
    if (sets_at + set_words > words) {
        if (tid == 0) ctr->flags = kGraphPairs;
        return;
    }
    u64* const sets = reinterpret_cast<u64*>(scratch + sets_at);
    for (uint32_t x = tid; x < set_words / 2u; x += T) sets[x] = 0ull;
    __syncthreads();
    for (uint32_t e = tid; e < n_found; e += T) {
        const u32x2 l = G.links[e];
        const uint32_t from = l.x & kGoalEdge, d = l.x >> kDigitShift;
        if (l.y == kGoalEdge || reaches(l.y, M - 1 - depth_of(from))) atomicOr(&sets[(size_t)G.use_id[from] * W + (d >> 6)], 1ull << (d & 63u));
        else G.links[e] = u32x2{~0u, 0u};
    }
    __syncthreads();
    uint32_t n_edges = 0u;
    for (uint32_t u0 = 0; u0 < n_use; u0 += T) {
        const uint32_t u = u0 + tid;
        uint32_t n = 0u;
        if (u < n_use)
            for (int x = 0; x < W; ++x) n += (uint32_t)__popcll(sets[(size_t)u * W + x]);
        u64 total;
        const uint32_t first = n_edges + (uint32_t)block_scan<T>(n, total, wave_sums);
        if (u < n_use) G.first_edge[u] = u32x2{first, first + n};
        n_edges += (uint32_t)total;
    }
    if (n_edges > G.cap_edges) {                         // (the same for every thread)
        if (tid == 0) ctr->flags = kGraphFull;
        return;
    }
    if (tid == 0) {
        ctr->n_edges = n_edges;
        ctr->n_judged = n_nodes;
        uint32_t n = 0u;
        for (int r = 1; r <= M; ++r) n += r == 1 ? (uint32_t)bytes[0] : scratch[at[r]];
        ctr->n_total = n;
    }
    __syncthreads();
    for (uint32_t e = tid; e < n_found; e += T) {
        const u32x2 l = G.links[e];
        if (l.x == ~0u) continue;
        const uint32_t from = l.x & kGoalEdge, d = l.x >> kDigitShift, u = G.use_id[from];
        uint32_t to = G.first_edge[u].x + (uint32_t)__popcll(sets[(size_t)u * W + (d >> 6)] & ((1ull << (d & 63u)) - 1ull));
        for (uint32_t x = 0; x < (d >> 6); ++x) to += (uint32_t)__popcll(sets[(size_t)u * W + x]);
        G.edges[to] = (d << kDigitShift) | (l.y == kGoalEdge ? kGoalEdge : G.use_id[l.y]);
        if (G.skeleton) G.edge_path[to] = G.node_path[from];
        else G.edge_state[to] = G.node_state[from];
    }
}

// Bound by latency: a state's lane exchanges, then a look at the table and a place in the lists.  Launches per level, not one
// kernel for all: a level needs the whole chip (17 274 states of 64 devices, six levels: 370 us a launch beside other groups'
// kernels) and the next one all of it.  The 18 structures of 140 queries of [4 8 8], five levels: 180 us, where walking the
// stems (k_eval_shared), the groups that it hands over and the programs' costs took 3.5 ms; 26 queries of [4 2 4]: 54 of
// 110 us.
constexpr int kLevelThreads = 256;
template <int kPairs>
__global__ __launch_bounds__(kLevelThreads) void k_graph_level(const DevGraph* __restrict__ graphs, const GraphBlock* __restrict__ blocks, int level) {
    __shared__ Found found[kLevelThreads / kWave];
    __shared__ uint32_t shape[kGraphPatterns];           // log2 g | log2 s << 4
    __shared__ u64 part[kGraphPatterns];
    const GraphBlock b = blocks[blockIdx.x];
    const DevGraph& D = graphs[b.graph];
    const Graph<InDevice> G = open_in_device(D);
    if (level >= G.max_len) return;
    if ((int)threadIdx.x < G.n_pat) { shape[threadIdx.x] = D.shape[threadIdx.x]; part[threadIdx.x] = D.part[threadIdx.x]; }
    __syncthreads();
    const uint32_t waves = kLevelThreads / kWave, wave = threadIdx.x / kWave;
    graph_level<kPairs>(G, shape, part, level, wave * b.count + b.index, b.count * waves, found[wave], nullptr);
}

__global__ __launch_bounds__(kFinishThreads) void k_graph_finish(const DevGraph* __restrict__ graphs, const uint32_t* __restrict__ list, uint32_t words) {
    extern __shared__ __attribute__((aligned(16))) uint32_t scratch[];
    __shared__ FinishShared S;
    const Graph<InDevice> G = open_in_device(graphs[list[blockIdx.x]]);
    const uint32_t trouble = G.ctr->flags;
    __syncthreads();                                     // (every thread has read it before the block can set it)
    graph_finish<kFinishThreads>(G, (P2_GLOBAL const u64*)G.ctr->found, trouble, S, scratch, words);
}

// Structures of one or two levels: a block goes through all levels and the counts by itself, with everything it works on
// in LDS, two pairs a device (no such structure needs more).  Bound by the chain of the levels in one block; launches per
// level would add some 5 us each, and their lists' round trips to L2.  [2 4], three levels: 28 us, where the walk, the groups handed
// over and the costs took 32 in three launches; [4 16], five levels: 68 us, where they took 120.
__global__ __launch_bounds__(kAloneThreads) void k_graph_alone(const DevGraph* __restrict__ graphs, const uint32_t* __restrict__ list) {
    extern __shared__ __attribute__((aligned(16))) u64x2 planes[];
    __shared__ Found found[kAloneThreads / kWave];
    __shared__ AloneShared A;
    __shared__ FinishShared S;
    __shared__ uint32_t shape[kGraphPatterns];
    __shared__ u64 part[kGraphPatterns];
    __shared__ __attribute__((aligned(16))) uint32_t scratch[kAloneScratch];
    const DevGraph& D = graphs[list[blockIdx.x]];
    const Graph<InBlock> G = open_in_block(D, A, planes);
    for (uint32_t x = threadIdx.x; x < kAloneSlots; x += kAloneThreads) { A.table[x] = 0ull; A.table_node[x] = 0u; }
    if (threadIdx.x <= P2_MAX_LEN) A.found[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) A.n_planes = A.flags = 0u;
    if ((int)threadIdx.x < G.n_pat) { shape[threadIdx.x] = D.shape[threadIdx.x]; part[threadIdx.x] = D.part[threadIdx.x]; }
    __syncthreads();
    for (int level = 0; level < G.max_len; ++level) {
        graph_level<2>(G, shape, part, level, threadIdx.x / kWave, kAloneThreads / kWave, found[threadIdx.x / kWave], &A);
        __syncthreads();
    }
    const uint32_t trouble = A.flags;
    if (threadIdx.x == 0 && trouble != 0u) G.ctr->flags = trouble;
    if (trouble == 0u) {                                 // (the states that the edges' costs are worked out from)
        const uint32_t n = (A.n_planes + 1u) * (uint32_t)G.R;
        for (uint32_t x = threadIdx.x; x < n; x += kAloneThreads) G.planes_out[x] = planes[x];
    }
    graph_finish<kAloneThreads>(G, (P2_LOCAL const u64*)A.found, trouble, S, scratch, kAloneScratch);
}

// What every edge on the way to a goal adds to the bandwidth sum of each query of its structure: a wavefront per edge.
// Where all groups of the pattern hold the same number of rows (four fifths of the edges) the busiest unit of a level
// carries that number times the level's largest sum of multiplicities, and a lane answers for a query; else the
// queries' bandwidth rows are walked, one query after the other.  Bound by L2 latency: an edge is a chain of its state, the
// pattern's entry and the rows.  [2 4]: 8 us, [4 16], three sizes: 26; 512 queries of [2 4 8 8]: 0.9 ms of the call's 15.5.
constexpr int kStepWaves = 4;
__global__ __launch_bounds__(kStepWaves * kWave) void k_graph_steps(const DevQuery* __restrict__ queries, const DevGraph* __restrict__ graphs,
                                                                    const GraphBlock* __restrict__ blocks) {
    __shared__ uint16_t srows[kStepWaves][P2_MAX_DEVICES];
    const GraphBlock b = blocks[blockIdx.x];
    const Graph<InDevice> G = open_in_device(graphs[b.graph]);
    if (G.ctr->flags != 0u) return;
    const DevQuery& q = queries[G.query];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int R = G.R;
    uint16_t* const rows = srows[wave];                  // (a wavefront's own: no barriers)
    const uint32_t n_edges = G.ctr->n_edges, per_pass = b.count * (uint32_t)kStepWaves;
    for (uint32_t e = b.index * (uint32_t)kStepWaves + (uint32_t)wave; e < n_edges; e += per_pass) {
        const uint32_t state = G.edge_state[e];
        const uint32_t ins = q.instr_of_digit[G.edges[e] >> kDigitShift];
        const int pid = (int)(ins >> 3), op = (int)(ins & 7u);
        const int g = q.pat[pid].g, s = q.pat[pid].s, master = q.pat[pid].master, ng = q.pat[pid].n_groups;
        // rows held by every device (its pairs' rows are disjoint)
        if (!G.links_ready) {
            const P2_GLOBAL u64x2* const plane = G.planes + (size_t)(state & kPlaneMask) * R;
            if (lane < R) {
                int c = 0;
                for (uint32_t p = 0; p < (state >> 28); ++p) c += __popcll(plane[(size_t)p * R + lane].x);
                rows[lane] = (uint16_t)c;
            }
        } else {
            const int np = (int)(state >> 28), plane = R * G.wq;
            const P2_GLOBAL u32x4* const at = G.large[np - 1] + (size_t)(state & kPlaneMask) * (size_t)(np * plane);
            for (int d = lane; d < R; d += kWave) {
                int c = 0;
                for (int p = 0; p < np; ++p)
                    for (int x = 0; x < G.qk; ++x) {
                        const u32x4 v = at[p * plane + d * G.wq + x];
                        c += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
                    }
                rows[d] = (uint16_t)c;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // the chunks that set a group's bytes, at its first device: the members' common ones, the root's, or all that an
        // AllGather brings together
        auto base_of = [&](int i) { return master ? i * g * s : (i / s) * g * s + i % s; };
        if (op == OP_AG)
            for (int i = lane; i < ng; i += kWave) {
                const int base = base_of(i);
                uint32_t c = 0u;
                for (int m = 0; m < g; ++m) c += rows[base + m * s];
                rows[base] = (uint16_t)c;                // (the groups do not meet)
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t c0 = rows[0];                     // (device 0 is a root of every pattern)
        bool same = true;
        for (int i = lane; i < ng; i += kWave) same &= rows[base_of(i)] == c0;
        P2_GLOBAL double* const out = G.best + (size_t)e * G.n_members;
        if (!__any(!same)) {
            for (int j = lane; j < G.n_members; j += kWave) {
                const DevQuery& cq = queries[G.members[j]];
                const DevRows& rw = *cq.rows;
                const long long n = (long long)c0 * (long long)(cq.k / G.rows_kept);
                double best = 0.0;
                for (int l = 0; l < cq.n_levels; ++l) best = fmax(best, (double)(n * (long long)rw.level_max[pid][l]) * cq.inv_bw[l]);
                out[j] = best;
            }
        } else {
            for (int j = 0; j < G.n_members; ++j) {
                const DevQuery& cq = queries[G.members[j]];
                const DevRows& rw = *cq.rows;
                const long long per = (long long)(cq.k / G.rows_kept);
                double best = 0.0;
                for (int row = rw.pat_begin[pid] + lane; row < rw.pat_begin[pid + 1]; row += kWave) {
                    long long dot = 0;
                    int x = rw.row_ptr[row];
                    const int end = rw.row_ptr[row + 1];
                    for (; x + 8 <= end; x += 8) {       // (eight entries in flight)
                        uint32_t ent[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) ent[u] = rw.entries[x + u];
#pragma unroll
                        for (int u = 0; u < 8; ++u) dot += (long long)entry_cnt(ent[u]) * (long long)rows[entry_base(ent[u])];
                    }
                    for (; x < end; ++x) {
                        const uint32_t ent = rw.entries[x];
                        dot += (long long)entry_cnt(ent) * (long long)rows[entry_base(ent)];
                    }
                    best = fmax(best, (double)(dot * per) * cq.inv_bw[rw.row_level[row]]);
                }
                for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off, kWave));
                if (lane == 0) out[j] = best;
            }
        }
    }
}

// The same for a skeleton of five or six levels (p2_skeleton.hip has the smaller ones), from the instructions that lead to an edge's
// state: a wavefront per edge, a lane per query.
__global__ __launch_bounds__(kStepWaves * kWave) void k_graph_costs(const DevQuery* __restrict__ queries, const DevGraph* __restrict__ graphs,
                                                                    const GraphBlock* __restrict__ blocks) {
    __shared__ PatternTable T;
    const GraphBlock b = blocks[blockIdx.x];
    const DevGraph& D = graphs[b.graph];
    const Graph<InDevice> G = open_in_device(D);
    if (G.ctr->flags != 0u) return;
    const P2_GLOBAL DevMember* const sizes = in_global<const DevMember>(D.sizes);
    const uint32_t n_edges = G.ctr->n_edges;
    T.open(D, queries[G.query]);
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t chunks = ((uint32_t)G.n_members + kWave - 1u) / kWave, items = n_edges * chunks, per_pass = b.count * (uint32_t)kStepWaves;
    for (uint32_t it = b.index * (uint32_t)kStepWaves + wave; it < items; it += per_pass) {
        const uint32_t e = it / chunks, member = (it - e * chunks) * kWave + (uint32_t)lane;
        const bool mine = member < (uint32_t)G.n_members;
        HeldRows<kSkeletonLevels> rows;
        rows.start(sizes[mine ? member : 0u], G.R);
        rows.follow(G.edge_path[e], T);
        const double best = rows.busiest(T.of(G.edges[e] >> kDigitShift), sizes[mine ? member : 0u]);
        if (mine) G.best[(size_t)e * G.n_members + member] = best;
    }
}

// a + b * c with the product rounded first, whatever the compiler may contract elsewhere.
__device__ __forceinline__ double add_rounded(double a, double b, double c) {
#pragma clang fp contract(off)
    const double p = b * c;
    return a + p;
}

// The rows of the valid programs, a thread each: program t of the ascending order is found by walking the edges from the
// first node, leaving out as many programs as lie behind the edges before; its cost is the sum over its edges in order.
// Which query's rows a block writes follows from the counts of the graphs (the host need not know them): the queries' rows
// come one after the other, 256 to a block.  With `segs` the host says where they go (a call with queries of other engines).
// progs and costs may be host memory: a block's rows are written side by side.
__global__ __launch_bounds__(256) void k_graph_emit(const DevQuery* __restrict__ queries, const DevGraph* __restrict__ graphs,
                                                    const GraphCounters* __restrict__ ctrs, const GraphQuery* __restrict__ asked, int n_queries,
                                                    const GraphRows* __restrict__ segs, int n_segs, u64 cap_rows, u64* __restrict__ sorted,
                                                    p2_program* __restrict__ progs, double* __restrict__ costs, uint4* __restrict__ ctrs_out, int n_graphs,
                                                    u32x4* __restrict__ walks) {
    constexpr uint32_t kAhead = 8u;
    __shared__ u64 wave_sums[256 / kWave];
    __shared__ uint32_t s_query, s_graph, s_member, s_block, s_count, s_fused;
    __shared__ u64 s_first;
    __shared__ double s_sum[2][256];
    __shared__ double s_steps[kGraphPatterns * 5], s_alpha[kGraphPatterns * 5], s_per[kGraphPatterns * 5];   // what a step costs, by digit
    __shared__ uint8_t s_instr[kGraphPatterns * 5];
    const uint32_t tid = threadIdx.x;
    if (ctrs_out && blockIdx.x == gridDim.x - 1u) {       // (the host reads the counts with the rows)
        const uint4* const from = reinterpret_cast<const uint4*>(ctrs);
        for (uint32_t x = tid; x < (uint32_t)n_graphs * (uint32_t)(sizeof(GraphCounters) / 16); x += 256u) ctrs_out[x] = from[x];
    }
    if (segs) {
        int a = 0, z = n_segs - 1;
        while (a < z) {
            const int mid = (a + z + 1) >> 1;
            if (segs[mid].first_block <= blockIdx.x) a = mid; else z = mid - 1;
        }
        if (tid == 0) {
            const GraphRows seg = segs[a];
            s_query = seg.query; s_graph = seg.graph; s_member = seg.member; s_count = seg.count; s_first = seg.out_first; s_fused = seg.fused;
            s_block = blockIdx.x - seg.first_block;
        }
    } else {
        if (tid == 0) s_count = 0u;
        __syncthreads();
        u64 run = 0ull;                                   // rows << 32 | blocks before
        for (int q0 = 0; q0 < n_queries; q0 += 256) {
            const int q = q0 + (int)tid;
            uint32_t n = 0u, g = 0u;
            if (q < n_queries) { g = asked[q].graph; n = g == ~0u ? 0u : ctrs[g].n_total; }
            const u64 mine = ((u64)n << 32) | ((n + 255u) / 256u);
            u64 total;
            const u64 before = run + block_scan<256>(mine, total, wave_sums);
            if (n > 0u && blockIdx.x >= (uint32_t)before && blockIdx.x < (uint32_t)(before + mine)) {
                s_query = (uint32_t)q; s_graph = g; s_member = asked[q].member; s_count = n; s_first = before >> 32;
                s_fused = asked[q].fused;
                s_block = blockIdx.x - (uint32_t)before;
            }
            run += total;
            if (blockIdx.x < (uint32_t)run) break;        // (the same for every thread)
        }
    }
    __syncthreads();
    const uint32_t t0 = s_block * 256u, t = t0 + tid;
    if (segs && tid == 0) { const uint32_t n = graphs[s_graph].ctr->n_total; if (n < s_count) s_count = n; }
    if (segs) __syncthreads();
    if (t0 >= s_count) return;
    const uint32_t rows = s_count - t0 < 256u ? s_count - t0 : 256u;
    const u64 row0 = s_first + t0;
    if (row0 + rows > cap_rows) return;                   // (the host sees that there are more, and asks again with room)
    const Graph<InDevice> G = open_in_device(graphs[s_graph]);
    const DevQuery& q = queries[s_query];
    const bool with_costs = q.n_msg > 0 && s_member != ~0u;
    // (worked out once per block: with two divisions a step in every row, the kernel took 900 us for 8.2 million rows of
    //  four levels, and takes 780)
    for (uint32_t d = tid; d < (uint32_t)q.alphabet; d += 256u) {
        const uint32_t ins = q.instr_of_digit[d];
        const int pid = (int)(ins >> 3), op = (int)(ins & 7u);
        s_instr[d] = (uint8_t)(pid * 5 + op);
        if (with_costs) {
            const DevPattern& P = q.pat[pid];
            double ring_steps, mult;
            step_factors(op, P.g, q.algo, ring_steps, mult);
            s_steps[d] = ring_steps; s_alpha[d] = q.alpha[P.span_level]; s_per[d] = mult / (double)q.k;
        }
    }
    __syncthreads();
    if (tid < rows) {
        const uint32_t member = s_member;
        uint32_t j = t;
        int len = 1;
#pragma unroll
        for (int l = 1; l < P2_MAX_LEN; ++l) {            // (the counts of lengths past the size limit are zero)
            const uint32_t n = G.ctr->n_valid[l];
            if (len == l && l < G.max_len && j >= n) { j -= n; ++len; }
        }
        p2_program pr;
        pr.len = (uint8_t)len;
        u64 number = 0ull;
        double sum_alpha = 0.0, sum_beta = 0.0;
        uint32_t node = 0u, walk[8];
        walk[7] = ~0u;
#pragma unroll
        for (int s = 0; s < P2_MAX_LEN; ++s) {
            pr.instr[s] = 0;
            walk[s] = ~0u;
            if (s >= len) continue;
            const int left = len - s;                     // instructions from here on
            // (eight edges' counts in flight: edge after edge, each count a load behind its edge's, the walks were the whole of
            //  the kernel.  571 rows of three levels and 83 920 of four, us: four edges 15.5 and 27.3, eight 13.8 and 22.9, sixteen
            //  14.7 and 23.2)
            const u32x2 own = G.first_edge[node];
            uint32_t e = own.x, edge = 0u;
            const uint32_t end = own.y;
            for (bool found = false; !found && e < end;) {
                uint32_t some[kAhead], n[kAhead];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) some[u] = G.edges[e + u < end ? e + u : end - 1u];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) {
                    const uint32_t target = some[u] & kGoalEdge;
                    const uint32_t ends = G.use_ends[(size_t)(target == kGoalEdge ? 0u : target) * 8 + (left > 1 ? left - 1 : 0)];
                    n[u] = e + u >= end ? 0u : target == kGoalEdge ? (left == 1 ? 1u : 0u) : left > 1 ? ends : 0u;
                }
                uint32_t at = e + kAhead < end ? e + kAhead : end;
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) {
                    if (found) continue;
                    if (j < n[u]) { found = true; edge = some[u]; at = e + u; }
                    else j -= n[u];
                }
                e = at;
            }
            const uint32_t digit = edge >> kDigitShift;
            pr.instr[s] = s_instr[digit];
            number = number * (u64)q.alphabet + digit;
            node = left > 1 && e < end ? edge & kGoalEdge : node;
            if (e < end) walk[s] = digit << kDigitShift | e;
            if (with_costs && e < end) {
                const double ring_steps = s_steps[digit], alpha = s_alpha[digit], per = s_per[digit], best = G.best[(size_t)e * G.n_members + member];
                // (rounded as in the engines whose place this one takes: the walk's costs are fused, the frontier's steps are not)
                if (s_fused != 0u) { sum_alpha = fma(ring_steps, alpha, sum_alpha); sum_beta = fma(per, best, sum_beta); }
                else { sum_alpha = add_rounded(sum_alpha, ring_steps, alpha); sum_beta = add_rounded(sum_beta, per, best); }
            }
        }
        pr.index = q.base[len] + number;
        if (sorted) sorted[row0 + tid] = pr.index;
        progs[row0 + tid] = pr;
        s_sum[0][tid] = sum_alpha; s_sum[1][tid] = sum_beta;
        if (member == ~0u) {
            walks[(row0 + tid) * 2] = u32x4{walk[0], walk[1], walk[2], walk[3]};
            walks[(row0 + tid) * 2 + 1] = u32x4{walk[4], walk[5], walk[6], walk[7]};
        }
    }
    if (!with_costs) return;
    __syncthreads();
    const uint32_t n_msg = (uint32_t)q.n_msg;
    for (uint32_t x = tid; x < rows * n_msg; x += 256u) {
        const uint32_t r = x / n_msg, m = x - r * n_msg;
        costs[row0 * n_msg + x] = fma(q.msg_bytes[m], s_sum[1][r], s_sum[0][r]);
    }
}

// The costs of a graph's rows for every query that shares it, where the rows themselves have been written once (k_graph_emit, member
// ~0, with the edges of each).  Half a wavefront holds 32 queries of one row, so that what an edge adds is read in runs of 256
// bytes; what a step costs each query lies in LDS; 64 rows at a time are turned round there, so that the costs leave in runs of 512
// bytes.  With a walk per row and query, lanes on rows, the gathers along the edges were the whole cost: 512 queries of [2 4 8 8],
// 8.2 million rows, 690 us, and 114 so with 22 for the rows: half of it instructions to issue, 1.6 TB/s between the caches and memory.
constexpr int kSumThreads = 512, kSumTile = 64;
__global__ __launch_bounds__(kSumThreads) void k_graph_sums(const DevQuery* __restrict__ queries, const DevGraph* __restrict__ graphs,
                                                            const GraphSums* __restrict__ sums, int n_sums, const GraphColumn* __restrict__ columns,
                                                            const u32x4* __restrict__ walks, double* __restrict__ costs, uint32_t rows_of_block) {
    constexpr uint32_t C = kSumMembers, kTeams = kSumThreads / C, kOwn = kSumTile / kTeams;
    __shared__ double s_steps[kSumDigits][C], s_per[kSumDigits][C], s_alpha[kSumDigits / 5][C], s_tile[kSumTile][C + 1];
    __shared__ u64 s_out[C];
    int a = 0, z = n_sums - 1;
    while (a < z) {
        const int mid = (a + z + 1) >> 1;
        if (sums[mid].first_block <= blockIdx.x) a = mid; else z = mid - 1;
    }
    const GraphSums J = sums[a];
    const DevGraph& D = graphs[J.graph];
    const uint32_t n_total = D.ctr->n_total, n_rows = n_total < J.most ? n_total : J.most, c0 = blockIdx.y * C;
    const uint32_t begin = (blockIdx.x - J.first_block) * rows_of_block, end = begin + rows_of_block < n_rows ? begin + rows_of_block : n_rows;
    if (c0 >= J.n_columns || begin >= n_rows) return;
    const uint32_t tid = threadIdx.x, col = tid % C, team = tid / C, n_cols = J.n_columns - c0 < C ? J.n_columns - c0 : C;
    // (the lanes behind the last query do its work again, and leave nothing)
    const uint32_t member = c0 + (col < n_cols ? col : n_cols - 1u);
    const GraphColumn own = columns[J.first_column + member];
    const DevQuery& q = queries[own.query];
    for (uint32_t pid = team; pid < (uint32_t)q.n_patterns; pid += kTeams) {
        const DevPattern& P = q.pat[pid];
        const int g = P.g;
        s_alpha[pid][col] = q.alpha[P.span_level];
        for (uint32_t op = 0; op < 5u; ++op) {           // (skeletons have all five operations)
            double ring_steps, mult;
            step_factors((int)q.ops[op], g, q.algo, ring_steps, mult);
            s_steps[pid * 5u + op][col] = ring_steps; s_per[pid * 5u + op][col] = mult / (double)q.k;
        }
    }
    if (team == 0u) s_out[col] = own.out_first;
    __syncthreads();
    const P2_GLOBAL double* const best = in_global<const double>(D.best);
    const uint32_t n_members = (uint32_t)D.n_members, n_msg = (uint32_t)q.n_msg;
    const double* const msg_bytes = q.msg_bytes;
    const int max_len = D.max_len;
    const bool fused = J.fused != 0u;
    for (uint32_t row0 = begin; row0 < end; row0 += kSumTile) {
        double sum_alpha[kOwn], sum_beta[kOwn];
        u32x4 walk[kOwn][2];
#pragma unroll
        for (uint32_t x = 0; x < kOwn; ++x) {
            const uint32_t row = row0 + team + x * kTeams;
            const u32x4* const at = walks + (J.first_row + (row < end ? row : end - 1u)) * 2u;
            walk[x][0] = at[0]; walk[x][1] = at[1];
            sum_alpha[x] = sum_beta[x] = 0.0;
        }
#pragma unroll
        for (int s = 0; s < P2_MAX_LEN; ++s) {
            if (s >= max_len) break;
            double b[kOwn];
#pragma unroll
            for (uint32_t x = 0; x < kOwn; ++x) {
                const uint32_t step = walk[x][s / 4][s % 4];
                b[x] = best[(size_t)(step != ~0u ? step & ((1u << kDigitShift) - 1u) : 0u) * n_members + member];
            }
#pragma unroll
            for (uint32_t x = 0; x < kOwn; ++x) {
                const uint32_t step = walk[x][s / 4][s % 4], digit = step != ~0u ? step >> kDigitShift : 0u;
                const double ring_steps = s_steps[digit][col], alpha = s_alpha[digit / 5u][col], per = s_per[digit][col];
                // (rounded as k_graph_emit rounds)
                double next_alpha, next_beta;
                if (fused) { next_alpha = fma(ring_steps, alpha, sum_alpha[x]); next_beta = fma(per, b[x], sum_beta[x]); }
                else { next_alpha = add_rounded(sum_alpha[x], ring_steps, alpha); next_beta = add_rounded(sum_beta[x], per, b[x]); }
                if (step != ~0u) { sum_alpha[x] = next_alpha; sum_beta[x] = next_beta; }
            }
        }
        for (uint32_t m = 0; m < n_msg; ++m) {
            const double bytes = msg_bytes[m];
#pragma unroll
            for (uint32_t x = 0; x < kOwn; ++x) s_tile[team + x * kTeams][col] = fma(bytes, sum_beta[x], sum_alpha[x]);
            __syncthreads();
            for (uint32_t x = tid; x < n_cols * kSumTile; x += kSumThreads) {
                const uint32_t c = x / kSumTile, r = x % kSumTile;
                if (row0 + r < end) costs[(s_out[c] + row0 + r) * n_msg + m] = s_tile[r][c];
            }
            __syncthreads();
        }
    }
}

}  // namespace

uint32_t graph_planes_left(uint32_t blocks, int max_len) { return kChunk * (uint32_t)(kLevelThreads / kWave) * blocks * (uint32_t)(max_len > 1 ? max_len - 1 : 1); }
bool graph_alone_holds(uint32_t nodes) { return nodes <= kAloneNodes; }
hipError_t launch_graph_alone(const DevGraph* graphs, const uint32_t* list, unsigned n, int max_R, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const size_t bytes = sizeof(u64x2) * kAlonePlanes * (size_t)max_R, most = sizeof(u64x2) * kAlonePlanes * 64;
    if (bytes > 64 * 1024 - sizeof(AloneShared) - sizeof(Found) * (kAloneThreads / kWave) - 8192) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_graph_alone), hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_graph_alone, dim3(n), dim3(kAloneThreads), bytes, stream, graphs, list);
    return hipGetLastError();
}
hipError_t launch_graph_level(const DevGraph* graphs, const GraphBlock* blocks, unsigned n_blocks, int level, int max_len, hipStream_t stream) {
    if (n_blocks == 0) return hipSuccess;
    // (programs of five instructions need no third pair, whatever the levels)
    if (max_len <= 5) hipLaunchKernelGGL(k_graph_level<2>, dim3(n_blocks), dim3(kLevelThreads), 0, stream, graphs, blocks, level);
    else hipLaunchKernelGGL(k_graph_level<kMostPairs>, dim3(n_blocks), dim3(kLevelThreads), 0, stream, graphs, blocks, level);
    return hipGetLastError();
}
hipError_t launch_graph_finish(const DevGraph* graphs, const uint32_t* list, unsigned n, size_t lds_bytes, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const size_t most = 160 * 1024 - 1024;               // (beside the wavefronts' sums)
    const size_t bytes = lds_bytes < most ? lds_bytes : most;
    if (bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_graph_finish), hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_graph_finish, dim3(n), dim3(kFinishThreads), bytes, stream, graphs, list, (uint32_t)(bytes / 4));
    return hipGetLastError();
}
hipError_t launch_graph_steps(const DevQuery* queries, const DevGraph* graphs, const GraphBlock* blocks, unsigned n_blocks, hipStream_t stream) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_graph_steps, dim3(n_blocks), dim3(kStepWaves * kWave), 0, stream, queries, graphs, blocks);
    return hipGetLastError();
}
hipError_t launch_graph_costs(const DevQuery* queries, const DevGraph* graphs, const GraphBlock* blocks, unsigned n_blocks, hipStream_t stream) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_graph_costs, dim3(n_blocks), dim3(kStepWaves * kWave), 0, stream, queries, graphs, blocks);
    return hipGetLastError();
}
hipError_t launch_graph_emit(const DevQuery* queries, const DevGraph* graphs, const GraphCounters* ctrs, const GraphQuery* asked, int n_queries,
                             const GraphRows* segs, int n_segs, unsigned n_blocks, unsigned long long cap_rows, unsigned long long* sorted,
                             p2_program* progs, double* costs, void* ctrs_out, int n_graphs, void* walks, hipStream_t stream) {
    if (n_blocks == 0) return hipSuccess;
    static_assert(sizeof(GraphCounters) % 16 == 0, "copied in 16-byte words");
    hipLaunchKernelGGL(k_graph_emit, dim3(n_blocks), dim3(256), 0, stream, queries, graphs, ctrs, asked, n_queries, segs, n_segs, cap_rows, sorted,
                       progs, costs, static_cast<uint4*>(ctrs_out), n_graphs, static_cast<u32x4*>(walks));
    return hipGetLastError();
}
hipError_t launch_graph_sums(const DevQuery* queries, const DevGraph* graphs, const GraphSums* sums, int n_sums, const GraphColumn* columns,
                             unsigned n_blocks, unsigned most_columns, unsigned rows_of_block, const void* walks, double* costs, hipStream_t stream) {
    if (n_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_graph_sums, dim3(n_blocks, (most_columns + kSumMembers - 1) / kSumMembers), dim3(kSumThreads), 0, stream, queries, graphs, sums, n_sums,
                       columns, static_cast<const u32x4*>(walks), costs, rows_of_block);
    return hipGetLastError();
}

}  // namespace p2
