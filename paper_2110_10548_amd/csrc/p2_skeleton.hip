// State graphs of skeletons (see p2_graph.hip) of up to four levels: at most 16 devices, and a state is written out, for every
// device the mask of every row (16 bits a device at two levels, 16 words at four).  Then no rule needs to know which rows go
// together: the union of a group's members is the bitwise one, for AllReduce, Reduce, ReduceScatter and AllGather alike, and
// what tells them apart is a few tests.  The devices of a state are lanes of one DPP row, which exchange without LDS.
//
// A block takes 64 / R states (times as many as fit with few patterns) and a wavefront one pattern of them: everything about a
// pattern is the same for the whole wavefront, and the block knows all edges of its states, which it writes next to each other
// in the order of their digits.  The counts can then walk every state's edges without sorting them first.
#include "p2_graph_dev.h"

namespace p2 {

namespace {

constexpr int kLevelThreads = 1024, kLevelWaves = kLevelThreads / kWave;
constexpr int kEntries = 256;               // (state, pattern) pairs of a block at a time
constexpr int kEntryPatterns = 16;
constexpr uint32_t kSlotMask = 0x7fffffu, kFreshEdge = 1u << 31;
// a skeleton of one or two levels has at most 42 states, and 93 edges that are not left out at the size limit
constexpr uint32_t kAloneSlots = 256, kAloneNodes = 64, kAloneEdges = 160, kAloneScratch = 1024;

struct LevelShared {
    u64 hash[kEntries * 5];                 // of the child's state; 0: the goal
    uint32_t edge[kEntries * 5];            // state within the block | digit << 16
    uint32_t fresh[kLevelWaves];            // by wavefront: children that are new
    u64 path[kEntries];
    __attribute__((aligned(8))) uint16_t code[kEntries];      // by (state, pattern): children | goals << 5; past the last one, nothing
    uint32_t shape[kEntryPatterns], part[kEntryPatterns];
    uint32_t base, node0, flags;
};
struct AloneLists {
    u64 table[kAloneSlots], found[P2_MAX_LEN + 1], path[kAloneNodes];
    uint32_t table_node[kAloneSlots], node_state[kAloneNodes], node_edges[kAloneNodes], planes[kAloneEdges * 8];
    u32x2 links[kAloneEdges];
};
struct InDevice {
    template <class T> using at = P2_GLOBAL T*;
    static constexpr int scope = __HIP_MEMORY_SCOPE_AGENT;
};
struct InBlock {
    template <class T> using at = P2_LOCAL T*;
    static constexpr int scope = __HIP_MEMORY_SCOPE_WORKGROUP;
};
template <class Where>
struct Skeleton {
    int n_pat, n_ops, max_len;
    uint32_t op_mask, op_ranks, cap_nodes, cap_found, cap_edges, table_mask;
    uint32_t k, size[kNarrowLevels];        // split: the group's own chunks and levels
    bool split;
    P2_GLOBAL GraphCounters* ctr;
    typename Where::template at<u64> found, table, node_path;
    typename Where::template at<uint32_t> table_node, node_state, node_edges, planes;
    typename Where::template at<u32x2> links;
    P2_GLOBAL uint32_t *use_ends, *use_list;
    P2_GLOBAL u32x2 *count2, *first_edge;
    P2_GLOBAL uint8_t* nearest;
};
template <class Where>
__device__ __forceinline__ void open_skeleton(Skeleton<Where>& G, const DevGraph& D) {
    G.n_pat = D.n_pat; G.n_ops = D.n_ops; G.max_len = D.max_len; G.op_mask = D.op_mask; G.op_ranks = D.op_ranks;
    G.cap_nodes = D.cap_nodes; G.cap_found = D.cap_found; G.cap_edges = D.cap_edges; G.table_mask = D.table_mask;
    G.split = D.split_check != 0u;
    G.k = D.own_chunks;
#pragma unroll
    for (int l = 0; l < kNarrowLevels; ++l) G.size[l] = D.own_size[l];
    G.ctr = in_global<GraphCounters>(D.ctr);
    G.use_ends = in_global<uint32_t>(D.use_ends); G.nearest = in_global<uint8_t>(D.nearest); G.use_list = in_global<uint32_t>(D.use_id); G.count2 = in_global<u32x2>(D.count2);
    G.first_edge = in_global<u32x2>(D.first_edge);
}
__device__ __forceinline__ Skeleton<InDevice> open_in_device(const DevGraph& D) {
    Skeleton<InDevice> G;
    open_skeleton(G, D);
    G.found = in_global<u64>(D.ctr->found); G.table = in_global<u64>(D.table); G.node_path = in_global<u64>(D.node_path);
    G.table_node = in_global<uint32_t>(D.table_node); G.node_state = in_global<uint32_t>(D.node_state); G.node_edges = in_global<uint32_t>(D.node_edges);
    G.planes = in_global<uint32_t>(D.narrow_planes); G.links = in_global<u32x2>(D.links);
    return G;
}
__device__ __forceinline__ Skeleton<InBlock> open_in_block(const DevGraph& D, AloneLists& A) {
    Skeleton<InBlock> G;
    open_skeleton(G, D);
    G.found = (P2_LOCAL u64*)A.found; G.table = (P2_LOCAL u64*)A.table; G.node_path = (P2_LOCAL u64*)A.path;
    G.table_node = (P2_LOCAL uint32_t*)A.table_node; G.node_state = (P2_LOCAL uint32_t*)A.node_state; G.node_edges = (P2_LOCAL uint32_t*)A.node_edges;
    G.planes = (P2_LOCAL uint32_t*)A.planes; G.links = (P2_LOCAL u32x2*)A.links;
    G.table_mask = kAloneSlots - 1u;
    if (G.cap_nodes > kAloneNodes) G.cap_nodes = kAloneNodes;
    if (G.cap_found > kAloneEdges) G.cap_found = kAloneEdges;
    return G;
}

// The word of the lane whose device differs in bit B.
template <int B>
__device__ __forceinline__ uint32_t across(uint32_t v) {
    static_assert(B >= 0 && B < 4, "within a row of 16 lanes");
    if constexpr (B == 0) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);          // quad_perm 1 0 3 2
    else if constexpr (B == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);     // quad_perm 2 3 0 1
    else if constexpr (B == 2)                                                                              // half mirror, quad_perm 3 2 1 0
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
    else return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);                          // row_ror 8
}
// f(bit's number) for every bit of the device number that `range` has, unrolled
template <int L, class F>
__device__ __forceinline__ void for_bits(uint32_t range, const F& f) {
    if constexpr (L > 0) if (range & 1u) f(std::integral_constant<int, 0>());
    if constexpr (L > 1) if (range & 2u) f(std::integral_constant<int, 1>());
    if constexpr (L > 2) if (range & 4u) f(std::integral_constant<int, 2>());
    if constexpr (L > 3) if (range & 8u) f(std::integral_constant<int, 3>());
}

// One device of a state: the masks of its rows, packed, the rows that have one, and where chunks are no multiple of the devices
// (split) the chunks that it holds.
template <int L>
struct Device {
    static constexpr int N = 1 << L, W = L <= 2 ? 1 : N * N / 32, kStride = N * (W + 1);       // (words of a state in memory: the masks, then rows | chunks << 16)
    static constexpr uint32_t kRows = (1u << N) - 1u, kWord = L == 1 ? 0xfu : L == 2 ? 0xffffu : 0xffffffffu;
    uint32_t w[W], rows, held;
    __device__ __forceinline__ bool full() const {
        uint32_t a = kWord;
#pragma unroll
        for (int i = 0; i < W; ++i) a &= w[i];
        return a == kWord;
    }
    template <class At>
    __device__ __forceinline__ void load(At at, int dev) {
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = at[dev * W + i];
        const uint32_t v = at[N * W + dev];
        rows = v & 0xffffu; held = v >> 16;
    }
    template <class At>
    __device__ __forceinline__ void store(At at, int dev) const {
#pragma unroll
        for (int i = 0; i < W; ++i) at[dev * W + i] = w[i];
        at[N * W + dev] = rows | held << 16;
    }
    // masks of the given rows
    static __device__ __forceinline__ uint32_t word_of(uint32_t rows, int i) {
        constexpr int per = N < 32 / N ? N : 32 / N;     // rows in a word
        uint32_t m = 0u;
#pragma unroll
        for (int j = 0; j < per; ++j) m |= (0u - (rows >> (i * per + j) & 1u)) & (kRows << (j * N));
        return m;
    }
};
// A wavefront's pattern and its lanes' devices.
template <int L>
struct Team {
    int lane, dev, base;
    uint32_t range;                         // varied bits of the device number
    int lg, ls;
    bool in;                                // the device takes part
    // f(bit) for the varied bits, and the word of the lane whose device differs in it.  Four levels: unrolled, DPP moves, for a level
    // there has instructions to issue for a third of its time.  Fewer: a loop and LDS exchanges, since what counts there is one block's time, and most of
    // that goes into fetching instructions for the first time ([3 4 6]: 11.1 us a level unrolled, 9.9 so).
    template <class F>
    __device__ __forceinline__ void each(const F& f) const {
        if constexpr (L == 4) for_bits<L>(range, f);
        else {
#pragma unroll 1
            for (int b = ls; b < ls + lg; ++b) f(b);
        }
    }
    template <int B>
    __device__ __forceinline__ uint32_t over(uint32_t v, std::integral_constant<int, B>) const { return across<B>(v); }
    __device__ __forceinline__ uint32_t over(uint32_t v, int b) const { return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ (1 << b)) << 2, (int)v); }
    // the first group member's word
    __device__ __forceinline__ uint32_t root(uint32_t v) const {
        if constexpr (L == 4) {
            for_bits<L>(range, [&](auto b) { const uint32_t o = across<b.value>(v); v = (dev >> b.value) & 1 ? o : v; });
            return v;
        } else return (uint32_t)__builtin_amdgcn_ds_bpermute((int)((uint32_t)lane & ~range) << 2, (int)v);
    }
};
struct Verdict { uint32_t kids, goals; };   // by op: the rule holds and the child is not the goal; it is the goal

// The same bits for all devices of a state: those that any of them has.
template <int L>
__device__ __forceinline__ uint32_t together(uint32_t bits) {
    for_bits<L>(0xfu, [&](auto b) { bits |= across<b.value>(bits); });
    return bits;
}
// A state and a pattern, by the state's lanes together (the rules of Sec. 3.2).  all: the group's members together, the masks and
// the rows; first: the group's first member.  What a device has against a rule is a bit of a word, and the words are put together
// once.
template <int L, class Where>
__device__ __forceinline__ Verdict judge(const Skeleton<Where>& G, const Team<L>& t, const Device<L>& own, Device<L>& all, Device<L>& first, bool active, bool last) {
    using Dev = Device<L>;
    uint32_t beyond = 0u, differ = 0u;                   // of the first member's: something that it has not, anything
#pragma unroll
    for (int i = 0; i < Dev::W; ++i) {
        first.w[i] = t.root(own.w[i]);
        beyond |= own.w[i] & ~first.w[i];
        differ |= own.w[i] ^ first.w[i];
    }
    first.rows = t.root(own.rows);
    all = own;
    uint32_t against = 0u, shared = 0u;                  // AllReduce: rows that differ, contributions in common; AllGather: rows in common
    t.each([&](auto b) {
#pragma unroll
        for (int i = 0; i < Dev::W; ++i) {
            const uint32_t o = t.over(all.w[i], b);
            against |= o & all.w[i];
            all.w[i] |= t.in ? o : 0u;
        }
        const uint32_t o = t.over(all.rows, b);
        against |= o ^ all.rows; shared |= o & all.rows;
        all.rows |= t.in ? o : 0u;
        differ |= t.over(differ, b);                     // (in every group some member must differ from the first)
    });
    bool uneven = (__popc(own.rows) & ((1 << t.lg) - 1)) != 0;
    if (G.split) {                                       // (a group's chunks may not divide where its rows, as many as devices, do)
        uint32_t g = 1u;
        for_bits<L>(t.range, [&](auto b) { g *= G.size[b.value]; });
        uneven |= own.held % g != 0u;
    }
    const bool own_full = own.full(), all_full = all.full(), first_full = first.full();
    uint32_t f = t.in ? (against != 0u ? 1u : 0u) | (shared != 0u || own.rows == 0u ? 2u : 0u) | (beyond != 0u || differ == 0u ? 4u : 0u) | (own.rows != 0u ? 8u : 0u) |
                            (all_full ? 0u : 16u) | (first_full ? 0u : 32u) | (uneven ? 64u : 0u)
                      : own_full ? 0u : 48u;
    f = together<L>(f);
    const uint32_t holds = ((f & 9u) == 8u ? 1u << OP_AR | 1u << OP_RD | ((f & 64u) == 0u ? 1u << OP_RS : 0u) : 0u) | ((f & 2u) == 0u ? 1u << OP_AG : 0u) |
                           ((f & 4u) == 0u ? 1u << OP_BC : 0u);
    Verdict V;
    // (a Reduce leaves devices with nothing and a ReduceScatter with a part: neither ends at the goal)
    V.goals = active ? holds & G.op_mask & (((f & 16u) == 0u ? 1u << OP_AR | 1u << OP_AG : 0u) | ((f & 32u) == 0u ? 1u << OP_BC : 0u)) : 0u;
    V.kids = active && !last ? holds & G.op_mask & ~V.goals : 0u;
    return V;
}

// `rows` without its `n` lowest
__device__ __forceinline__ uint32_t without_lowest(uint32_t rows, int n) {
    for (int i = 0; i < n; ++i) rows &= rows - 1u;
    return rows;
}
// The child of a state under an instruction whose rule holds (op: the same for the wavefront).
template <int L, class Where>
__device__ __forceinline__ void make_child(Device<L>& ch, const Skeleton<Where>& G, const Team<L>& t, const Device<L>& own, const Device<L>& all, const Device<L>& first, int op) {
    using Dev = Device<L>;
    uint32_t keep = Dev::kRows;                          // rows that stay with the device
    if (op == OP_RD) keep = ((uint32_t)t.dev & t.range) != 0u ? 0u : Dev::kRows;
    if (op == OP_RS) {
        // the member of rank p keeps the p-th block of the rows in ascending order
        const int per = __popc(own.rows) >> t.lg, p = (t.dev >> t.ls) & ((1 << t.lg) - 1);
        const uint32_t from = without_lowest(own.rows, t.in ? p * per : 0);
        keep = from & ~without_lowest(from, per);
    }
    const bool bc = op == OP_BC, part = op == OP_RD || op == OP_RS;
#pragma unroll
    for (int i = 0; i < Dev::W; ++i) {
        uint32_t v = bc ? first.w[i] : all.w[i];
        if (part) v &= Dev::word_of(keep, i);
        ch.w[i] = t.in ? v : own.w[i];
    }
    const uint32_t rows = (bc ? first.rows : all.rows) & keep;
    ch.rows = t.in ? rows : own.rows;
    ch.held = own.held;
    if (G.split) {
        uint32_t c = own.held;
        if (op == OP_RS) {
            uint32_t g = 1u;
            for_bits<L>(t.range, [&](auto b) { g *= G.size[b.value]; });
            c /= g;
        } else if (op == OP_AG) {
            for_bits<L>(t.range, [&](auto b) {
                const uint32_t o = across<b.value>(c);
                const bool upper = ((t.dev >> b.value) & 1) != 0;
                c = (upper ? o : c) + (upper ? c : o) * (G.size[b.value] - 1u);
            });
        } else if (op == OP_RD) c = keep == 0u ? 0u : c;
        else if (bc) c = t.root(c);
        ch.held = t.in ? c : own.held;
    }
}
template <int L>
__device__ __forceinline__ u64 hash_of(const Device<L>& d, int dev) {
    constexpr uint32_t key[8] = {0x9e3779b1u, 0x85ebca77u, 0xc2b2ae3du, 0x27d4eb2fu, 0x165667b1u, 0xd3a2646du, 0xfd7046c5u, 0xb55a4f09u};
    u64 x = (u64)(d.rows | d.held << 16) * 0x94d049bb133111ebull;
#pragma unroll
    for (int i = 0; i < Device<L>::W; ++i) x += (u64)d.w[i] * (u64)key[i];
    x ^= x >> 29;
    u64 h = (x + (u64)(uint32_t)(dev + 1) * 0x9e3779b97f4a7c15ull) * 0xbf58476d1ce4e5b9ull;
    h ^= h >> 32;
    for_bits<L>(0xfu, [&](auto b) { h += (u64)across<b.value>((uint32_t)h) | (u64)across<b.value>((uint32_t)(h >> 32)) << 32; });
    return h == 0ull ? 1ull : h;
}
// Inclusive sums over the wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);     // row_shr 1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);     // the rows before: row_bcast 15, 31
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
    return v;
}

// The level's nodes and the edges that led to them, as far as there was room.
struct Range { uint32_t first, count, edge0, edges, next_first, next_edge; };
template <class Where>
__device__ __forceinline__ Range range_of(const Skeleton<Where>& G, int level) {
    // (these counts do not change while the level is worked on; a list that has outgrown its room, which the call will say
    //  and repeat, is read as far as it was written)
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const u64 f = lane >= 1 && lane <= level ? G.found[lane] : 0ull;
    const uint32_t nodes = lane == 0 ? 1u : (uint32_t)f, edges = (uint32_t)(f >> 32), nodes_upto = wave_scan(nodes), edges_upto = wave_scan(edges);
    Range r;
    r.count = (uint32_t)__builtin_amdgcn_readlane((int)nodes, level); r.edges = (uint32_t)__builtin_amdgcn_readlane((int)edges, level);
    r.next_first = (uint32_t)__builtin_amdgcn_readlane((int)nodes_upto, level); r.next_edge = (uint32_t)__builtin_amdgcn_readlane((int)edges_upto, level);
    r.first = r.next_first - r.count; r.edge0 = r.next_edge - r.edges;
    if (r.first > G.cap_nodes) r.first = G.cap_nodes;
    if (r.count > G.cap_nodes - r.first) r.count = G.cap_nodes - r.first;
    if (r.edge0 > G.cap_found) r.edge0 = G.cap_found;
    if (r.edges > G.cap_found - r.edge0) r.edges = G.cap_found - r.edge0;
    return r;
}

// The states first reached by `level` instructions, judged against every pattern by block `block` of n_blocks, and the children of
// what holds built and looked up.
template <int L, class Where>
__device__ void skeleton_level(const Skeleton<Where>& G, LevelShared& S, int level, uint32_t block, uint32_t n_blocks) {
    using Dev = Device<L>;
    constexpr int N = Dev::N, kTeams = kWave / N;
    const uint32_t tid = threadIdx.x;
    const int n_pat = G.n_pat;
    const bool last = level + 1 >= G.max_len;
    const Range range = range_of(G, level);
    const uint32_t first = range.first, count = range.count;
    Team<L> t;
    t.lane = (int)(tid & (kWave - 1));
    t.dev = t.lane & (N - 1);
    t.base = t.lane & ~(N - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(tid / kWave)), team = t.lane >> L;
    int subs = kLevelWaves / n_pat;
    if (subs * kTeams * n_pat > kEntries) subs = kEntries / (kTeams * n_pat);
    const uint32_t per_block = (uint32_t)(subs * kTeams);
    const int sub = wave / n_pat, pat = wave - sub * n_pat;
    const bool judges = sub < subs;
    const uint32_t shape = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.shape[judges ? pat : 0]);
    t.lg = (int)(shape & 15u); t.ls = (int)(shape >> 4);
    t.range = ((1u << t.lg) - 1u) << t.ls;
    t.in = (S.part[judges ? pat : 0] >> t.dev & 1u) != 0u;
    uint32_t flags = 0u;
    if (level == 0 && block == 0u && tid == 0) { G.node_path[0] = 0ull; G.node_state[0] = 0u; }
    for (uint32_t g0 = block * per_block; g0 < count; g0 += n_blocks * per_block) {
        const uint32_t local = (uint32_t)(sub * kTeams + team), entry = local * (uint32_t)n_pat + (uint32_t)pat;
        const bool active = judges && g0 + local < count;
        const uint32_t node = first + g0 + (active ? local : 0u);
        Dev own, all, root;
        // Sec. 3.5: device i holds column i in every row
#pragma unroll
        for (int i = 0; i < Dev::W; ++i) own.w[i] = (L == 1 ? 5u : L == 2 ? 0x1111u : L == 3 ? 0x01010101u : 0x00010001u) << t.dev;
        own.rows = Dev::kRows; own.held = G.split ? G.k : 0u;
        Verdict V{0u, 0u};
        if (judges) {
            u64 path = 0ull;
            if (level > 0) {
                path = G.node_path[node];
                own.load(G.planes + (size_t)G.node_state[node] * Dev::kStride, t.dev);
            }
            bool go = active;
            // The goal can only come from an AllReduce on devices that all hold every row, an AllGather on devices whose rows
            // all carry every column, or a Broadcast whose roots, device 0 among them, are at the goal.
            if (last) {
                uint32_t bits = 0u;
#pragma unroll
                for (int i = 0; i < Dev::W; ++i) bits += (uint32_t)__popc(own.w[i]);
                const bool r_off = own.rows != Dev::kRows, m_off = own.rows == 0u || bits != (uint32_t)__popc(own.rows) * N;
                go = active && together<L>((r_off ? 1u : 0u) | (m_off ? 2u : 0u) | (t.dev == 0 && (r_off || m_off) ? 4u : 0u)) != 7u;
            }
            if (__any(go)) V = judge<L>(G, t, own, all, root, go, last);
            if (t.dev == 0) {
                S.code[entry] = (uint16_t)(V.kids | V.goals << 5);
                if (pat == 0) S.path[local] = path;
            }
        }
        const bool leader = t.dev == 0;
        __syncthreads();
        // the edges' places within the block, state by state, in the order of the digits (four entries a lane, every wavefront for
        // itself); goals in the upper halves
        uint32_t sums, packed = 0u, total;
        {
            const uint2 codes = reinterpret_cast<const uint2*>(S.code)[t.lane];
            const uint32_t c[4] = {codes.x & 0xffffu, codes.x >> 16, codes.y & 0xffffu, codes.y >> 16};
            uint32_t run = 0u;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                packed |= (run & 15u) << (4 * x) | (run >> 16) << (16 + 4 * x);
                run += (uint32_t)__popc(c[x]) | (uint32_t)__popc(c[x] >> 5) << 16;
            }
            const uint32_t upto = wave_scan(run);
            sums = upto - run;
            total = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
        }
        const uint32_t n_edges = total & 0xffffu;
        auto before = [&](uint32_t e) {                    // edges | goals << 16 before entry e (all lanes ask)
            const uint32_t p = (uint32_t)__shfl((int)packed, (int)(e >> 2), kWave) >> (4u * (e & 3u));
            return (uint32_t)__shfl((int)sums, (int)(e >> 2), kWave) + (p & 15u) + (p & 0xf0000u);
        };
        const uint32_t both = V.kids | V.goals, at = before(judges ? entry : 0u) & 0xffffu;
        uint32_t base = 0u;
        // built twice, for the hash and, once every edge has its place, for the lists (a child is a few selections)
#pragma unroll 1
        for (int pass = 0; pass < 2 && n_edges != 0u; ++pass) {
            if (pass == 1) {
                __syncthreads();
                // the children looked up, a lane each (a second one where a block of small states has more edges than threads)
                uint32_t slot[2] = {kGoalEdge, kGoalEdge};
                bool fresh[2] = {false, false};
                uint32_t n_fresh = 0u;
    #pragma unroll
                for (uint32_t x = 0; x < 2u; ++x) {
                    if ((uint32_t)wave * kWave + x * kLevelThreads >= n_edges) continue;
                    const uint32_t le = tid + x * kLevelThreads;
                    const u64 h = le < n_edges ? S.hash[le] : 0ull;
                    if (h != 0ull) {
                        uint32_t s = (uint32_t)h & G.table_mask, tries = 0u;
#pragma unroll 1
                        for (; tries < kMostTries; ++tries) {  // (the table is at most half full while the nodes have room)
                            u64 old = 0ull;
                            fresh[x] = __hip_atomic_compare_exchange_strong(G.table + s, &old, h, __ATOMIC_RELAXED, __ATOMIC_RELAXED, Where::scope);
                            if (fresh[x] || old == h) break;
                            s = (s + 1u) & G.table_mask;
                        }
                        if (tries >= kMostTries) { flags |= kGraphFull; fresh[x] = false; s = 0u; }
                        slot[x] = s;
                    }
                    n_fresh += (uint32_t)__popcll(__ballot(fresh[x]));
                }
                if (t.lane == 0) S.fresh[wave] = n_fresh;
                __syncthreads();
                // (one addition a block: those to one address take turns, some 18 ns each)
                uint32_t rank = 0u;
                if (wave == 0) {
                    const uint32_t v = t.lane < kLevelWaves ? S.fresh[t.lane] : 0u, upto = wave_scan(v);
                    if (t.lane < kLevelWaves) S.fresh[t.lane] = upto - v;
                    if (t.lane == kLevelWaves - 1) {
                        const u64 was = __hip_atomic_fetch_add(G.found + level + 1, (u64)n_edges << 32 | upto, __ATOMIC_RELAXED, Where::scope);
                        S.base = range.next_edge + (uint32_t)(was >> 32); S.node0 = range.next_first + (uint32_t)was;
                    }
                }
                __syncthreads();
                base = S.base;
                rank = S.node0 + S.fresh[wave];
    #pragma unroll
                for (uint32_t x = 0; x < 2u; ++x) {
                    if ((uint32_t)wave * kWave + x * kLevelThreads >= n_edges) continue;
                    const uint32_t le = tid + x * kLevelThreads, e = base + le;
                    const u64 firsts = __ballot(fresh[x]);
                    const uint32_t n = rank + (uint32_t)__popcll(firsts & ((1ull << t.lane) - 1ull));
                    rank += (uint32_t)__popcll(firsts);
                    if (le >= n_edges) continue;
                    const uint32_t edge = S.edge[le], digit = edge >> 16, from = edge & 0xffffu;
                    if (fresh[x] && n < G.cap_nodes) {
                        G.node_state[n] = e < G.cap_found ? e : 0u;
                        G.node_path[n] = S.path[from] << 8 | (digit + 1u);
                        G.table_node[slot[x]] = n + 1u;
                    } else if (fresh[x]) flags |= kGraphFull;
                    if (e < G.cap_found) G.links[e] = u32x2{(first + g0 + from) | digit << kDigitShift, slot[x] | (fresh[x] ? kFreshEdge : 0u)};
                    else flags |= kGraphFull;
                }
            }
#pragma unroll 1
            for (int op = 0; op < 5; ++op) {
                const bool kid = ((V.kids >> op) & 1u) != 0u, edge = ((both >> op) & 1u) != 0u;
                if (!__any(pass == 0 ? edge : kid)) continue;
                const uint32_t le = at + (uint32_t)__popc(both & ((1u << op) - 1u));
                Dev ch;
                make_child<L>(ch, G, t, own, all, root, op);
                if (pass == 0) {
                    const u64 h = hash_of<L>(ch, t.dev);
                    if (leader && edge) {
                        S.hash[le] = kid ? h : 0ull;
                        S.edge[le] = local | ((uint32_t)pat * (uint32_t)G.n_ops + ((G.op_ranks >> (4 * op)) & 15u)) << 16;
                    }
                } else if (kid && base + le < G.cap_found) ch.store(G.planes + (size_t)(base + le) * Dev::kStride, t.dev);
            }
        }
        // where a state's edges are: the first, how many, how many of them goals
        if (wave == kLevelWaves - 1)
            for (uint32_t i0 = 0; i0 < per_block; i0 += kWave) {
                const uint32_t i = i0 + (uint32_t)t.lane, e0 = i * (uint32_t)n_pat, e1 = e0 + (uint32_t)n_pat;
                const uint32_t from = before(e0 < kEntries ? e0 : 0u), to = before(e1 < kEntries ? e1 : 0u), end = e1 < kEntries ? to : total;
                if (i < per_block && g0 + i < count)
                    G.node_edges[first + g0 + i] = n_edges == 0u ? 0u : (S.base + (from & 0xffffu)) << 14 | ((end - from) & 0xffffu) << 7 | (end - from) >> 16;
            }
        __syncthreads();
    }
    if (flags != 0u) atomicOr(&S.flags, flags);
}
// The edges that led to a level get their nodes, and what the level before found to have the hash of an earlier state is compared
// with it, by thread `at` of `step`.
template <int L, class Where>
__device__ void skeleton_links(const Skeleton<Where>& G, LevelShared& S, int level, uint32_t at, uint32_t step) {
    using Dev = Device<L>;
    constexpr uint32_t N = Dev::N;
    const Range range = range_of(G, level);
    const int dev = (int)(threadIdx.x & (N - 1u));
    uint32_t flags = 0u;
    for (uint32_t e = range.edge0 + at / N; e < range.edge0 + range.edges; e += step / N) {
        const u32x2 link = G.links[e];
        const uint32_t slot = link.y & kSlotMask;
        if (slot == kGoalEdge) continue;
        const uint32_t n = G.table_node[slot];
        if (n == 0u || n > G.cap_nodes) { flags |= kGraphFull; continue; }
        if ((link.y & kFreshEdge) == 0u) {
            Dev a, b;
            a.load(G.planes + (size_t)e * Dev::kStride, dev);
            b.load(G.planes + (size_t)G.node_state[n - 1u] * Dev::kStride, dev);
            bool differ = a.rows != b.rows || a.held != b.held;
#pragma unroll
            for (int i = 0; i < Dev::W; ++i) differ |= a.w[i] != b.w[i];
            if (differ) flags |= kGraphCollision;
        }
        if (dev == 0) G.links[e] = u32x2{link.x, n - 1u};
    }
    if (flags != 0u) atomicOr(&S.flags, flags);
}

struct FinishShared {
    uint32_t end[P2_MAX_LEN + 1], lim[P2_MAX_LEN + 1], at[P2_MAX_LEN + 1];       // nodes first reached by at most d instructions; how many nodes count r is kept for, and where
    uint32_t edges, targets, valid;
    u64 used;                               // nodes on the way to a goal | their edges << 32
};

constexpr uint32_t kFewEdges = 4;            // edges of a thread where they are counted edge by edge

// The counts of every node, from one instruction left to the size limit, by one block.  Count r of a node that `d` instructions
// reach first is asked for up to r = max_len - d, so the lists of counts get short quickly (16 798 nodes: 7 880 counts for r =
// 2, then 2 500, 495, 48 and 1).  They stay in LDS, the first one (goals, at most 80) as bytes.
//  `few` (every graph of the launch has room for at most kFewEdges * T edges; [3 4 6] has some 1 200): a thread for every edge and
// both kinds of count at once.  The additions to a node's count take turns, up to some forty of a cycle or two, where its walk
// along as many edges would be a chain of LDS reads.
//  Otherwise k_skeleton_two has left count 2, and every further round is a walk of each node along its own edges, whose targets
// stay in LDS as well; first for the programs whose rules all hold, short of the goal, then for those that end there.
// [2 4 8 8], six levels: 37 us and 8 of k_skeleton_two; 71 us where the block did all of it.
template <int T, bool few, class Where>
__device__ void skeleton_finish(const Skeleton<Where>& G, FinishShared& S, uint32_t* scratch, uint32_t words) {
    const uint32_t tid = threadIdx.x;
    P2_GLOBAL GraphCounters* const ctr = G.ctr;
    const int M = G.max_len;
    if (tid < kWave) {
        const u64 f = tid >= 1u && tid <= (uint32_t)M ? G.found[tid] : 0ull;
        const uint32_t end = wave_scan(tid == 0u ? 1u : tid < (uint32_t)M ? (uint32_t)f : 0u), edges = wave_scan((uint32_t)(f >> 32));
        const uint32_t mirror = __shfl(end, M - (int)tid < 0 ? 0 : M - (int)tid, kWave), lim = tid >= 2u && tid <= (uint32_t)M ? mirror : 0u, at = wave_scan(lim);
        if (tid <= P2_MAX_LEN) { S.end[tid] = end; S.lim[tid] = lim; S.at[tid] = at - lim; }
        if (tid == P2_MAX_LEN) { S.edges = edges; S.used = 0ull; }
        if ((int)tid == (M > 2 ? M - 2 : 0)) S.targets = edges;
    }
    __syncthreads();
    const uint32_t n_nodes = S.end[P2_MAX_LEN], n_edges = S.edges, n_words = S.at[P2_MAX_LEN] + S.lim[P2_MAX_LEN];
    // (the rounds after the second follow the edges of nodes that at most max_len - 3 instructions reach)
    const uint32_t n_targets = few ? 0u : S.targets;
    const uint32_t byte_words = (n_nodes + 3u) / 4u, target_words = (n_targets + 1u) / 2u;
    if (3u * byte_words + target_words + (few ? 2u : 1u) * n_words > words || n_nodes > 0xfff0u || (few && n_edges > kFewEdges * T)) {
        if (tid == 0) ctr->flags = kGraphPairs;          // (no structure that has_skeleton lets through has as many states)
        return;
    }
    uint8_t* const goal1 = reinterpret_cast<uint8_t*>(scratch);                        // programs of one instruction to the goal
    uint8_t* const prefix1 = reinterpret_cast<uint8_t*>(scratch + byte_words);         // ... short of it
    uint8_t* const nearest = reinterpret_cast<uint8_t*>(scratch + 2u * byte_words);    // instructions of the shortest program to the goal; 255: none
    uint16_t* const target = reinterpret_cast<uint16_t*>(scratch + 3u * byte_words);
    uint32_t* const count = scratch + 3u * byte_words + target_words;
    auto note = [&](uint32_t n, uint32_t r) {
        goal1[n] = (uint8_t)(r & 127u); prefix1[n] = (uint8_t)((r >> 7 & 127u) - (r & 127u)); nearest[n] = (r & 127u) != 0u ? 1 : 255;
    };
    for (uint32_t n0 = tid; n0 < n_nodes; n0 += 8u * T) {
        uint32_t r[8];
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) r[j] = n0 + j * T < n_nodes ? G.node_edges[n0 + j * T] : 0u;
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) if (n0 + j * T < n_nodes) note(n0 + j * T, r[j]);
    }
    for (uint32_t e0 = tid; e0 < n_targets; e0 += 8u * T) {
        uint32_t to[8];
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) to[j] = e0 + j * T < n_targets ? G.links[e0 + j * T].y : kGoalEdge;
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) if (e0 + j * T < n_targets) target[e0 + j * T] = (uint16_t)(to[j] == kGoalEdge ? 0xffffu : to[j]);
    }
    __syncthreads();
    if constexpr (few) {
        uint32_t* const prefixes = count + n_words;
        for (uint32_t x = tid; x < 2u * n_words; x += T) count[x] = 0u;
        uint32_t from[kFewEdges], to[kFewEdges];
#pragma unroll
        for (uint32_t j = 0; j < kFewEdges; ++j) {
            const uint32_t e = tid + j * T;
            const u32x2 l = e < n_edges ? G.links[e] : u32x2{0u, kGoalEdge};
            from[j] = l.x & kGoalEdge; to[j] = l.y;
        }
        __syncthreads();
        for (int r = 2; r <= M; ++r) {
            const uint32_t lim = S.lim[r], at = S.at[r], before = S.at[r - 1];
#pragma unroll
            for (uint32_t j = 0; j < kFewEdges; ++j) {
                if (to[j] == kGoalEdge || from[j] >= lim) continue;
                const uint32_t g = r == 2 ? (uint32_t)goal1[to[j]] : count[before + to[j]], p = r == 2 ? (uint32_t)prefix1[to[j]] : prefixes[before + to[j]];
                if (g != 0u) {
                    atomicAdd(&count[at + from[j]], g);
                    if (nearest[from[j]] == 255) nearest[from[j]] = (uint8_t)r;       // (whoever comes first: all write the same)
                }
                if (p != 0u) atomicAdd(&prefixes[at + from[j]], p);
            }
            __syncthreads();
        }
        if (tid >= 1u && tid <= (uint32_t)M) {
            ctr->n_valid[tid] = tid == 1u ? (uint32_t)goal1[0] : count[S.at[tid]];
            if (tid < (uint32_t)M) ctr->n_prefixes[tid] = tid == 1u ? (uint32_t)prefix1[0] : prefixes[S.at[tid]];
        }
    } else for (int kind = 0; kind < 2; ++kind) {
        const uint8_t* const one = kind == 0 ? prefix1 : goal1;
        for (uint32_t n0 = tid; n0 < S.lim[2]; n0 += 8u * T) {
            u32x2 c[8];
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) c[j] = n0 + j * T < S.lim[2] ? G.count2[n0 + j * T] : u32x2{0u, 0u};
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) {
                const uint32_t n = n0 + j * T;
                if (n >= S.lim[2]) continue;
                count[n] = kind == 0 ? c[j].y : c[j].x;
                if (kind == 1 && c[j].x != 0u && nearest[n] == 255) nearest[n] = 2;
            }
        }
        __syncthreads();
        for (int r = 3; r <= M; ++r) {
            const uint32_t lim = S.lim[r], at = S.at[r], before = S.at[r - 1];
            // (the nodes of the first levels have up to forty edges: sixteen lanes to one)
            const uint32_t lanes = r >= 4 ? 16u : 1u, own_lane = tid & (lanes - 1u);
            for (uint32_t n = tid / lanes; n < lim; n += T / lanes) {
                const uint32_t own = G.node_edges[n], end = (own >> 14) + (own >> 7 & 127u);
                uint32_t s = 0u;
                for (uint32_t e = (own >> 14) + own_lane; e < end; e += 4u * lanes) {     // (four edges in flight)
                    uint32_t to[4], n_to[4];
#pragma unroll
                    for (uint32_t x = 0; x < 4u; ++x) to[x] = e + x * lanes < end ? (uint32_t)target[e + x * lanes] : 0xffffu;
#pragma unroll
                    for (uint32_t x = 0; x < 4u; ++x) n_to[x] = count[before + (to[x] != 0xffffu ? to[x] : 0u)];
#pragma unroll
                    for (uint32_t x = 0; x < 4u; ++x) s += to[x] != 0xffffu ? n_to[x] : 0u;
                }
                if (lanes > 1u) { s += across<0>(s); s += across<1>(s); s += across<2>(s); s += across<3>(s); }
                if (own_lane == 0u) {
                    count[at + n] = s;
                    if (kind == 1 && s != 0u && nearest[n] == 255) nearest[n] = (uint8_t)r;
                }
            }
            __syncthreads();
        }
        if (tid >= 1u && tid <= (uint32_t)M) {
            const uint32_t n = tid == 1u ? (uint32_t)one[0] : count[S.at[tid]];
            if (kind == 1) ctr->n_valid[tid] = n;
            else if (tid < (uint32_t)M) ctr->n_prefixes[tid] = n;
        }
        __syncthreads();
    }
    if (tid < kWave) {
        const uint32_t all = wave_scan(tid == 1u ? (uint32_t)goal1[0] : tid >= 2u && tid <= (uint32_t)M ? count[S.at[tid]] : 0u);
        if (tid == kWave - 1) { S.valid = all; ctr->n_judged = n_nodes; }
    }
    // the nodes on the way to a goal, in any order, what lies behind them, and room for their edges (one after the other: what is kept of
    // every edge and query is sized by these, 8 765 of the 31 660 edges of four levels and six instructions)
    for (uint32_t n = tid; n < (n_nodes + kWave - 1u) / kWave * kWave; n += T) {
        const uint32_t lane = tid & (kWave - 1u);
        const uint8_t near = n < n_nodes ? nearest[n] : 255;
        const u64 used = __ballot(near != 255);
        const uint32_t own = near != 255 ? (uint32_t)goal1[n] + (uint32_t)prefix1[n] : 0u, upto = wave_scan(own);
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
        u64 was = 0ull;
        if (lane == 0u && used != 0ull) was = atomicAdd(&S.used, (u64)__popcll(used) | (u64)all << 32);
        const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)was) + (uint32_t)__popcll(used & ((1ull << lane) - 1ull));
        const uint32_t place = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(was >> 32)) + upto - own;
        if (n < n_nodes) G.nearest[n] = near;
        if (near == 255) continue;
        G.use_list[at] = n;
        G.first_edge[n] = u32x2{place, place};
        u32x4 lo = {0u, goal1[n], 0u, 0u}, hi = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 2; r <= P2_MAX_LEN; ++r) {
            const uint32_t c = r <= M && n < S.lim[r] ? count[S.at[r] + n] : 0u;
            if (r < 4) lo[r] = c; else hi[r - 4] = c;
        }
        P2_GLOBAL u32x4* const out = (P2_GLOBAL u32x4*)(G.use_ends + (size_t)n * 8);
        out[0] = lo; out[1] = hi;
    }
    __syncthreads();
    if (tid == 0) {
        // (no rows are written before the number of valid programs is)
        if ((uint32_t)(S.used >> 32) > G.cap_edges) ctr->flags = kGraphFull;
        else { ctr->n_edges = (uint32_t)S.used; ctr->n_total = S.valid; }
    }
}

// A block's graph, and its place among the graph's blocks.
struct Place { uint32_t graph, block, blocks, links; };
__device__ __forceinline__ Place place_of(const SkeletonGrid& grid, uint32_t at) {
    Place p{0u, at, 0u, 0u};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const uint32_t per = grid.blocks[c] + grid.links[c], all = grid.graphs[c] * per;
        if (p.blocks != 0u) continue;
        if (p.block >= all) { p.block -= all; p.graph += grid.graphs[c]; continue; }
        if (grid.graphs[c] > 1u) { const uint32_t g = p.block / per; p.graph += g; p.block -= g * per; }
        p.blocks = grid.blocks[c]; p.links = grid.links[c];
    }
    return p;
}

__device__ __forceinline__ void open_level(LevelShared& S, const DevGraph& D) {
    if ((int)threadIdx.x < kEntryPatterns) { S.shape[threadIdx.x] = D.shape[threadIdx.x]; S.part[threadIdx.x] = (uint32_t)D.part[threadIdx.x]; }
    if (threadIdx.x < kEntries) S.code[threadIdx.x] = 0;
    if (threadIdx.x == 0) S.flags = 0u;
    __syncthreads();
}
// One level of the graphs: the last blocks of a graph work on the edges that led to the level, the others on its states.  Bound by the
// chain of one block's steps where a level has few states (three levels: some 10 us a launch).  Where it has many, vector instructions
// take a third of the time to issue and the wavefronts wait for 60 to 70 % of theirs, for the block's barriers, the table and the nodes'
// states: [2 4 8 8], six levels, 193 us, where a team of lanes per (state, pattern) in p2_graph.hip takes 382; a third of that is the
// fifth level, 5 400 states.
// Every graph gets the blocks that its levels can do with: with those of the largest for all of them, 300 of three levels beside one
// of four took 2 270 us a call, and 949 on their own devices.
template <int L>
__device__ void level_of(const Skeleton<InDevice>& G, LevelShared& S, int level, const Place& p) {
    if (p.block < p.blocks) skeleton_level<L>(G, S, level, p.block, p.blocks);
    else skeleton_links<L>(G, S, level, (p.block - p.blocks) * kLevelThreads + threadIdx.x, p.links * kLevelThreads);
}
__global__ __launch_bounds__(kLevelThreads) void k_skeleton_level(const DevGraph* __restrict__ graphs, SkeletonGrid grid, int level) {
    __shared__ LevelShared S;
    const Place p = place_of(grid, blockIdx.x);
    const DevGraph& D = graphs[p.graph];
    const Skeleton<InDevice> G = open_in_device(D);
    if (level >= G.max_len) return;
    open_level(S, D);
    switch (D.R) {
    case 2: level_of<1>(G, S, level, p); break;
    case 4: level_of<2>(G, S, level, p); break;
    case 8: level_of<3>(G, S, level, p); break;
    default: level_of<4>(G, S, level, p); break;
    }
    __syncthreads();
    if (threadIdx.x == 0 && S.flags != 0u) atomicOr(&D.ctr->flags, S.flags);
}

// The programs of two instructions from every node, to the goal and short of it, which the edges of its children are enough for: by
// many blocks, for with four levels two thirds of the counting is this.
__global__ __launch_bounds__(256) void k_skeleton_two(const DevGraph* __restrict__ graphs, SkeletonGrid grid) {
    const Place p = place_of(grid, blockIdx.x);
    const Skeleton<InDevice> G = open_in_device(graphs[p.graph]);
    const int lane = (int)(threadIdx.x & (kWave - 1));
    if (G.ctr->flags != 0u) return;
    // (count 2 is asked for where two instructions are left)
    const u64 f = lane >= 1 && lane <= G.max_len - 2 ? G.found[lane] : 0ull;
    const uint32_t lim = G.max_len < 2 ? 0u : 1u + (uint32_t)__builtin_amdgcn_readlane((int)wave_scan((uint32_t)f), kWave - 1);
    for (uint32_t n = p.block * 256u + threadIdx.x; n < lim; n += p.blocks * 256u) {
        const uint32_t own = G.node_edges[n], end = (own >> 14) + (own >> 7 & 127u);
        uint32_t goals = 0u, prefixes = 0u;
        for (uint32_t e = own >> 14; e < end; e += 4u) {
            uint32_t to[4], rec[4];
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x) to[x] = e + x < end ? G.links[e + x].y : kGoalEdge;
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x) rec[x] = to[x] != kGoalEdge ? G.node_edges[to[x]] : 0u;
#pragma unroll
            for (uint32_t x = 0; x < 4u; ++x) { goals += rec[x] & 127u; prefixes += (rec[x] >> 7 & 127u) - (rec[x] & 127u); }
        }
        G.count2[n] = u32x2{goals, prefixes};
    }
}

template <bool few>
__global__ __launch_bounds__(kFinishThreads) void k_skeleton_finish(const DevGraph* __restrict__ graphs, uint32_t words) {
    extern __shared__ __attribute__((aligned(16))) uint32_t scratch[];
    __shared__ FinishShared S;
    const Skeleton<InDevice> G = open_in_device(graphs[blockIdx.x]);
    const uint32_t trouble = G.ctr->flags;
    __syncthreads();                                     // (every thread has read it before the block can set it)
    if (trouble == 0u) skeleton_finish<kFinishThreads, few>(G, S, scratch, words);
}

// Skeletons of one or two levels: a block goes through all levels and the counts by itself, with everything in LDS.  Bound by the chain
// of one block's steps, some 4 us a level: [2 4], three levels, 21 us, [4 16], five, 30, where p2_graph.hip's takes 27 and 39.
template <int L>
__device__ void alone_of(const Skeleton<InBlock>& G, LevelShared& S) {
    for (int level = 0; level < G.max_len; ++level) {
        skeleton_level<L>(G, S, level, 0u, 1u);
        skeleton_links<L>(G, S, level, threadIdx.x, kAloneThreads);
        __syncthreads();
    }
}
__global__ __launch_bounds__(kAloneThreads) void k_skeleton_alone(const DevGraph* __restrict__ graphs) {
    __shared__ LevelShared S;
    __shared__ AloneLists A;
    __shared__ FinishShared F;
    __shared__ __attribute__((aligned(16))) uint32_t scratch[kAloneScratch];
    const DevGraph& D = graphs[blockIdx.x];
    const Skeleton<InBlock> G = open_in_block(D, A);
    for (uint32_t x = threadIdx.x; x < kAloneSlots; x += kAloneThreads) { A.table[x] = 0ull; A.table_node[x] = 0u; }
    if (threadIdx.x <= P2_MAX_LEN) A.found[threadIdx.x] = 0ull;
    open_level(S, D);
    if (D.R == 2) alone_of<1>(G, S); else alone_of<2>(G, S);
    if (S.flags != 0u) {
        if (threadIdx.x == 0) G.ctr->flags = S.flags;
        return;
    }
    skeleton_finish<kAloneThreads, true>(G, F, scratch, kAloneScratch);
    // (for the costs)
    if (threadIdx.x < F.end[P2_MAX_LEN]) {
        in_global<uint32_t>(D.node_edges)[threadIdx.x] = A.node_edges[threadIdx.x];
        in_global<u64>(D.node_path)[threadIdx.x] = A.path[threadIdx.x];
    }
    if (threadIdx.x < F.edges) in_global<u32x2>(D.links)[threadIdx.x] = A.links[threadIdx.x];
}

// The edges on the way to a goal, at the front of the room that their state's have, and what each adds to the bandwidth sum of every query: a
// block per state on the way to a goal, a wavefront for every fourth or eighth edge, a lane per query.  An edge is kept if the goal can be
// reached behind it with the instructions that are left there.
template <int LOG>
constexpr int kCostWaves = LOG <= 3 ? 8 : 4;      // (four levels: 17.5 us with four, 23 with eight; three: 11 and 9)
template <int LOG>
__global__ __launch_bounds__(kCostWaves<LOG> * kWave) void k_skeleton_costs(const DevQuery* __restrict__ queries, const DevGraph* __restrict__ graphs, SkeletonGrid grid, int with_costs) {
    __shared__ PatternTable T;
    const Place p = place_of(grid, blockIdx.x);
    const DevGraph& D = graphs[p.graph];
    const P2_GLOBAL GraphCounters* const ctr = in_global<const GraphCounters>(D.ctr);
    const uint32_t n_use = ctr->n_edges, n_members = (uint32_t)D.n_members, member = blockIdx.y * kWave + (threadIdx.x & (kWave - 1));
    if (ctr->flags != 0u || p.block >= n_use || blockIdx.y * kWave >= n_members) return;
    T.open(D, queries[D.query]);
    const P2_GLOBAL uint8_t* const nearest = in_global<const uint8_t>(D.nearest);
    const P2_GLOBAL uint32_t* const list = in_global<const uint32_t>(D.use_id);
    const P2_GLOBAL uint32_t* const node_edges = in_global<const uint32_t>(D.node_edges);
    const P2_GLOBAL u64* const node_path = in_global<const u64>(D.node_path);
    const P2_GLOBAL u32x2* const links = in_global<const u32x2>(D.links);
    P2_GLOBAL uint32_t* const edges = in_global<uint32_t>(D.edges);
    P2_GLOBAL u32x2* const first_edge = in_global<u32x2>(D.first_edge);
    P2_GLOBAL double* const best = in_global<double>(D.best);
    const bool mine = member < n_members;
    const P2_GLOBAL DevMember& own = in_global<const DevMember>(D.sizes)[mine ? member : 0u];
    const int M = D.max_len, R = D.R;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    __syncthreads();
    for (uint32_t u = p.block; u < n_use; u += p.blocks) {
        const uint32_t node = list[u], rec = node_edges[node], first = rec >> 14, count = rec >> 7 & 127u, place = first_edge[node].x;
        const u64 path = node_path[node];
        int left = M - 1;
        for (u64 x = path; x != 0ull; x >>= 8) --left;
        bool kept[2];
        u32x2 link[2];
        u64 keepers[2];
#pragma unroll
        for (uint32_t x = 0; x < 2u; ++x) {              // (at most 80 edges)
            const uint32_t j = lane + x * kWave;
            link[x] = j < count ? links[first + j] : u32x2{0u, 0u};
            const uint32_t near = j < count && link[x].y != kGoalEdge ? (uint32_t)nearest[link[x].y] : 0u;
            kept[x] = j < count && (int)near <= left;
            keepers[x] = __ballot(kept[x]);
        }
        const uint32_t n0 = (uint32_t)__popcll(keepers[0]), n_kept = n0 + (uint32_t)__popcll(keepers[1]);
        if (wave == 0u && blockIdx.y == 0u) {
            const u64 below = (1ull << lane) - 1ull;
            if (kept[0]) edges[place + (uint32_t)__popcll(keepers[0] & below)] = (link[0].x & ~kGoalEdge) | link[0].y;
            if (kept[1]) edges[place + n0 + (uint32_t)__popcll(keepers[1] & below)] = (link[1].x & ~kGoalEdge) | link[1].y;
            if (lane == 0u) ((P2_GLOBAL uint32_t*)(first_edge + node))[1] = place + n_kept;      // (the blocks of the other queries read the place)
        }
        if (with_costs == 0 || wave >= n_kept) continue;
        HeldRows<LOG> rows;
        rows.start(own, R);
        rows.follow(path, T);
        uint32_t at = 0u;
#pragma unroll
        for (uint32_t x = 0; x < 2u; ++x)
            for (u64 rest = keepers[x]; rest != 0ull; rest &= rest - 1ull, ++at) {
                if (at % kCostWaves<LOG> != wave) continue;
                const uint32_t digit = (uint32_t)__builtin_amdgcn_readlane((int)link[x].x, __ffsll((long long)rest) - 1) >> kDigitShift;
                const double b = rows.busiest(T.of(digit), own);
                if (mine) best[(size_t)(place + at) * n_members + member] = b;
            }
    }
}

}  // namespace

int skeleton_state_words(int levels) {
    return levels == 1 ? Device<1>::kStride : levels == 2 ? Device<2>::kStride : levels == 3 ? Device<3>::kStride : Device<4>::kStride;
}
hipError_t launch_skeleton_alone(const DevGraph* graphs, unsigned n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_skeleton_alone, dim3(n), dim3(kAloneThreads), 0, stream, graphs);
    return hipGetLastError();
}
static unsigned blocks_of(const SkeletonGrid& grid) {
    unsigned n = 0;
    for (int c = 0; c < 3; ++c) n += grid.graphs[c] * (grid.blocks[c] + grid.links[c]);
    return n;
}
hipError_t launch_skeleton_level(const DevGraph* graphs, const SkeletonGrid& grid, int level, hipStream_t stream) {
    if (blocks_of(grid) == 0) return hipSuccess;
    hipLaunchKernelGGL(k_skeleton_level, dim3(blocks_of(grid)), dim3(kLevelThreads), 0, stream, graphs, grid, level);
    return hipGetLastError();
}
static constexpr size_t kMostLds = 160 * 1024 - 1024;     // (beside what the block shares)
template <bool few>
static hipError_t launch_finish(const DevGraph* graphs, unsigned n, size_t bytes, hipStream_t stream) {
    if (bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_skeleton_finish<few>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMostLds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_skeleton_finish<few>, dim3(n), dim3(kFinishThreads), bytes, stream, graphs, (uint32_t)(bytes / 4));
    return hipGetLastError();
}
hipError_t launch_skeleton_finish(const DevGraph* graphs, const SkeletonGrid& grid, uint32_t most_nodes, uint32_t most_edges, int max_len, hipStream_t stream) {
    const unsigned n = grid.graphs[0] + grid.graphs[1] + grid.graphs[2];
    if (n == 0) return hipSuccess;
    // (edge by edge: for a node three bytes and two lists of counts, from two instructions)
    const size_t few = ((size_t)most_nodes + 3) / 4 * 12 + sizeof(uint32_t) * 2 * (size_t)(max_len > 1 ? max_len - 1 : 0) * most_nodes;
    if (most_edges <= kFewEdges * (uint32_t)kFinishThreads && few <= kMostLds) return launch_finish<true>(graphs, n, few, stream);
    hipLaunchKernelGGL(k_skeleton_two, dim3(blocks_of(grid)), dim3(256), 0, stream, graphs, grid);
    return launch_finish<false>(graphs, n, kMostLds, stream);
}

hipError_t launch_skeleton_costs(const DevQuery* queries, const DevGraph* graphs, const SkeletonGrid& grid, unsigned members, int with_costs, hipStream_t stream) {
    if (blocks_of(grid) == 0) return hipSuccess;
    const dim3 blocks(blocks_of(grid), (members + kWave - 1) / kWave);
    if (grid.graphs[2] > 0) hipLaunchKernelGGL(k_skeleton_costs<kNarrowLevels>, blocks, dim3(kCostWaves<kNarrowLevels> * kWave), 0, stream, queries, graphs, grid, with_costs);
    else if (grid.graphs[1] > 0) hipLaunchKernelGGL(k_skeleton_costs<3>, blocks, dim3(kCostWaves<3> * kWave), 0, stream, queries, graphs, grid, with_costs);
    else hipLaunchKernelGGL(k_skeleton_costs<2>, blocks, dim3(kCostWaves<2> * kWave), 0, stream, queries, graphs, grid, with_costs);
    return hipGetLastError();
}

}  // namespace p2
