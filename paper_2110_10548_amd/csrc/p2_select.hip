// Ordering kernels: rank-sort of the (few) valid candidate indices, and top-k selection of
// (cost, index) pairs by filtering against a bound (the simulator's shortlist, Sec. 5).
#include "p2_device.h"

#include <mutex>

namespace p2 {

namespace {

constexpr int kWave = 64;

// sorted[rank(in[i])] = in[i], rank = number of smaller keys, per segment.  Keys are distinct
// candidate indices and a query has few valid ones next to its candidate space, so the quadratic
// count is the cheap way to a deterministic ascending order after an unordered atomic append.
__global__ __launch_bounds__(256) void k_rank_sort(const unsigned long long* __restrict__ valid,
                                                   const unsigned long long* __restrict__ valid2,
                                                   unsigned long long* __restrict__ sorted,
                                                   const DevPostSeg* __restrict__ segs, int n_segs) {
    __shared__ unsigned long long tile[256];
    const DevPostSeg seg = find_post_seg(segs, n_segs, blockIdx.x);
    const unsigned long long* in = (seg.in_off >> 63) ? valid2 + (seg.in_off & ~(1ull << 63)) : valid + seg.in_off;
    const uint32_t n = seg.count;
    const uint32_t i = (blockIdx.x - seg.first_block) * 256u + threadIdx.x;
    const unsigned long long key = i < n ? in[i] : 0ull;
    uint32_t rank = 0;
    for (uint32_t t0 = 0; t0 < n; t0 += 256u) {
        const uint32_t j = t0 + threadIdx.x;
        tile[threadIdx.x] = j < n ? in[j] : ~0ull;
        __syncthreads();
        const uint32_t lim = n - t0 < 256u ? n - t0 : 256u;
        for (uint32_t u = 0; u < lim; ++u) rank += tile[u] < key;
        __syncthreads();
    }
    if (i < n) sorted[seg.out_off + rank] = key;
}

// A barrier for what the block keeps in LDS.  __syncthreads() also waits for every global load in flight (loads and
// stores share a counter), which would end the loads ahead of a walk at each of its barriers.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- selection of the K smallest (cost, index, position) triples --------------------------------------------
// One block walks its share of the list a tile at a time (NT threads x kSelUnroll costs each, the next tile in flight)
// and keeps in a buffer in LDS what does not lie above a bound: a cost with at least K entries at or below it.  A first
// bound costs no sort: every lane keeps the smallest cost it has met, a wavefront sorts its 64 of them in registers, and
// the largest over the wavefronts of the ceil(K / wavefronts)-th smallest has K entries at or below it whatever the data.
// When the buffer cannot take a tile's entries, a histogram over both (equal steps of the costs' bit patterns between the
// smallest and the largest) gives the next bound, which some K entries pass; costs that a histogram does not tell apart
// are sorted instead.  Only entries that are sorted or handed on have their index read: a list entry costs 8 bytes.
constexpr int kSelUnroll = 8;

// costs in ascending order as unsigned integers (-0 and +0 compare equal), and back
__device__ inline unsigned long long cost_key(double c) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(c + 0.0);
    return b ^ ((unsigned long long)((long long)b >> 63) | 0x8000000000000000ull);
}
__device__ inline double key_cost(unsigned long long k) {
    return __longlong_as_double((long long)((k >> 63) ? k ^ 0x8000000000000000ull : ~k));
}

// The buffer: an entry is its cost as a key and its place in what is read; idx is filled for a sort.
template <int NT, int B>
struct SelShared {
    unsigned long long key[B], idx[B], pos[B];
    uint32_t bound[NT / kWave];
    unsigned long long lo[NT / kWave], hi[NT / kWave];
    uint32_t rank[B];                      // ranks, places or the bins of a histogram
    uint32_t sum[NT / kWave];
    uint32_t total[3];
    uint32_t flag, edge;
};

// What a block goes by: entries above (cost, index) = (Tc, Ti) are out.
struct SelState {
    uint32_t cnt;
    double Tc;
    unsigned long long Ti;
};

// What a selection reads: costs `stride` apart with a candidate index each; their positions are where they stand, or in
// `pos`.  chunk > 1: of every chunk x 64 entries only the first 64 (whole lines: a sample costs its share of the bytes).
struct SelSource {
    const double* cost;
    const unsigned long long *idx, *pos;
    long long stride, chunk;
    __device__ unsigned long long position(unsigned long long e) const { return pos ? pos[e] : e; }
};

// The value of lane (own lane xor J): a move within a row of 16 lanes where J allows it (the exchange networks below are
// chains of these, and a trip through LDS takes several times as long), else through LDS.
template <int J>
__device__ inline uint32_t lane_xor(uint32_t v) {
    const int x = (int)v;
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);            // quad_perm [1,0,3,2]
    if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true);            // quad_perm [2,3,0,1]
    if constexpr (J == 4)                                                                               // (xor 7, then xor 3)
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true);           // row_ror:8
    return (uint32_t)__shfl_xor(x, J, kWave);
}
template <int J>
__device__ inline unsigned long long lane_xor(unsigned long long v) {
    return (unsigned long long)lane_xor<J>((uint32_t)v) | (unsigned long long)lane_xor<J>((uint32_t)(v >> 32)) << 32;
}

// Over a row of 16 lanes: every lane gets the largest value / the sum.
__device__ inline uint32_t row_max(uint32_t v) {
    uint32_t o;
    o = lane_xor<1>(v); v = o > v ? o : v; o = lane_xor<2>(v); v = o > v ? o : v;
    o = lane_xor<4>(v); v = o > v ? o : v; o = lane_xor<8>(v); return o > v ? o : v;
}
__device__ inline uint32_t row_sum(uint32_t v) {
    v += lane_xor<1>(v); v += lane_xor<2>(v); v += lane_xor<4>(v);
    return v + lane_xor<8>(v);
}

// Bitonic sort of a wavefront's 64 values.
template <int K, int J>
__device__ inline void wave_merge(uint32_t& v, uint32_t lane) {
    const uint32_t o = lane_xor<J>(v);
    v = ((lane & (uint32_t)J) == 0u) == ((lane & (uint32_t)K) == 0u) ? (o < v ? o : v) : (o > v ? o : v);
    if constexpr (J > 1) wave_merge<K, J / 2>(v, lane);
}
__device__ inline void row_sort(uint32_t& v, uint32_t lane) {     // (of every 16; the first 16 ascending)
    wave_merge<2, 1>(v, lane); wave_merge<4, 2>(v, lane); wave_merge<8, 4>(v, lane); wave_merge<16, 8>(v, lane);
}
__device__ inline void wave_sort(uint32_t& v, uint32_t lane) {
    row_sort(v, lane);
    wave_merge<32, 16>(v, lane); wave_merge<64, 32>(v, lane);
}

// Bitonic sort of the buffer (E entries per thread, entry r * NT + thread), keys and buffer places in registers: an
// exchange over fewer than 64 places is one between lanes, over fewer than NT goes through LDS, and over NT stays in the
// thread.  Equal keys are told apart by what the places hold.
template <int NT, int B, int E>
struct SelBitonic {
    SelShared<NT, B>& S;
    const SelSource& src;
    uint32_t cnt, tid;
    unsigned long long key[E];
    uint32_t at[E];
    __device__ bool less(unsigned long long ka, uint32_t pa, unsigned long long kb, uint32_t pb) const {
        if (__builtin_expect(ka != kb, 1)) return ka < kb;
        if (pa >= cnt || pb >= cnt) return pa < pb;
        const unsigned long long ia = S.idx[pa], ib = S.idx[pb];
        return ia != ib ? ia < ib : src.position(S.pos[pa]) < src.position(S.pos[pb]);
    }
    __device__ void take(int r, unsigned long long ko, uint32_t po, uint32_t k, uint32_t j) {
        const uint32_t a = (uint32_t)r * NT + tid;
        const bool low = ((a & j) == 0u) == ((a & k) == 0u);
        if (less(ko, po, key[r], at[r]) == low) { key[r] = ko; at[r] = po; }
    }
    template <int J>
    __device__ void lanes(uint32_t k) {
        if (k > (uint32_t)J)
#pragma unroll
            for (int r = 0; r < E; ++r) take(r, lane_xor<J>(key[r]), lane_xor<J>(at[r]), k, (uint32_t)J);
    }
    __device__ void run() {
#pragma unroll
        for (int r = 0; r < E; ++r) {
            at[r] = (uint32_t)r * NT + tid;
            key[r] = at[r] < cnt ? S.key[at[r]] : ~0ull;
        }
        lds_barrier();                                 // (S.key and S.rank are the exchange area from here on)
#pragma unroll 1
        for (uint32_t k = 2; k <= (uint32_t)(E * NT); k *= 2) {
#pragma unroll 1
            for (uint32_t j = k / 2; j >= 64u; j /= 2) {
                if (E == 2 && j == (uint32_t)NT) {       // (the last merge: ascending)
                    if (less(key[E - 1], at[E - 1], key[0], at[0])) {
                        const unsigned long long kt = key[0]; key[0] = key[E - 1]; key[E - 1] = kt;
                        const uint32_t pt = at[0]; at[0] = at[E - 1]; at[E - 1] = pt;
                    }
                    continue;
                }
#pragma unroll
                for (int r = 0; r < E; ++r) { S.key[(uint32_t)r * NT + tid] = key[r]; S.rank[(uint32_t)r * NT + tid] = at[r]; }
                lds_barrier();
                unsigned long long ko[E];
                uint32_t po[E];
#pragma unroll
                for (int r = 0; r < E; ++r) { ko[r] = S.key[(uint32_t)r * NT + (tid ^ j)]; po[r] = S.rank[(uint32_t)r * NT + (tid ^ j)]; }
                lds_barrier();
#pragma unroll
                for (int r = 0; r < E; ++r) take(r, ko[r], po[r], k, j);
            }
            lanes<32>(k); lanes<16>(k); lanes<8>(k); lanes<4>(k); lanes<2>(k); lanes<1>(k);
        }
        unsigned long long p[E];
#pragma unroll
        for (int r = 0; r < E; ++r) p[r] = at[r] < cnt ? S.pos[at[r]] : 0ull;
        lds_barrier();
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint32_t a = (uint32_t)r * NT + tid;
            if (a < cnt) { S.key[a] = key[r]; S.pos[a] = p[r]; }
        }
    }
};

// The buffer in ascending order, cut to K.  Ties: one cost alone may be all there is (where lists are sorted a block each that
// test costs the others 15 %, 2 549 to 83 920 programs, K = 1024: 31 -> 36 and 101 -> 118 us, in registers that spill).
template <bool Ties, int NT, int B>
__device__ inline void sel_sort(SelShared<NT, B>& S, SelState& st, const SelSource& src, uint32_t K) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    lds_barrier();
    {   // what came in before the bound was as low as it is now goes first
        constexpr int kOwn = B / NT;
        unsigned long long k[kOwn], p[kOwn];
        bool in[kOwn];
        const unsigned long long top = cost_key(st.Tc);
#pragma unroll
        for (int r = 0; r < kOwn; ++r) {
            const uint32_t j = (uint32_t)r * NT + tid;
            k[r] = j < st.cnt ? S.key[j] : ~0ull; p[r] = j < st.cnt ? S.pos[j] : 0ull;
            in[r] = j < st.cnt && k[r] <= top;
        }
        if (tid == 0) S.flag = 0u;
        lds_barrier();
#pragma unroll
        for (int r = 0; r < kOwn; ++r) {
            const unsigned long long m = __ballot(in[r]);
            uint32_t at = 0;
            if (lane == 0 && m) at = atomicAdd(&S.flag, (uint32_t)__popcll(m));
            at = (uint32_t)__shfl((int)at, 0, kWave) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (in[r]) { S.key[at] = k[r]; S.pos[at] = p[r]; }
        }
        lds_barrier();
    }
    const uint32_t cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.flag);
    if (cnt <= (uint32_t)NT / 2u) {
        // few entries: everyone's rank is counted, the threads that share an entry take turns through the others (upper
        // halves first; candidate indices are read only if some of those are equal)
        uint32_t P = 32;
        while (P < cnt) P *= 2;
        const uint32_t item = tid & (P - 1u), part = tid / P, parts = (uint32_t)NT / P;
        if (tid < cnt) S.rank[tid] = 0u;
        const unsigned long long k = item < cnt ? S.key[item] : 0ull, p = item < cnt ? S.pos[item] : 0ull;
        const uint32_t kh = (uint32_t)(k >> 32);
        const uint32_t* upper = reinterpret_cast<const uint32_t*>(S.key) + 1;
        uint32_t below = 0, equal = 0;
        if (item < cnt)
#pragma unroll 8
            for (uint32_t j = part; j < cnt; j += parts) {
                const uint32_t o = upper[2u * j];
                below += o < kh ? 1u : 0u;
                equal += o == kh ? 1u : 0u;
            }
        const bool ties = item < cnt && equal > (item % parts == part ? 1u : 0u);
        if (__syncthreads_or(ties ? 1 : 0)) {
            for (uint32_t j = tid; j < cnt; j += NT) S.idx[j] = src.idx[S.pos[j]];
            lds_barrier();
            if (ties) {
                const unsigned long long i = S.idx[item];
                for (uint32_t j = part; j < cnt; j += parts) {
                    const unsigned long long o = S.key[j];
                    if ((uint32_t)(o >> 32) != kh || j == item) continue;
                    const unsigned long long ij = S.idx[j];
                    below += o != k ? (o < k ? 1u : 0u) : ij != i ? (ij < i ? 1u : 0u) : src.position(S.pos[j]) < src.position(p) ? 1u : 0u;
                }
            }
        }
        if (below) atomicAdd(&S.rank[item], below);
        lds_barrier();
        if (part == 0 && item < cnt) {
            const uint32_t r = S.rank[item];
            S.key[r] = k; S.pos[r] = p;
        }
    } else {
        // (nothing but one cost: the indices are sorted as if they were the keys, instead of being looked up at every exchange;
        //  10 000 equal costs, K = 16: 81 -> 64 us in a p2_topk_device call)
        const unsigned long long one = S.key[0];
        bool differ = false;
        for (uint32_t j = tid; j < cnt; j += NT) { S.idx[j] = src.idx[S.pos[j]]; differ |= Ties && S.key[j] != one; }
        const bool same = Ties && __syncthreads_or(differ ? 1 : 0) == 0;
        if (same) for (uint32_t j = tid; j < cnt; j += NT) S.key[j] = S.idx[j];
        if (cnt <= (uint32_t)NT) SelBitonic<NT, B, 1>{S, src, cnt, tid, {}, {}}.run();
        else SelBitonic<NT, B, B / NT>{S, src, cnt, tid, {}, {}}.run();
        if (same) {
            lds_barrier();
            for (uint32_t j = tid; j < cnt; j += NT) S.key[j] = one;
        }
    }
    lds_barrier();
    st.cnt = cnt < K ? cnt : K;
    if (st.cnt == K && key_cost(S.key[K - 1u]) <= st.Tc) { st.Tc = key_cost(S.key[K - 1u]); st.Ti = src.idx[S.pos[K - 1u]]; }
}

// A bound that some K of the buffer's entries and the tile's (kSelUnroll keys per thread, ~0 where there is none) pass,
// and what passes it into the buffer.  False, with nothing changed: too many would stay.
template <int NT, int B, class Key, class Place>
__device__ inline bool sel_cut(SelShared<NT, B>& S, SelState& st, uint32_t K, Key key, Place place) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    constexpr int kOwn = B / NT;
    unsigned long long lo = ~0ull, hi = 0ull;
    lds_barrier();
    unsigned long long own[kOwn];
#pragma unroll
    for (int r = 0; r < kOwn; ++r) own[r] = (uint32_t)r * NT + tid < st.cnt ? S.key[(uint32_t)r * NT + tid] : ~0ull;
    auto see = [&](unsigned long long v) { lo = v < lo ? v : lo; hi = v != ~0ull && v > hi ? v : hi; };
#pragma unroll
    for (int r = 0; r < kOwn; ++r) see(own[r]);
#pragma unroll
    for (int u = 0; u < kSelUnroll; ++u) see(key(u));
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long a = __shfl_xor(lo, o, kWave), b = __shfl_xor(hi, o, kWave);
        lo = a < lo ? a : lo; hi = b > hi ? b : hi;
    }
    if (lane == 0) { S.lo[wave] = lo; S.hi[wave] = hi; }
    for (uint32_t j = tid; j < (uint32_t)B; j += NT) S.rank[j] = 0u;
    lds_barrier();
    for (int w = 0; w < NT / kWave; ++w) { lo = S.lo[w] < lo ? S.lo[w] : lo; hi = S.hi[w] > hi ? S.hi[w] : hi; }
    const int bits = hi > lo ? 64 - __clzll((long long)(hi - lo)) : 0;
    const int shift = bits > __builtin_ctz(B) ? bits - __builtin_ctz(B) : 0;
    auto count = [&](unsigned long long v) { if (v != ~0ull) atomicAdd(&S.rank[(uint32_t)((v - lo) >> shift)], 1u); };
#pragma unroll
    for (int r = 0; r < kOwn; ++r) count(own[r]);
#pragma unroll
    for (int u = 0; u < kSelUnroll; ++u) count(key(u));
    lds_barrier();
    // the first bin up to which there are K entries: B / NT bins per thread
    uint32_t mine = 0;
#pragma unroll
    for (int r = 0; r < kOwn; ++r) mine += S.rank[tid * kOwn + (uint32_t)r];
    uint32_t upto = mine;
    for (int o = 1; o < 64; o <<= 1) { const uint32_t v = (uint32_t)__shfl_up((int)upto, o, kWave); if (lane >= (uint32_t)o) upto += v; }
    if (lane == 63u) S.sum[wave] = upto;
    lds_barrier();
    { const uint32_t w = lane & 15u; upto += row_sum(w < wave ? S.sum[w] : 0u); }
    uint32_t before = upto - mine;
    if (before < K && upto >= K)
#pragma unroll
        for (int r = 0; r < kOwn; ++r) {
            const uint32_t h = S.rank[tid * kOwn + (uint32_t)r];
            if (before < K && before + h >= K) { S.edge = tid * kOwn + (uint32_t)r; S.flag = before + h; }
            before += h;
        }
    lds_barrier();
    const uint32_t stay = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.flag), edge = S.edge;
    lds_barrier();
    if (stay > (uint32_t)B) return false;
    unsigned long long at[kOwn];
#pragma unroll
    for (int r = 0; r < kOwn; ++r) at[r] = (uint32_t)r * NT + tid < st.cnt ? S.pos[(uint32_t)r * NT + tid] : 0ull;
    if (tid == 0) S.flag = 0u;
    lds_barrier();
    auto keep = [&](unsigned long long v, unsigned long long e) {
        const bool ok = v != ~0ull && (uint32_t)((v - lo) >> shift) <= edge;
        const unsigned long long m = __ballot(ok);
        if (m == 0ull) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&S.flag, (uint32_t)__popcll(m));
        base = (uint32_t)__shfl((int)base, 0, kWave);
        if (ok) {
            const uint32_t o = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            S.key[o] = v; S.pos[o] = e;
        }
    };
#pragma unroll
    for (int r = 0; r < kOwn; ++r) keep(own[r], at[r]);
#pragma unroll
    for (int u = 0; u < kSelUnroll; ++u) keep(key(u), place(u));
    const unsigned long long last = lo + ((((unsigned long long)edge + 1ull) << shift) - 1ull);
    st.cnt = stay;
    st.Tc = fmin(st.Tc, key_cost(last < lo || last > hi ? hi : last));
    st.Ti = ~0ull;
    return true;
}

// Tiles first, first + step, ... of the source's n entries go through the buffer; true: a NaN was among this lane's.
template <bool Ties, int NT, int B>
__device__ inline bool sel_consume(SelShared<NT, B>& S, SelState& st, const SelSource& src, long long n, long long first, long long step,
                                   uint32_t K, bool bounded) {
    constexpr long long kTile = (long long)NT * kSelUnroll;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    if (tid < 3u) S.total[tid] = 0u;
    lds_barrier();
    const long long lane_off = (long long)lane * src.stride, row_off = src.chunk * 64ll * src.stride;
    double next[kSelUnroll];
    uint32_t mine = ~0u;                                 // upper half of the smallest key so far
    bool nan = false;
    // (entries 64 by 64: row `at / 64` of a wavefront is a base that all its lanes share)
    auto rest_of = [&](long long t, int u) { return n - (t * kTile + (long long)u * NT + (long long)wave * 64ll); };
    auto load = [&](long long t) {
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {           // (loads without a condition: all of them in flight together)
            const long long rest = rest_of(t, u);
            const long long row = rest > 0 ? ((n - rest) >> 6) : 0ll;
            const double* p = src.cost + row * row_off;
            next[u] = p[(long long)lane < rest ? lane_off : 0ll];
        }
    };
    const long long tiles = (n + kTile - 1) / kTile;
    uint32_t round = 0;
    if (first < tiles) load(first);
#pragma unroll 1
    for (long long t = first; t < tiles; t += step, ++round) {
        double c[kSelUnroll];
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {
            c[u] = (long long)lane < rest_of(t, u) ? next[u] : __longlong_as_double(0x7ff8000000000000ll);
            nan |= c[u] != c[u] && (long long)lane < rest_of(t, u);
            const uint32_t h = (uint32_t)__double2hiint(c[u]), k = c[u] == c[u] ? h ^ ((uint32_t)((int)h >> 31) | 0x80000000u) : ~0u;
            mine = k < mine ? k : mine;
        }
        if (t + step < tiles) load(t + step);
        if (!bounded && (round & (round + 1u)) == 0u) {  // after 1, 2, 4, ... tiles
            const long long seen = round > 0u ? kTile : n - t * kTile;
            const uint32_t waves = seen >= NT ? NT / kWave : (uint32_t)((seen + kWave - 1) / kWave);
            const uint32_t r = (K + waves - 1u) / waves;
            if (r <= 64u) {
                uint32_t v = mine;
                wave_sort(v, lane);
                if (lane == r - 1u) S.bound[wave] = v;
                lds_barrier();
                const uint32_t w = lane & (uint32_t)(NT / kWave - 1);
                const uint32_t T = row_max(w < waves ? S.bound[w] : 0u);
                const double Tc = key_cost((unsigned long long)T << 32 | 0xffffffffull);      // (a NaN where T says nothing)
                if (Tc < st.Tc) { st.Tc = Tc; st.Ti = ~0ull; }
            }
        }
        auto entry = [&](int u) { return ((n - rest_of(t, u)) >> 6) * (src.chunk * 64ll) + (long long)lane; };
        auto passes = [&](int u, double v) {
            bool ok = v <= st.Tc;                        // (false for a NaN and past the end)
            if (st.Ti != ~0ull && __ballot(ok && v == st.Tc) != 0ull) ok = ok && (v < st.Tc || src.idx[entry(u)] <= st.Ti);
            return ok;
        };
        uint32_t in = 0, n_wave = 0;
#pragma unroll
        for (int u = 0; u < kSelUnroll; ++u) {
            const bool ok = passes(u, c[u]);
            in |= ok ? 1u << u : 0u;
            n_wave += (uint32_t)__popcll(__ballot(ok));
        }
        uint32_t base = 0;
        if (n_wave) {
            if (lane == 0) base = atomicAdd(&S.total[round % 3u], n_wave);
            base = (uint32_t)__shfl((int)base, 0, kWave);
        }
        lds_barrier();
        const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.total[round % 3u]);
        if (tid == 0) S.total[(round + 2u) % 3u] = 0u;   // (last read before the barrier, used again in two rounds)
        if (__builtin_expect(st.cnt + total <= (uint32_t)B, 1)) {
            if (n_wave) {
                uint32_t at = st.cnt + base;
#pragma unroll
                for (int u = 0; u < kSelUnroll; ++u) {
                    const unsigned long long m = __ballot((in >> u) & 1u);
                    if ((in >> u) & 1u) {
                        const uint32_t o = at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                        S.key[o] = cost_key(c[u]); S.pos[o] = (unsigned long long)entry(u);
                    }
                    at += (uint32_t)__popcll(m);
                }
            }
            st.cnt += total;
        } else if (sel_cut(S, st, K, [&](int u) { return (in >> u) & 1u ? cost_key(c[u]) : ~0ull; },
                           [&](int u) { return (unsigned long long)entry(u); })) {
        } else {
            // too many alike: NT at a time, the buffer sorted and cut to K where even those do not fit
#pragma unroll 1
            for (int u = 0; u < kSelUnroll; ++u) {
                unsigned long long m;
                uint32_t at, more;
                const double v = (long long)lane < rest_of(t, u) ? src.cost[entry(u) * src.stride] : __longlong_as_double(0x7ff8000000000000ll);
                bool ok;
#pragma unroll 1
                for (;;) {
                    lds_barrier();
                    if (tid == 0) S.flag = 0u;
                    lds_barrier();
                    ok = passes(u, v);
                    m = __ballot(ok);
                    at = 0;
                    if (lane == 0 && m) at = atomicAdd(&S.flag, (uint32_t)__popcll(m));
                    at = (uint32_t)__shfl((int)at, 0, kWave);
                    lds_barrier();
                    more = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.flag);
                    if (st.cnt + more <= (uint32_t)B) break;
                    sel_sort<Ties>(S, st, src, K);                // (leaves room for NT: this happens once)
                }
                if (ok) {
                    const uint32_t o = st.cnt + at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    S.key[o] = cost_key(v); S.pos[o] = (unsigned long long)entry(u);
                }
                st.cnt += more;
            }
        }
    }
    return nan;
}

// Words that the blocks of a launch share.  All zero between launches (the last block leaves them so).
struct SelControl {
    uint32_t done, cursor, nan, pad;
    double bound;                      // a cost with K entries at or below it, left by a launch over a sample
};

constexpr int kSelThreads = 1024, kSelBuffer = 2048;
constexpr long long kSelTile = (long long)kSelThreads * kSelUnroll;
// Blocks of a launch: a tile each, at most one per compute unit (a block keeps 64 KiB of loads in flight, and the registers
// of 1024 threads with 8 costs at hand and 8 on their way leave no room for a second one).  One block where two tiles are
// all there is: no lists, no hand-over (10 007 entries: 25 us; the hand-over alone takes 5).
inline unsigned sel_blocks(long long n) {
    const long long tiles = (n + kSelTile - 1) / kSelTile;
    return tiles <= 2 ? 1u : (unsigned)(tiles < 256 ? tiles : 256);
}
// Entries that one block may leave for the last one: not cut to K as long as they are few (a sort saved).
inline __host__ __device__ uint32_t sel_share(int K) {
    const uint32_t c = 3u * (uint32_t)K + 128u;
    return c < (uint32_t)kSelBuffer ? c : (uint32_t)kSelBuffer;
}
// Long columns are looked at twice: first one entry in 64 (64 in a row, so that whole lines are used), which leaves a
// bound that some 64 K entries pass; without it every one of the blocks keeps K of its own, and the last block walks
// them all.  A second launch and its wait for the first cost some 40 us: 1.3 M entries, K = 64 (159 lists) takes 41 us of
// kernel time without, and K * blocks of 32 768 is where the last block's walk takes as long as the sample.
constexpr long long kSelSample = 64;
inline bool sel_sampled(long long n, int K) { return n >= (1ll << 22) || (n >= (1ll << 18) && (long long)sel_blocks(n) * K >= 32768); }

// Measured (a whole p2_topk_device call, host wait included; before: one wavefront per block inserting into a sorted list
// of K, then one wavefront walking all the lists): 10 007 entries, K = 10: 89 -> 25 us, of which the kernel is 15, a chain
// of some ten memory and barrier latencies (few entries to keep: below); 1.3 M of stride 3, K = 64: 1190 -> 56 us, half of it the last block's walk;
// 50 M, K = 100: 3170 -> 160 us, of which 100 read 400 MB at 4 TB/s (a large copy reaches 4.9) and 40 find the bound.
// K smallest of a column by all blocks together: every block leaves what it kept, the last one to finish goes through
// that and writes the positions (or, over a sample, the bound).  The lists hold `cap` entries, all that the blocks of one
// call can leave; calls that overlap on one scratch against the rule (the fixed one below) add to the same cursor, so the
// cursor is held against `cap` before a store and after the hand-over, and what comes out is a position of this column
// or -1 also where the lists were another call's: a wrong answer then, never an access out of range.
__global__ __launch_bounds__(kSelThreads) void k_topk_column(SelSource src, long long n, int K, int sample, int bounded,
                                                             SelControl* __restrict__ ctl, double* lc, unsigned long long* li,
                                                             unsigned long long* lp, uint32_t cap, long long* __restrict__ out_pos,
                                                             long long n_out, uint32_t* __restrict__ nan_out) {
    __shared__ SelShared<kSelThreads, kSelBuffer> S;
    const uint32_t tid = threadIdx.x;
    const unsigned long long n_column = (unsigned long long)n;
    SelState st{0u, __longlong_as_double(0x7ff0000000000000ll), ~0ull};
    if (bounded) st.Tc = ctl->bound;
    long long first = blockIdx.x, step = gridDim.x;
    bool last = gridDim.x == 1u, nan = false;
    for (;;) {
        nan |= sel_consume<true>(S, st, src, n, first, step, (uint32_t)K, bounded != 0);
        if (last || st.cnt > sel_share(K)) sel_sort<true>(S, st, src, (uint32_t)K);
        if (last) break;
        if (nan) __hip_atomic_fetch_or(&ctl->nan, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (tid == 0) S.flag = st.cnt ? __hip_atomic_fetch_add(&ctl->cursor, st.cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        __syncthreads();
        const uint32_t base = S.flag;
        const uint32_t room = base < cap ? cap - base : 0u;
        for (uint32_t j = tid; j < (st.cnt < room ? st.cnt : room); j += kSelThreads) {
            const unsigned long long e = S.pos[j];
            lc[base + j] = key_cost(S.key[j]); li[base + j] = src.idx[e]; lp[base + j] = e;
        }
        __syncthreads();                                 // (the block's stores have been made; thread 0 hands them over)
        if (tid == 0) {
            __threadfence();
            S.flag = __hip_atomic_fetch_add(&ctl->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence();
        }
        __syncthreads();
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)S.flag) != gridDim.x - 1u) return;
        // the last block goes through what all of them have left, its own entries among it; its bound still holds
        const uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(&ctl->cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        n = (long long)(left < cap ? left : cap);
        st.cnt = 0u;
        src = SelSource{lc, li, lp, 1, 1};
        first = 0; step = 1; bounded = 0;
        last = true;
    }
    if (!sample)
        for (long long j = tid; j < n_out; j += kSelThreads) {
            const unsigned long long p = j < (long long)st.cnt ? src.position(S.pos[j]) : ~0ull;
            out_pos[j] = p < n_column ? (long long)p : -1ll;
        }
    const bool any = __syncthreads_or(nan ? 1 : 0) != 0;
    if (tid == 0) {
        ctl->bound = sample && st.cnt == (uint32_t)K ? key_cost(S.key[K - 1]) : __longlong_as_double(0x7ff0000000000000ll);
        const uint32_t other = __hip_atomic_load(&ctl->nan, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (nan_out && (other || any)) *nan_out = 1u;
        ctl->nan = 0u; ctl->done = 0u; ctl->cursor = 0u;
    }
}

// A job whose number of entries the device knows; the rows that such a job has picked, written out by thread j.
__device__ __forceinline__ void open_job(DevTopkJob& J) {
    if (J.n_from && (long long)*J.n_from < J.n) J.n = (long long)*J.n_from;
}
// (false: there is none)
__device__ __forceinline__ bool write_row(const DevTopkJob& J, uint32_t j, long long pos) {
    if (!J.progs) return true;
    if (pos < 0) return false;
    J.out_progs[j] = J.progs[pos];
    for (int c = 0; c < J.n_cost; ++c) J.out_costs[(size_t)j * (size_t)J.n_cost + c] = J.costs[(size_t)pos * (size_t)J.n_cost + c];
    return true;
}
// What a job has to report, put together in LDS where the job has a word of its own: the host reads it without a copy behind the
// selections (queries of [3 4 6], four instructions, 121.5 us a call with the copy, 119.2 so; searches on 4 x 16 110.3 and 107.8).
__device__ __forceinline__ void note_trouble(const DevTopkJob& J, uint32_t& trouble, uint32_t bits) {
    if (J.own_flag) atomicOr(&trouble, bits);
    else if (bits & 1u) atomicOr(J.nan_flag, 1u);
}
__device__ __forceinline__ void report_trouble(const DevTopkJob& J, const uint32_t& trouble) {
    if (!J.own_flag) return;
    __syncthreads();
    if (threadIdx.x == 0) *J.own_flag = trouble;
}
// Many selections in one launch: block b does job b from start to end (k_few_jobs where few() says so).  A launch of lists of at most 512 entries (a tile,
// K <= 64) takes a wavefront each: nothing there is worth a barrier between wavefronts.  A tile of lists of at most 2048
// entries (K <= 256) is 256 threads wide, so that several jobs share a compute unit; longer lists take 1024.
template <int NT, int B>
__global__ __launch_bounds__(NT) void k_topk_jobs(const DevTopkJob* __restrict__ jobs) {
    __shared__ SelShared<NT, B> S;
    __shared__ uint32_t trouble;
    DevTopkJob J = jobs[blockIdx.x];
    open_job(J);
    if (threadIdx.x == 0) trouble = 0u;
    __syncthreads();
    if (J.n <= 0) { report_trouble(J, trouble); return; }
    SelState st{0u, __longlong_as_double(0x7ff0000000000000ll), ~0ull};
    const SelSource src{J.cost, J.index, nullptr, J.stride, 1};
    if (sel_consume<false>(S, st, src, J.n, 0, 1, (uint32_t)J.k, false)) note_trouble(J, trouble, 1u);
    sel_sort<false>(S, st, src, (uint32_t)J.k);
    const long long n_out = J.k < J.n ? J.k : J.n;
    for (long long j = threadIdx.x; j < n_out; j += NT) {
        const long long pos = j < (long long)st.cnt ? (long long)S.pos[j] : -1ll;
        J.out_pos[j] = pos;
        if (!write_row(J, (uint32_t)j, pos)) note_trouble(J, trouble, 2u);
    }
    report_trouble(J, trouble);
}

// ---- the same selection for a few entries -------------------------------------------------------------------
// A shortlist of at most kFewMax entries fits in a wavefront's lanes, and then nothing depends on how the costs are spread
// or ordered: a wavefront goes through tiles of 512 entries (the next one in flight) and, where a tile has an entry that
// does not lie above the K-th so far, picks the K smallest of the tile and its list in K rounds of a minimum over the
// lanes; indices are read for such tiles only.  The block's wavefronts share the lowest K-th through LDS and merge their
// lists at the end.
// Where the line to the buffers above lies (whole p2_topk_device calls, us, buffers / this form): they take longer where a
// column is sorted or full of ties, 10 000 equal costs: K = 1 80 / 22, 4 81 / 30, 10 81 / 30, 1 M: 91 / 33, 103 / 43,
// 104 / 85 (a sorted list with insertion, which ties in ascending order suit, took 25, 29, 36 and 34, 61, 120).  On random
// costs both take about the same up to 10 kept entries, 3 000: 20 / 17, 20 / 19, 21 / 23, 10 000: 24 / 20, 24 / 22, 24 / 23,
// while 16 took 24 / 37, and from 5 on this form is the slower one for long columns, 1 M, 10 kept: 34 / 39.  So: up to 4,
// and up to 10 of 2^18.
constexpr int kFewMax = 16, kFewUnroll = 8, kFewWaves = 16;
constexpr long long kFewTile = (long long)kWave * kFewUnroll;

struct FewList { unsigned long long key, idx, pos; };    // lane i: the i-th smallest (key ~0: none)
struct FewShared {
    unsigned long long key[kFewWaves * kFewMax], idx[kFewWaves * kFewMax], pos[kFewWaves * kFewMax];
    unsigned long long bound;                            // a key that K of the block's entries do not exceed
    uint32_t least[kFewWaves];
    uint32_t flag;
};

__device__ inline unsigned long long of_lane(unsigned long long v, int lane) {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane) |
           (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32;
}

__device__ inline bool before(const FewList& a, const FewList& b) {
    return a.key != b.key ? a.key < b.key : a.idx != b.idx ? a.idx < b.idx : a.pos < b.pos;
}
// Bitonic sort of a wavefront's entries.
template <int K, int J>
__device__ inline void few_merge_lanes(FewList& v, uint32_t lane) {
    const FewList o{lane_xor<J>(v.key), lane_xor<J>(v.idx), lane_xor<J>(v.pos)};
    if (before(o, v) == (((lane & (uint32_t)J) == 0u) == ((lane & (uint32_t)K) == 0u))) v = o;
    if constexpr (J > 1) few_merge_lanes<K, J / 2>(v, lane);
}
__device__ inline uint32_t lane_below(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xf, 0xf, false); }      // row_shr:1
__device__ inline unsigned long long lane_below(unsigned long long v) {
    return (unsigned long long)lane_below((uint32_t)v) | (unsigned long long)lane_below((uint32_t)(v >> 32)) << 32;
}

template <int J>
__device__ inline void few_least(FewList& v) {
    const FewList o{lane_xor<J>(v.key), lane_xor<J>(v.idx), lane_xor<J>(v.pos)};
    if (before(o, v)) v = o;
    if constexpr (J > 1) few_least<J / 2>(v);
}

// The K smallest of the list L and E entries per lane (bit i of `left`: there is one).  Where some lanes have one they go
// in one by one; otherwise the lanes' smallest, the list's among them, are sorted, and what a lane has besides goes in
// where it lies before the K-th.
template <int E>
__device__ inline FewList few_pick(const FewList& L, const unsigned long long (&key)[E], const unsigned long long (&idx)[E],
                                   const unsigned long long (&pos)[E], uint32_t left, int K) {
    const uint32_t lane = threadIdx.x & 63u;
    const FewList none{~0ull, ~0ull, ~0ull};
    uint32_t mine = 0u;
    auto smallest = [&]() {
        FewList b = none;
        mine = 0u;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const FewList e{key[i], idx[i], pos[i]};
            if (((left >> i) & 1u) && before(e, b)) { b = e; mine = 1u << i; }
        }
        return b;
    };
    FewList out = L;
    if (K == 1 || __popcll(__ballot(left != 0u)) > 6) {
        FewList b = smallest();
        if (before(L, b)) b = L; else { left &= ~mine; }
        const bool held = K > 1 && lane < (uint32_t)K && L.key != ~0ull && b.pos != L.pos;       // (a list entry that its lane's own goes before)
        out = b;
        if (K == 1) {
            few_least<32>(out);
            if (lane != 0u) out = none;
            return out;
        }
        few_merge_lanes<2, 1>(out, lane); few_merge_lanes<4, 2>(out, lane); few_merge_lanes<8, 4>(out, lane);
        few_merge_lanes<16, 8>(out, lane); few_merge_lanes<32, 16>(out, lane); few_merge_lanes<64, 32>(out, lane);
        if (lane >= (uint32_t)K) out = none;
        left |= held ? 1u << E : 0u;
    }
#pragma unroll 1
    for (;;) {
        const FewList last{of_lane(out.key, K - 1), of_lane(out.idx, K - 1), of_lane(out.pos, K - 1)};
        FewList b = smallest();
        if (((left >> E) & 1u) && before(L, b)) { b = L; mine = 1u << E; }
        const unsigned long long m = __ballot(before(b, last));
        if (m == 0ull) return out;
        const int w = __ffsll((long long)m) - 1;
        const FewList it{of_lane(b.key, w), of_lane(b.idx, w), of_lane(b.pos, w)};
        if ((int)lane == w) left &= ~mine;
        const uint32_t at = (uint32_t)__popcll(__ballot(lane < (uint32_t)K && before(out, it)));
        const FewList up{lane_below(out.key), lane_below(out.idx), lane_below(out.pos)};
        if (lane == at) out = it;
        else if (lane > at && lane < (uint32_t)K) out = up;
    }
}

// Tiles first, first + step, ... go into the wavefront's list (all wavefronts of the block together); true: a NaN was
// among this lane's entries.
__device__ inline bool few_scan(FewShared& S, FewList& L, const SelSource& src, long long n, long long first, long long step, int K) {
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = blockDim.x >> 6;
    const long long tiles = (n + kFewTile - 1) / kFewTile;
    double next[kFewUnroll];
    bool nan = false;
    auto entry = [&](long long t, int u) { const long long e = t * kFewTile + (long long)u * 64 + (long long)lane; return e < n ? e : 0ll; };
    auto there = [&](long long t, int u) { return t * kFewTile + (long long)u * 64 + (long long)lane < n; };
    auto load = [&](long long t) {
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) next[u] = src.cost[entry(t, u) * src.stride];
    };
    if (first < tiles) load(first);
    bool begun = waves == 1u;
#pragma unroll 1
    for (long long t = first; t < tiles || !begun; t += step) {
        unsigned long long key[kFewUnroll], idx[kFewUnroll], pos[kFewUnroll];
        unsigned long long least = ~0ull;
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            const double c = next[u];
            const bool ok = there(t, u);
            nan |= ok && c != c;
            key[u] = ok && c == c ? cost_key(c) : ~0ull;
            least = key[u] < least ? key[u] : least;
        }
        if (t + step < tiles) load(t + step);
        if (!begun) {                                    // a first bound for the block, as above: so that few go into the lists
            begun = true;
            const uint32_t r = ((uint32_t)K + waves - 1u) / waves;
            uint32_t v = (uint32_t)(least >> 32);
            wave_sort(v, lane);
            if (lane == r - 1u) S.least[wave] = v;
            __syncthreads();
            uint32_t T = lane < waves ? S.least[lane] : ~0u;
            row_sort(T, lane);
            T = (uint32_t)__builtin_amdgcn_readlane((int)T, (int)(((uint32_t)K + r - 1u) / r) - 1);
            if (threadIdx.x == 0 && T != ~0u) __hip_atomic_fetch_min(&S.bound, (unsigned long long)T << 32 | 0xffffffffull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __syncthreads();
        }
        const unsigned long long kth = of_lane(L.key, K - 1), shared = __hip_atomic_load(&S.bound, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const unsigned long long bound = kth < shared ? kth : shared;
        uint32_t left = 0u;
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) left |= key[u] <= bound && key[u] != ~0ull ? 1u << u : 0u;
        if (__ballot(left != 0u) == 0ull) continue;
#pragma unroll
        for (int u = 0; u < kFewUnroll; ++u) {
            const unsigned long long e = (unsigned long long)entry(t, u);
            idx[u] = src.idx[e]; pos[u] = src.position(e);
        }
        L = few_pick(L, key, idx, pos, left, K);
        const unsigned long long now = of_lane(L.key, K - 1);
        if (lane == 0u && now != ~0ull) __hip_atomic_fetch_min(&S.bound, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return nan;
}

// The lists of the block's wavefronts into the first one's.
__device__ inline void few_merge(FewShared& S, FewList& L, int K) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, n = (blockDim.x >> 6) * (uint32_t)K;
    if (blockDim.x == (uint32_t)kWave) return;
    if (lane < (uint32_t)K) { S.key[wave * K + lane] = L.key; S.idx[wave * K + lane] = L.idx; S.pos[wave * K + lane] = L.pos; }
    __syncthreads();
    if (wave == 0u) {
        constexpr int kE = kFewWaves * kFewMax / kWave;
        unsigned long long key[kE], idx[kE], pos[kE];
#pragma unroll
        for (int i = 0; i < kE; ++i) {
            const uint32_t j = (uint32_t)i * 64u + lane;
            key[i] = j < n ? S.key[j] : ~0ull; idx[i] = j < n ? S.idx[j] : ~0ull; pos[i] = j < n ? S.pos[j] : ~0ull;
        }
        uint32_t left = 0u;
#pragma unroll
        for (int i = 0; i < kE; ++i) left |= key[i] != ~0ull ? 1u << i : 0u;
        L = few_pick(FewList{~0ull, ~0ull, ~0ull}, key, idx, pos, left, K);
    }
    __syncthreads();
}

// One column by all blocks: every block leaves its K in a slot of the lists, the last one to finish merges them.  `fresh`
// (one block): the NaN word is written either way.
__global__ __launch_bounds__(kWave * kFewWaves) void k_few_column(SelSource src, long long n, int K, SelControl* __restrict__ ctl, double* lc,
                                                                  unsigned long long* li, unsigned long long* lp, long long* __restrict__ out_pos,
                                                                  long long n_out, uint32_t* __restrict__ nan_out, int fresh) {
    __shared__ FewShared S;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, waves = blockDim.x >> 6;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const unsigned long long n_column = (unsigned long long)n;
    FewList L{~0ull, ~0ull, ~0ull};
    if (tid == 0) S.bound = ~0ull;
    __syncthreads();
    const bool nan = few_scan(S, L, src, n, (long long)blockIdx.x * waves + wave, (long long)gridDim.x * waves, K);
    few_merge(S, L, K);
    if (gridDim.x > 1u) {
        if (nan) __hip_atomic_fetch_or(&ctl->nan, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid < (uint32_t)K) {
            const size_t o = (size_t)blockIdx.x * (size_t)K + tid;
            lc[o] = L.key != ~0ull ? key_cost(L.key) : __longlong_as_double(0x7ff8000000000000ll); li[o] = L.idx; lp[o] = L.pos;
        }
        __syncthreads();                                 // (the block's stores have been made; thread 0 hands them over)
        if (tid == 0) {
            __threadfence();
            S.flag = __hip_atomic_fetch_add(&ctl->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence();
            S.bound = ~0ull;
        }
        __syncthreads();
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)S.flag) != gridDim.x - 1u) return;
        L = FewList{~0ull, ~0ull, ~0ull};
        (void)few_scan(S, L, SelSource{lc, li, lp, 1, 1}, (long long)gridDim.x * K, wave, waves, K);      // (a slot that is empty holds a NaN)
        few_merge(S, L, K);
    }
    if (wave == 0u && (long long)lane < n_out) out_pos[lane] = L.key != ~0ull && L.pos < n_column ? (long long)L.pos : -1ll;
    const bool any = __syncthreads_or(nan ? 1 : 0) != 0;
    if (tid != 0) return;
    const uint32_t other = gridDim.x > 1u ? __hip_atomic_load(&ctl->nan, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (nan_out && (other || any || fresh)) *nan_out = other || any ? 1u : 0u;
    if (gridDim.x > 1u) { ctl->nan = 0u; ctl->done = 0u; }
}

__global__ __launch_bounds__(kWave * kFewWaves) void k_few_jobs(const DevTopkJob* __restrict__ jobs) {
    __shared__ FewShared S;
    __shared__ uint32_t trouble;
    DevTopkJob J = jobs[blockIdx.x];
    open_job(J);
    if (threadIdx.x == 0) trouble = 0u;
    if (J.n <= 0) { __syncthreads(); report_trouble(J, trouble); return; }
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    FewList L{~0ull, ~0ull, ~0ull};
    if (tid == 0) S.bound = ~0ull;
    __syncthreads();
    if (few_scan(S, L, SelSource{J.cost, J.index, nullptr, J.stride, 1}, J.n, wave, blockDim.x >> 6, J.k)) note_trouble(J, trouble, 1u);
    few_merge(S, L, J.k);
    if (wave == 0u && (long long)lane < (J.k < J.n ? (long long)J.k : J.n)) {
        const long long pos = L.key != ~0ull ? (long long)L.pos : -1ll;
        J.out_pos[lane] = pos;
        if (!write_row(J, lane, pos)) note_trouble(J, trouble, 2u);
    }
    report_trouble(J, trouble);
}
// Wavefronts of a block for so many entries, and blocks (one up to four tiles a wavefront: the hand-over takes as long as
// several; at most one per compute unit).
inline unsigned few_threads(long long n) {
    const long long tiles = (n + kFewTile - 1) / kFewTile;
    return (unsigned)(tiles < kFewWaves ? tiles : (long long)kFewWaves) * (unsigned)kWave;
}
inline unsigned few_blocks(long long n) {
    const long long b = (n + kFewTile * kFewWaves - 1) / (kFewTile * kFewWaves);
    return (unsigned)(b <= 4 ? 1 : b < 256 ? b : 256);
}
// (see above)
inline bool few(long long n, int K) { return K <= 4 || (K <= 10 && n <= (1ll << 18)); }

// Device memory -> pinned host memory, written by the GPU itself in 16-byte words.
__global__ __launch_bounds__(256) void k_copy_out(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

struct CopyOut { uint4* dst; const uint4* src; size_t n16; };
// Up to four copies between device memory and pinned host memory, or fills with zero, in one launch: a launch of its own
// for each would cost a small call several microseconds apiece.
constexpr int kCopyParts = 4;
struct CopyArgs { CopyOut part[kCopyParts]; };
__global__ __launch_bounds__(256) void k_copies(CopyArgs a) {
    size_t before = 0;
#pragma unroll
    for (int p = 0; p < kCopyParts; ++p) {
        // (a part's first word falls to the thread that follows the last one of the part before)
        const size_t step = (size_t)gridDim.x * 256, me = (size_t)blockIdx.x * 256 + threadIdx.x;
        for (size_t i = (me + step - before % step) % step; i < a.part[p].n16; i += step)
            a.part[p].dst[i] = a.part[p].src ? a.part[p].src[i] : make_uint4(0u, 0u, 0u, 0u);
        before += a.part[p].n16;
    }
}

}  // namespace

hipError_t launch_copy_out(void* dst_host, const void* src_dev, size_t bytes, hipStream_t stream) {
    if (bytes == 0) return hipSuccess;
    const size_t n16 = (bytes + 15) / 16;
    const size_t want = (n16 + 255) / 256;
    const unsigned blocks = (unsigned)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(k_copy_out, dim3(blocks), dim3(256), 0, stream, static_cast<uint4*>(dst_host),
                       static_cast<const uint4*>(src_dev), n16);
    return hipGetLastError();
}

hipError_t launch_copies(const CopyPart* what, int n, hipStream_t stream) {
    CopyArgs a;
    size_t n16 = 0;
    for (int i = 0; i < kCopyParts; ++i) {
        const bool there = i < n && what[i].bytes > 0;
        a.part[i] = CopyOut{there ? static_cast<uint4*>(what[i].dst) : nullptr, there ? static_cast<const uint4*>(what[i].src) : nullptr,
                            there ? (what[i].bytes + 15) / 16 : 0};
        n16 += a.part[i].n16;
    }
    if (n > kCopyParts) return hipErrorInvalidValue;
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + 255) / 256;
    hipLaunchKernelGGL(k_copies, dim3((unsigned)(want < 2048 ? want : 2048)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_rank_sort(const unsigned long long* valid, const unsigned long long* valid2, unsigned long long* sorted,
                            const DevPostSeg* segs, int n_segs, unsigned blocks, hipStream_t stream) {
    if (n_segs == 0 || blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rank_sort, dim3(blocks), dim3(256), 0, stream, valid, valid2, sorted, segs, n_segs);
    return hipGetLastError();
}

hipError_t launch_topk_jobs(const DevTopkJob* jobs, unsigned n_jobs, int max_k, long long max_n, hipStream_t stream) {
    if (n_jobs == 0) return hipSuccess;
    if (few(max_n, max_k)) hipLaunchKernelGGL(k_few_jobs, dim3(n_jobs), dim3(few_threads(max_n)), 0, stream, jobs);
    else if (max_k <= 64 && max_n <= 512) hipLaunchKernelGGL((k_topk_jobs<kWave, 128>), dim3(n_jobs), dim3(kWave), 0, stream, jobs);
    else if (max_k <= 256 && max_n <= 2048) hipLaunchKernelGGL((k_topk_jobs<256, 512>), dim3(n_jobs), dim3(256), 0, stream, jobs);
    else hipLaunchKernelGGL((k_topk_jobs<kSelThreads, kSelBuffer>), dim3(n_jobs), dim3(kSelThreads), 0, stream, jobs);
    return hipGetLastError();
}

__global__ __launch_bounds__(kWave) void k_gather_rows(const DevGatherSeg* __restrict__ segs, const p2_program* __restrict__ progs,
                                                       const double* __restrict__ costs, int n_cost, const long long* __restrict__ pos,
                                                       p2_program* __restrict__ sel_progs, double* __restrict__ sel_costs) {
    const DevGatherSeg S = segs[blockIdx.x];
    for (uint32_t t = threadIdx.x; t < S.rows; t += kWave) {
        const long long p = pos[S.pos_first + t];
        if (p < 0) continue;                         // (the host reports a selection that came back short)
        const size_t src = (size_t)(S.out_first + (unsigned long long)p), dst = (size_t)(S.pos_first + t);
        sel_progs[dst] = progs[src];
        for (int c = 0; c < n_cost; ++c) sel_costs[dst * n_cost + c] = costs[src * n_cost + c];
    }
}

hipError_t launch_gather_rows(const DevGatherSeg* segs, unsigned n_segs, const p2_program* progs, const double* costs, int n_cost,
                              const long long* pos, p2_program* sel_progs, double* sel_costs, hipStream_t stream) {
    if (n_segs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_rows, dim3(n_segs), dim3(kWave), 0, stream, segs, progs, costs, n_cost, pos, sel_progs, sel_costs);
    return hipGetLastError();
}

size_t topk_control_bytes() { return sizeof(SelControl); }
size_t topk_scratch_bytes(long long n, int k) { return (size_t)sel_blocks(n) * (size_t)sel_share(k) * 24; }

hipError_t launch_topk(const double* cost, long long stride, const unsigned long long* index, long long n, int k,
                       long long* out_pos, void* scratch, void* control, uint32_t* nan_out, hipStream_t stream, int fresh) {
    if (n <= 0 || k <= 0) return hipSuccess;
    const unsigned blocks = sel_blocks(n);
    const size_t cap = (size_t)blocks * sel_share(k);
    double* lc = static_cast<double*>(scratch);
    unsigned long long* li = static_cast<unsigned long long*>(scratch) + cap;
    SelControl* ctl = static_cast<SelControl*>(control);
    if (few(n, k)) {
        hipLaunchKernelGGL(k_few_column, dim3(few_blocks(n)), dim3(few_threads(n)), 0, stream, SelSource{cost, index, nullptr, stride, 1}, n, k, ctl, lc, li,
                           li + cap, out_pos, (long long)(k < n ? k : n), nan_out, fresh);
        return hipGetLastError();
    }
    const bool sampled = sel_sampled(n, k);
    if (sampled) {
        const long long m = n / (kSelSample * 64) * 64;
        hipLaunchKernelGGL(k_topk_column, dim3(sel_blocks(m)), dim3(kSelThreads), 0, stream, SelSource{cost, index, nullptr, stride, kSelSample}, m, k,
                           1, 0, ctl, lc, li, li + cap, (uint32_t)cap, nullptr, 0ll, nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_topk_column, dim3(blocks), dim3(kSelThreads), 0, stream, SelSource{cost, index, nullptr, stride, 1}, n, k, 0, sampled ? 1 : 0, ctl,
                       lc, li, li + cap, (uint32_t)cap, out_pos, (long long)(k < n ? k : n), nan_out);
    return hipGetLastError();
}

// ---- selection without any allocation ------------------------------------------------------------
// What the blocks of a selection leave for the last one (24 bytes an entry) and the words they share lie in device
// memory.  For callers that may not allocate, that memory is a fixed array in the library's device image: every GPU the
// library runs on holds its own copy at its own address for the life of the process, and all calls on one
// GPU share it.  Host code never uses the array's name as an address: the device address is asked for once
// per device and kept.
constexpr int kFixedTopkMaxK = 64;
constexpr size_t kFixedTopkListBytes = (size_t)3 << 20;                        // 256 blocks x 320 entries x 24 B fit
static __device__ __align__(256) unsigned char scratch[kFixedTopkListBytes + 256];   // lists, then the shared words

namespace {
constexpr int kMaxGpus = 64;
std::mutex g_fixed_mutex;
void* g_fixed_ptr[kMaxGpus] = {nullptr};

// The shared words and the flag cleared, and every position -1 beforehand: a block of an overlapping call can take the
// last block's turn away, and then nothing writes the positions.
__global__ __launch_bounds__(kFixedTopkMaxK) void k_clear_control(SelControl* c, uint32_t* flag, long long* out_pos, int n_out) {
    if ((int)threadIdx.x < n_out) out_pos[threadIdx.x] = -1ll;
    if (threadIdx.x != 0) return;
    *c = SelControl{0u, 0u, 0u, 0u, 0.0};
    if (flag) *flag = 0u;
}

// Device address of `scratch` on the current device.
hipError_t fixed_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxGpus) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_fixed_mutex);
    if (!g_fixed_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_fixed_ptr[dev] = p;
    }
    *out = g_fixed_ptr[dev];
    return hipSuccess;
}
}  // namespace

int topk_fixed_max_k() { return kFixedTopkMaxK; }

hipError_t launch_topk_fixed(const double* cost, long long stride, const unsigned long long* index, long long n, int k,
                             long long* out_pos, uint32_t* nan_flag, hipStream_t stream) {
    if (n <= 0 || k <= 0) return hipSuccess;
    if (k > kFixedTopkMaxK || topk_scratch_bytes(n, k) > kFixedTopkListBytes) return hipErrorInvalidValue;
    void* base = nullptr;
    hipError_t e = fixed_scratch(&base);
    if (e != hipSuccess) return e;
    // (the shared words are cleared here although a call leaves them clear: calls that overlapped against the rule must
    //  not spoil the ones after them.  A fill kernel, so that the call can be recorded into a graph)
    SelControl* ctl = reinterpret_cast<SelControl*>(static_cast<unsigned char*>(base) + kFixedTopkListBytes);
    if (few(n, k) && few_blocks(n) == 1u) return launch_topk(cost, stride, index, n, k, out_pos, base, ctl, nan_flag, stream, 1);
    hipLaunchKernelGGL(k_clear_control, dim3(1), dim3(kFixedTopkMaxK), 0, stream, ctl, nan_flag, out_pos, (int)(k < n ? k : n));
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_topk(cost, stride, index, n, k, out_pos, base, ctl, nan_flag, stream);
}

}  // namespace p2
