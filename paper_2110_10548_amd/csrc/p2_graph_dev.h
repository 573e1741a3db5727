// What the state-graph kernels of p2_graph.hip and p2_skeleton.hip share.
#pragma once
#include "p2_compact_dev.h"

#include <type_traits>

namespace p2 {
namespace {

using u64 = unsigned long long;
constexpr uint32_t kGoalEdge = 0x7fffffu;   // target of an edge that ends at the goal
constexpr int kDigitShift = 23;
constexpr uint32_t kMostTries = 256;    // slots looked at before a table counts as full
constexpr int kFinishThreads = 1024;
constexpr int kAloneThreads = 1024;

// Pointers to the global address space.  (Through plain pointers, where the compiler cannot tell, the accesses would be flat
// ones, which count as LDS accesses too: every lane exchange would wait for the stores before it.)
#define P2_GLOBAL __attribute__((address_space(1)))
#define P2_LOCAL __attribute__((address_space(3)))
typedef u64 u64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename To, typename From>
__device__ __forceinline__ P2_GLOBAL To* in_global(From* p) { return (P2_GLOBAL To*)p; }

// A skeleton's instructions by digit, in LDS: their levels and the devices that take part.
struct Instr {
    int op, lg, ls;
    uint32_t range;                         // varied bits of the device number
    u64 part;
};
struct PatternTable {
    uint32_t shape[kGraphPatterns];
    u64 part[kGraphPatterns];
    uint16_t instr[kGraphPatterns * 5];
    // (not read in place: both tables by one uniform index, the second was addressed by the compiler as base + index, + 7 * index,
    //  and a scalar load ignores the lowest bits of either)
    __device__ __forceinline__ void open(const DevGraph& D, const DevQuery& q) {
        if ((int)threadIdx.x < D.n_pat) { shape[threadIdx.x] = D.shape[threadIdx.x]; part[threadIdx.x] = D.part[threadIdx.x]; }
        if ((int)threadIdx.x < D.alphabet) instr[threadIdx.x] = q.instr_of_digit[threadIdx.x];
    }
    __device__ __forceinline__ Instr of(uint32_t digit) const {      // (the same for all lanes)
        const uint32_t ins = (uint32_t)__builtin_amdgcn_readfirstlane((int)instr[digit]);
        const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)shape[ins >> 3]);
        const u64 p = part[ins >> 3];
        Instr i;
        i.op = (int)(ins & 7u); i.lg = (int)(s & 15u); i.ls = (int)((s >> 4) & 15u);
        i.range = ((1u << i.lg) - 1u) << i.ls;
        i.part = (u64)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p) | (u64)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32;
        return i;
    }
};
// Rows held by the devices of one query's group while a program runs.  Devices whose digits are zero at the same levels hold
// equally many, so they are one number for each of the skeleton's devices, a digit other than zero standing for all of them.
// No state and no device but the skeleton's is looked at.  A lane works for a query: the lanes share the instructions and differ
// in sizes alone.
template <int LOG>
struct HeldRows {
    static constexpr int N = 1 << LOG;
    uint32_t size[LOG], cnt[N];
    __device__ __forceinline__ void start(const P2_GLOBAL DevMember& own, int skeleton) {
#pragma unroll
        for (int l = 0; l < LOG; ++l) size[l] = own.size[l];
#pragma unroll
        for (int d = 0; d < N; ++d) cnt[d] = d < skeleton ? (uint32_t)own.R : 0u;
    }
    __device__ __forceinline__ void step(const Instr& i) {
        if (i.op == OP_RS) {
            uint32_t g = 1u;
#pragma unroll
            for (int l = 0; l < LOG; ++l) g *= ((i.range >> l) & 1u) != 0u ? size[l] : 1u;
            const float share = 1.0f / (float)g;         // (at most 512 rows, and they divide: the nearest whole number is the quotient)
#pragma unroll
            for (int d = 0; d < N; ++d)
                if ((i.part >> d) & 1ull) cnt[d] = (uint32_t)((float)cnt[d] * share + 0.5f);
        } else if (i.op == OP_AG) {
#pragma unroll
            for (int l = 0; l < LOG; ++l) {
                if (((i.range >> l) & 1u) == 0u) continue;
#pragma unroll
                for (int d = 0; d < N; ++d) {
                    if ((d >> l) & 1) continue;
                    const uint32_t sum = cnt[d] + cnt[d | 1 << l] * (size[l] - 1u);
                    if ((i.part >> d) & 1ull) { cnt[d] = sum; cnt[d | 1 << l] = sum; }
                }
            }
        } else if (i.op == OP_RD) {
#pragma unroll
            for (int d = 0; d < N; ++d)
                if (((i.part >> d) & 1ull) != 0ull && ((uint32_t)d & i.range) != 0u) cnt[d] = 0u;
        } else if (i.op == OP_BC) {
#pragma unroll
            for (int l = 0; l < LOG; ++l) {
                if (((i.range >> l) & 1u) == 0u) continue;
#pragma unroll
                for (int d = 0; d < N; ++d)
                    if (((d >> l) & 1) != 0 && ((i.part >> d) & 1ull) != 0ull) cnt[d] = cnt[d & ~(1 << l)];
            }
        }
    }
    // the instructions of a path, a byte each (digit + 1), the last one lowest
    __device__ __forceinline__ void follow(u64 path, const PatternTable& T) {
        for (int at = 8 * (P2_MAX_LEN - 1); at >= 0; at -= 8) {
            const uint32_t code = (uint32_t)(path >> at) & 255u;
            if (code != 0u) step(T.of(code - 1u));
        }
    }
    // What the next instruction asks of the busiest uplink: at the groups' first devices the rows that set their bytes (the members'
    // common ones, the root's, or all together), summed over what a unit of each hardware level holds: all digits of the levels
    // further in, as far as they number groups.
    __device__ __forceinline__ double busiest(const Instr& i, const P2_GLOBAL DevMember& own) const {
        const uint32_t R = own.R, k = own.k, inside = own.inside;
        uint32_t w[N], most_of[LOG + 1];
#pragma unroll
        for (int d = 0; d < N; ++d) w[d] = cnt[d];
        if (i.op == OP_AG) {
#pragma unroll
            for (int l = 0; l < LOG; ++l)
                if (((i.range >> l) & 1u) != 0u)
#pragma unroll
                    for (int d = 0; d < N; ++d)
                        if (((d >> l) & 1) == 0) w[d] += w[d | 1 << l] * (size[l] - 1u);
        }
#pragma unroll
        for (int d = 0; d < N; ++d)
            if (((i.part >> d) & 1ull) == 0ull || ((uint32_t)d & i.range) != 0u) w[d] = 0u;
#pragma unroll
        for (int t = 0; t <= LOG; ++t) {
            uint32_t most = 0u;
            if (t <= i.ls) {
#pragma unroll
                for (int d = 0; d < N; ++d) most = w[d] > most ? w[d] : most;
            }
            most_of[t] = most * k / R;
            if (t < LOG && t < i.ls) {
#pragma unroll
                for (int d = 0; d < N; ++d)
                    if (((d >> t) & 1) == 0) { w[d] += w[d | 1 << t] * (size[t] - 1u); w[d | 1 << t] = 0u; }
            }
        }
        double best = 0.0;
#pragma unroll
        for (int j = 0; j < P2_MAX_LEVELS; ++j) {
            const int t = (int)((inside >> (4 * j)) & 15u), at = t < i.ls ? t : i.ls;
            uint32_t load = 0u;
#pragma unroll
            for (int x = 0; x <= LOG; ++x) load = x == at ? most_of[x] : load;
            if (t < i.ls + i.lg) best = fmax(best, (double)(load * own.copies[j]) * own.inv_bw[j]);
        }
        return best;
    }
};

}  // namespace
}  // namespace p2
