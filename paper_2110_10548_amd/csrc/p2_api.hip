// The C ABI of include/p2.h: argument checks, planning, table upload, kernel launches and
// copy-back.  All arithmetic of the method runs in the kernels; this file only moves data.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <exception>
#include <atomic>
#include <thread>
#include <limits>
#include <string>
#include <vector>

#include "p2_device.h"
#include "p2_plan.h"

namespace p2 {
hipError_t launch_cost_literal(const DevQuery* q, int R, int k, const unsigned long long* sorted, uint32_t n,
                               p2_program* out_prog, double* out_cost, int only_missing, void* gscratch,
                               hipStream_t stream);
}

namespace {

thread_local std::string g_err;

struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
    hipError_t ensure(size_t bytes) {
        if (bytes <= cap) return hipSuccess;
        if (p) (void)hipFree(p);
        p = nullptr; cap = 0;
        size_t want = std::max(bytes, (size_t)4096);
        want = (want + 4095) & ~(size_t)4095;
        hipError_t e = hipMalloc(&p, want);
        if (e == hipSuccess) cap = want;
        return e;
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr; cap = 0;
    }
};
// grow a device buffer to `bytes`, keeping its first `keep` bytes
hipError_t grow_keep(DevBuf& b, size_t bytes, size_t keep, hipStream_t stream) {
    if (bytes <= b.cap) return hipSuccess;
    size_t want = std::max(bytes, b.cap * 2);
    want = (want + 4095) & ~(size_t)4095;
    void* np = nullptr;
    hipError_t e = hipMalloc(&np, want);
    if (e != hipSuccess) return e;
    if (b.p && keep) {
        e = hipMemcpyAsync(np, b.p, keep, hipMemcpyDeviceToDevice, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) { (void)hipFree(np); return e; }
    }
    if (b.p) (void)hipFree(b.p);
    b.p = np; b.cap = want;
    return hipSuccess;
}

struct HostBuf {
    void* p = nullptr;
    size_t cap = 0;
    hipError_t ensure(size_t bytes) {
        if (bytes <= cap) return hipSuccess;
        if (p) (void)hipHostFree(p);
        p = nullptr; cap = 0;
        size_t want = std::max(bytes, (size_t)4096);
        want = (want + 4095) & ~(size_t)4095;
        hipError_t e = hipHostMalloc(&p, want, hipHostMallocDefault);
        if (e == hipSuccess) cap = want;
        return e;
    }
};

// Event pairs around single launches: a pool that grows on demand and is kept.
struct SpanRec {
    enum Kind { kClassify = 0, kLiteral = 1, kMaterialize = 2, kGroup = 3, kKinds = 4 };
    struct Span { int kind; size_t first; int dispatches; };
    bool on = false;
    bool kernels_only = false;         // only the classification and the building of children are timed
    bool open = false;                 // the span begun last is being recorded
    std::vector<hipEvent_t> pool;
    std::vector<Span> spans;
    size_t used = 0;
    hipError_t begin(int kind, hipStream_t stream, int dispatches = 1) {
        open = on && !(kernels_only && kind != kClassify && kind != kMaterialize);
        if (!open) return hipSuccess;
        while (pool.size() < used + 2) {
            hipEvent_t e = nullptr;
            const hipError_t rc = hipEventCreate(&e);
            if (rc != hipSuccess) return rc;
            pool.push_back(e);
        }
        spans.push_back(Span{kind, used, dispatches});
        used += 2;
        return hipEventRecord(pool[used - 2], stream);
    }
    hipError_t end(hipStream_t stream) { return open ? hipEventRecord(pool[used - 1], stream) : hipSuccess; }
    void reset() { spans.clear(); used = 0; }
    // after the stream has been waited for: time and launches per kind, added to what is there
    hipError_t collect(float ms[kKinds], int32_t launches[kKinds]) {
        for (const Span& sp : spans) {
            float t = 0.f;
            const hipError_t rc = hipEventElapsedTime(&t, pool[sp.first], pool[sp.first + 1]);
            if (rc != hipSuccess) return rc;
            ms[sp.kind] += t;
            launches[sp.kind] += sp.dispatches;
        }
        reset();
        return hipSuccess;
    }
    void release() {
        for (auto& e : pool) (void)hipEventDestroy(e);
        pool.clear(); reset();
    }
};

// What one enumeration of the frontier engine works in: its own stream (and a second one for the literal prefixes
// of a level), its lists, its counters.  A call runs as many enumerations side by side as there are slots, a host
// thread each: an enumeration is a chain of small launches with one host wait per level, and several chains fill
// the chip where one does not.
constexpr int kFrontSlots = 4;
struct FrontSlot {
    hipStream_t stream = nullptr;         // (created by Ctx::open_slot_streams)
    DevBuf f_entries[2], f_states[2], f_sums[2], f_entries2[2], f_states2[2], f_sums2[2], f_literal[2];
    DevBuf f_surv, f_surv_literal, f_unknown, f_ctr, lit_scratch;
    DevBuf f_hash[2], f_hash2[2], f_table, f_rep[2], f_replist[2], f_codes[2], f_unk[2];     // search for equal states
    DevBuf f_sid[2], f_sid2[2], f_delta[3], f_childof[2], f_ssurv;                           // prefixes -> states -> children
    DevBuf f_rowcnt[2];                                                                      // per row of codes: how many survivors by kind
    DevBuf f_lit_parent[2], f_rest;                                                          // literal prefixes: their parents' states
    DevBuf f_walk[2];                                                                        // the last level: states worth a walk
    HostBuf h_fctr;
    SpanRec spans;
    // what the slot's launches of this call worked on (the figures of p2_profile)
    double prof_prefixes = 0.0, prof_state_bytes = 0.0, prof_lane_ops = 0.0, prof_children = 0.0, prof_mat_bytes = 0.0, prof_entries = 0.0;
    int32_t rc = 0;
    std::string err;
    void release() {
        DevBuf* dev[] = {&f_entries[0], &f_entries[1], &f_states[0], &f_states[1], &f_sums[0], &f_sums[1], &f_entries2[0], &f_entries2[1],
                         &f_states2[0], &f_states2[1], &f_sums2[0], &f_sums2[1], &f_literal[0], &f_literal[1], &f_surv, &f_surv_literal,
                         &f_unknown, &f_ctr, &lit_scratch, &f_hash[0], &f_hash[1], &f_hash2[0], &f_hash2[1], &f_table, &f_rep[0], &f_rep[1],
                         &f_replist[0], &f_replist[1], &f_codes[0], &f_codes[1], &f_unk[0], &f_unk[1], &f_sid[0], &f_sid[1], &f_sid2[0],
                         &f_sid2[1], &f_delta[0], &f_delta[1], &f_delta[2], &f_childof[0], &f_childof[1], &f_ssurv, &f_walk[0], &f_walk[1], &f_rowcnt[0], &f_rowcnt[1], &f_lit_parent[0], &f_lit_parent[1], &f_rest};
        for (DevBuf* b : dev) { if (b->p) (void)hipFree(b->p); b->p = nullptr; b->cap = 0; }
        if (h_fctr.p) (void)hipHostFree(h_fctr.p);
        h_fctr.p = nullptr; h_fctr.cap = 0;
        spans.release();
        if (stream) { (void)hipStreamDestroy(stream); stream = nullptr; }
    }
};

// Device scratch owned by the library, one set per host thread, reused between calls.
struct Ctx {
    ~Ctx();
    void release();
    DevBuf rows, rows_hdr;
    DevBuf blob, valid, rerun, sorted, progs, costs, counters, topk_scratch, topk_control, topk_pos, topk_in, topk_jobs, lit_scratch, post;
    bool topk_control_clear = false;                        // the words that the blocks of a selection share are zero
    DevBuf walks;                                           // the edges of rows that several queries share
    DevBuf sel_progs, sel_costs, gather;                    // the rows that shortlists picked, and whose they are
    HostBuf h_gather;
    DevBuf g_zero, g_mem, g_large, g_rows;                  // state-graph engine: what starts from zero, the lists, the states of large groups, whose rows are written
    HostBuf h_gctr, h_grows;
    DevBuf f_finish;                                        // frontier engine: what every query's rows are written from
    HostBuf h_finish;
    DevBuf f_rank, f_rank_runs, f_share;                                 // frontier engine: ranks of the valid programs, queries of the enumerations
    std::vector<DevBuf> f_evalid, f_egsums;                 // ... per enumeration: valid candidate indices, their cost sums
    FrontSlot slots[kFrontSlots];
    static constexpr int kSpareStreams = 6;
    hipStream_t spare_streams[kSpareStreams] = {};          // created beside the slots' streams and found to share a queue with one: never used
    DevBuf probe_sink;
    hipError_t open_slot_streams(int n_slots);
    hipError_t open_topk_control(hipStream_t stream) {
        const void* before = topk_control.p;
        hipError_t e = topk_control.ensure(p2::topk_control_bytes());
        if (e == hipSuccess && (topk_control.p != before || !topk_control_clear)) e = hipMemsetAsync(topk_control.p, 0, p2::topk_control_bytes(), stream);
        return e;
    }
    hipEvent_t front_go = nullptr;                          // the call's stream has reached the enumerations
    hipEvent_t slot_done[kFrontSlots] = {};                 // a slot's stream has got through what it was given
    HostBuf h_rows, h_rows_hdr;
    hipStream_t copy_stream = nullptr;      // uploads that overlap with the kernels of the call's stream
    hipEvent_t copy_done = nullptr;
    HostBuf h_blob, h_counters, h_progs, h_costs, h_pos, h_post, h_topk_jobs, h_topk_nan, h_fshare;
};
thread_local Ctx g_ctx;

// The streams of the slots.  The runtime deals a process's streams out to its hardware queues (four unless the
// caller's environment says otherwise) as they are created, streams that share a queue take turns, and which queue a
// new stream lands on depends on every stream the process has created before.  So the library looks: it creates a
// handful of streams, runs a short one-block kernel on pairs of them (side by side: the time of one; taking turns:
// of two) and gives the slots streams that do not take turns with each other; the other streams stay unused.  With
// fewer independent queues than slots the remaining slots share.  Only the overlap depends on this, never a result;
// a pair that is wrongly taken to share (the host thread lost its turn while timing) costs overlap and nothing else.
// The look takes some 5 ms, once per thread, and a call with one enumeration has nothing to overlap: it opens slot 0's
// stream alone, and the look waits for the first call that uses a second slot (which starts from that stream).
__global__ __launch_bounds__(64) void k_queue_probe(uint32_t* sink, int n) {
    uint32_t x = threadIdx.x + 1u;
    for (int i = 0; i < n; ++i) x = x * 1664525u + 1013904223u;
    if (x == 0x9e3779b9u) sink[0] = x;               // (keeps the loop; the sink is the library's own word)
}
hipError_t Ctx::open_slot_streams(int n_slots) {
    if (slots[n_slots > 1 ? 1 : 0].stream) return hipSuccess;
    if (n_slots == 1) return hipStreamCreateWithFlags(&slots[0].stream, hipStreamNonBlocking);
    constexpr int kCandidates = kFrontSlots + kSpareStreams;
    constexpr int kProbeSteps = 8000;                 // some 0.1 ms: several times what a launch and a wait take
    hipStream_t made[kCandidates] = {};
    hipError_t e = probe_sink.ensure(256);
    made[0] = slots[0].stream;                       // (of an earlier call with one enumeration)
    for (int i = made[0] ? 1 : 0; i < kCandidates && e == hipSuccess; ++i) e = hipStreamCreateWithFlags(&made[i], hipStreamNonBlocking);
    auto timed = [&](hipStream_t a, hipStream_t b, double& ms) -> hipError_t {
        const auto t0 = std::chrono::steady_clock::now();
        hipLaunchKernelGGL(k_queue_probe, dim3(1), dim3(64), 0, a, static_cast<uint32_t*>(probe_sink.p), kProbeSteps);
        if (b) hipLaunchKernelGGL(k_queue_probe, dim3(1), dim3(64), 0, b, static_cast<uint32_t*>(probe_sink.p), kProbeSteps);
        hipError_t r = hipGetLastError();
        const hipError_t ra = hipStreamSynchronize(a);
        const hipError_t rb = b ? hipStreamSynchronize(b) : hipSuccess;
        ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        return r != hipSuccess ? r : ra != hipSuccess ? ra : rb;
    };
    int chosen[kFrontSlots], n_chosen = 0;
    bool taken[kCandidates] = {};
    if (e == hipSuccess) {
        double one = 1e30, t = 0.0;
        for (int rep = 0; rep < 4 && e == hipSuccess; ++rep) {        // (the first launch also loads the kernel)
            e = timed(made[0], nullptr, t);
            if (rep > 0) one = std::min(one, t);
        }
        for (int c = 0; c < kCandidates && n_chosen < kFrontSlots && e == hipSuccess; ++c) {
            bool apart = true;
            for (int k = 0; k < n_chosen && apart && e == hipSuccess; ++k) {
                double best = 1e30;
                for (int rep = 0; rep < 2 && e == hipSuccess; ++rep) { e = timed(made[chosen[k]], made[c], t); best = std::min(best, t); }
                apart = best < 1.5 * one;
            }
            if (apart && e == hipSuccess) { chosen[n_chosen++] = c; taken[c] = true; }
        }
        for (int c = 0; c < kCandidates && n_chosen < kFrontSlots; ++c)
            if (!taken[c]) { chosen[n_chosen++] = c; taken[c] = true; }
    }
    if (e != hipSuccess) {
        for (hipStream_t st : made) if (st && st != slots[0].stream) (void)hipStreamDestroy(st);
        return e;
    }
    for (int t = 0; t < kFrontSlots; ++t) slots[t].stream = made[chosen[t]];
    int n_spare = 0;
    for (int c = 0; c < kCandidates; ++c) if (!taken[c]) spare_streams[n_spare++] = made[c];
    return hipSuccess;
}

// Frontier lists shorter than this are judged entry by entry: grouping them by state would cost more than it saves.
constexpr uint32_t kGroupMin = 256;

struct Prof {
    ~Prof();
    void release();
    bool on = false;
    bool kernels_only = false;      // p2_set_profiling(2): of the frontier engine's launches, only classification and children
    hipEvent_t ev[6] = {};          // evaluation begin / end, post end, frontier begin / end, post begin
    p2_profile last = {};
};
thread_local Prof g_prof;

// What a host thread's calls have cached on the device is given back when the thread ends, or on request
// (p2_release_thread).  The thread that loaded the library is left alone at process exit: by then the HIP
// runtime may be shutting down, and the process's memory goes with it anyway.
const std::thread::id g_loader_thread = std::this_thread::get_id();

void Ctx::release() {
    DevBuf* dev[] = {&rows, &rows_hdr, &blob, &valid, &rerun, &sorted, &progs, &costs, &counters, &topk_scratch, &topk_control, &topk_pos,
                     &topk_in, &topk_jobs, &lit_scratch, &post, &f_rank, &f_rank_runs, &f_share, &walks, &sel_progs, &sel_costs, &gather, &f_finish, &probe_sink, &g_zero, &g_mem, &g_large, &g_rows};
    for (DevBuf* b : dev) { if (b->p) (void)hipFree(b->p); b->p = nullptr; b->cap = 0; }
    for (auto* v : {&f_evalid, &f_egsums}) {
        for (DevBuf& b : *v) if (b.p) (void)hipFree(b.p);
        v->clear();
    }
    for (FrontSlot& sl : slots) sl.release();
    for (hipStream_t& sp : spare_streams) { if (sp) (void)hipStreamDestroy(sp); sp = nullptr; }
    HostBuf* host[] = {&h_rows, &h_rows_hdr, &h_blob, &h_counters, &h_progs, &h_costs, &h_pos, &h_post, &h_topk_jobs, &h_topk_nan, &h_fshare, &h_gather, &h_finish, &h_gctr, &h_grows};
    for (HostBuf* b : host) { if (b->p) (void)hipHostFree(b->p); b->p = nullptr; b->cap = 0; }
    if (front_go) { (void)hipEventDestroy(front_go); front_go = nullptr; }
    for (hipEvent_t& ev : slot_done) { if (ev) (void)hipEventDestroy(ev); ev = nullptr; }
    if (copy_done) { (void)hipEventDestroy(copy_done); copy_done = nullptr; }
    if (copy_stream) { (void)hipStreamDestroy(copy_stream); copy_stream = nullptr; }
}
Ctx::~Ctx() { if (std::this_thread::get_id() != g_loader_thread) release(); }
void Prof::release() {
    for (auto& e : ev) { if (e) (void)hipEventDestroy(e); e = nullptr; }
    on = false;
}
Prof::~Prof() { if (std::this_thread::get_id() != g_loader_thread) release(); }

int32_t fail(int32_t code, const std::string& msg) {
    g_err = msg;
    return code;
}
// Stream of the call in progress on this thread.  When a HIP call fails or the host throws, what the call has
// queued so far on this stream, the uploads' and the slots' (kernels and copies that use the cached pinned and
// device buffers) is waited for before the error goes back to the caller, so that the next call does not reuse
// buffers that are still in flight.
thread_local hipStream_t g_call_stream = nullptr;
thread_local bool g_call_active = false;
void wait_for_call() {
    if (!g_call_active) return;
    (void)hipStreamSynchronize(g_call_stream);
    if (g_ctx.copy_stream) (void)hipStreamSynchronize(g_ctx.copy_stream);
    for (const FrontSlot& sl : g_ctx.slots) if (sl.stream) (void)hipStreamSynchronize(sl.stream);
    (void)hipGetLastError();
}
int32_t hip_fail(hipError_t e, const char* what) {
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    (void)hipGetLastError();
    wait_for_call();
    return P2_EDEVICE;
}
struct CallScope {
    int thrown = std::uncaught_exceptions();
    explicit CallScope(hipStream_t s) { g_call_stream = s; g_call_active = true; }
    ~CallScope() {
        if (std::uncaught_exceptions() > thrown) wait_for_call();
        g_call_active = false; g_call_stream = nullptr;
    }
};
#define P2_HIP(call)                                      \
    do {                                                  \
        hipError_t e_ = (call);                           \
        if (e_ != hipSuccess) return hip_fail(e_, #call); \
    } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Selections over at most this many valid programs go into one launch for the whole batch (one block each, at most 32
// tiles of 8192; the 11 of 83 920 programs take 32 us with 10 kept, 100 with 1024); longer lists are selected from by the
// whole chip, one after the other (371 970 programs: 50 and 135 us).
constexpr size_t kTopkJobMax = 1 << 18;
// Queries of one graph from which on their rows are written once for all of them: as many as a block of k_graph_sums takes side by
// side.  Whole calls, us, a walk per row and query / the rows once: queries of [2 4 8 8], six instructions, 83 920 rows each: 8
// 411 / 426, 16 472 / 464, 32 603 / 535; of [4 8 8], five instructions, 2 549 rows: 16 192 / 201, 32 270 / 272, 140 737 to 753 / 706 to 750; three
// instructions, 80 rows: 32 222 / 223.
constexpr size_t kSharedQueries = p2::kSumMembers;

// Room for the rows that shortlists may be selected from before their number is known: with all collectives and forms a query has
// as many as there is room for, with a narrowed alphabet it may have a handful of 83 920.
constexpr size_t kShortlistBytes = (size_t)4 << 30, kNarrowedShortlistBytes = (size_t)64 << 20;

// Engine AUTO walks candidate spaces of at most this many programs index by index ...
constexpr unsigned long long kWalkMax = 1ull << 30;
// ... where the shared-prefix engine can (its kernels need at most 64 devices and power-of-two patterns).  What is left
// for the compact engine, one candidate per lane with its state in LDS, is faster enumerated by size with pruning once the
// candidates or the states are many: the enumeration takes some 200 us plus 70 us a level whatever the candidates (3 x 4 x 6
// devices, 4.2 M programs: 0.55 ms against 14.3 ms; 16 x 12, 168 420: 0.59 against 11.6; 12 x 12, 420: 0.32 against
// 0.70), the compact engine less than that only for few devices and candidates (6 x 8 devices, 168 420 programs: 0.37 ms
// against 0.47; 3.4 M: 1.25 against 0.56; 3 x 4, 3.4 M: 0.32 against 0.52; 80 devices, 30 programs: 0.28 against 0.27).
// This is a query by itself; what a batch of them does, walks_together() says.
bool pruned_is_faster(const p2::Plan& pl) {
    bool shared = pl.R <= 64;
    for (const p2::Pattern& p : pl.patterns) shared = shared && p2::reg_shape_of(p.g, p.s, p.master, 6) >= 0;
    if (shared) return false;
    if (pl.R > 64) return pl.n_candidates >= 100;
    return pl.n_candidates * (unsigned long long)pl.R >= 80000000ull;
}

// Rows that the state-graph engine holds per device: one for every block of k / R chunks where the blocks come out even.
int graph_rows(const p2::Plan& pl) { return pl.k % pl.R == 0 ? pl.R : pl.k; }
// What the state-graph engine takes over from the others under AUTO: groups of up to 64 devices with power-of-two
// patterns (a lane plays a device), up to 64 rows (a 64-bit word holds a set of them).  The number of states depends on
// the levels and the size limit, hardly on the sizes of the levels: at most 42 for two levels, 1 008 for three, 17 427 for
// four with six instructions, 50 647 for five with five, 29 599 for six with four; past these the counts of a
// graph no longer fit in a compute unit's LDS.
bool graph_applies(const p2::Plan& pl) {
    if (pl.hierarchy != P2_HIERARCHY_COLLAPSED || pl.frontier_pairs != P2_FRONTIER_PAIRS_AUTO || pl.alphabet == 0) return false;
    if (pl.R < 2 || pl.R > 64 || graph_rows(pl) > 64) return false;
    const size_t n_pat = pl.patterns.size();
    if (n_pat > (size_t)p2::kGraphPatterns || pl.max_len > (n_pat <= 9 ? 7 : n_pat <= 16 ? 6 : n_pat <= 25 ? 5 : 4)) return false;
    for (const p2::Pattern& p : pl.patterns)
        if (p2::reg_shape_of(p.g, p.s, p.master, 6) < 0) return false;
    return true;
}
// What it takes over from the frontier engine under AUTO: the same size limits, any patterns; the states are worked on by
// the frontier's kernels, two pairs a device, which must fit in a compute unit's LDS.  The enumeration waits for the host
// after every level and keeps every program's sums; the graph keeps neither (one query of [3 4 6] 527 us by enumeration,
// 352 by the graph; [2 4 8 8], 512 devices, 6 300 and 3 230; 512 queries of [2 4 8 8] 39.7 ms and 15.5).  Past the
// size limits the counts of a graph no longer fit in LDS: the enumeration goes on there, and also for three levels and seven
// instructions with AllGathers among them, which lead to states of three pairs before the last two levels, where the graph
// would be given up ([3 4 6]: 1.24 ms enumerated, 1.80 with the graph tried first).
bool large_graph_applies(const p2::Plan& pl) {
    if (pl.hierarchy != P2_HIERARCHY_COLLAPSED || pl.frontier_pairs != P2_FRONTIER_PAIRS_AUTO || pl.alphabet == 0 || pl.R < 2) return false;
    const size_t n_pat = pl.patterns.size();
    const bool gathers = std::find(pl.ops, pl.ops + pl.n_ops, (int)p2::OP_AG) != pl.ops + pl.n_ops;
    const int nine = n_pat <= 4 || !gathers ? 7 : 6;
    if (n_pat > (size_t)p2::kGraphPatterns || pl.max_len > (n_pat <= 9 ? nine : n_pat <= 16 ? 6 : n_pat <= 25 ? 5 : 4)) return false;
    return p2::frontier_max_pairs(pl.R, graph_rows(pl)) == 2;
}
// A call that walks some of its queries in any case has its state graphs' queries walked beside them, in the same launches,
// if none has more candidates (times devices: a walk's cost) or patterns than this: the graphs' chain of launches would come
// on top.  Beside [3], three instructions, walked with it and with a graph: [4 4], four (2.7 million) 112 us and 126; ten
// groups of two and three levels, three (up to 0.8 million), 137 and 157; [2 4 4], three (3 million) 124 and 126; but [4 4 4], three (6
// million) 135 and 128, [2 2], five (14 million) 143 and 121, and with 16 patterns, two instructions, 167 and 119, with 25 216 and 120.
constexpr unsigned long long kWalkedBesideMax = 1ull << 22;
constexpr size_t kWalkedBesidePatterns = 9;
bool walks_beside(const p2::Plan& pl) {
    return pl.n_candidates <= kWalkedBesideMax / (unsigned long long)pl.R && pl.patterns.size() <= kWalkedBesidePatterns;
}
// Whether a structure's graph is that of its skeleton, the structure of as many levels of two devices each.  With rows that
// ReduceScatters cut into whole blocks, a rule sees of a state which chunk sets and masks are equal, disjoint or contained in
// each other, and these relations do not depend on how many devices a level has; where chunk sets of different shapes
// overlap (a ReduceScatter after an AllGather over an outer level, its blocks as large as the levels' sizes say) they do, but
// with three levels not before the sixth instruction, which only counts if it ends at the goal.  That is not a proof for every
// size, but there are finitely many, and tests/sweep_skeletons.py has compared programs, counts and costs with those of the devices' own
// graphs or enumerations, to the bit: all 15 407 lists of one to six levels with up to 512 devices, at the size limits below and at a
// smaller one each.  (Seven instructions of three levels are not the same: 3 x 4 x 2 has fewer prefixes.)
// Chunks that are no multiple of the devices (up to kNarrowLevels levels): with R / gcd(k, R) finer chunks for each the rows are
// blocks of a whole number of them, the programs are those of the full rows whose ReduceScatters all divide, and a state's rule
// needs no more than how many chunks a device holds, which the states keep.  Compared in the same way for the lists of one to four
// levels with every number of chunks that divides the devices and one that does not, 325 000 queries; and by
// tests/test_skeleton.py with the oracle, for few devices with every number of chunks.
// Used with all collectives and forms, with which it was checked (a narrowed alphabet's programs are among these, but how many
// prefixes it has was not compared), and for single instructions, which the first state decides.
constexpr int kSkeletonMaxLen[p2::kSkeletonLevels + 1] = {0, 7, 7, 6, 6, 5, 4};
int group_levels(const p2::Plan& pl) {
    int n = 0;
    for (int j = 0; j < pl.n; ++j) n += pl.f[j] > 1 ? 1 : 0;
    return n;
}
bool whole_alphabet(const p2::Plan& pl) { return pl.op_mask == 31u && pl.form_mask == 7u; }
bool has_skeleton(const p2::Plan& pl) {
    const int levels = group_levels(pl);
    return (whole_alphabet(pl) || pl.max_len == 1) && levels <= p2::kSkeletonLevels && pl.max_len <= kSkeletonMaxLen[levels] &&
           (pl.k % pl.R == 0 || levels <= p2::kNarrowLevels);
}
// What a query's costs need beside the skeleton's graph.
void describe_member(const p2::Plan& pl, p2::DevMember& m) {
    std::memset(&m, 0, sizeof m);
    m.R = (uint16_t)pl.R; m.k = (uint16_t)pl.k;
    for (int l = 0; l < p2::kSkeletonLevels; ++l) m.size[l] = 1;
    int copies = pl.D / pl.R, inside = group_levels(pl);
    for (int j = 0; j < pl.n; ++j) {
        copies /= pl.h[j] / pl.f[j];
        if (pl.f[j] > 1) m.size[--inside] = (uint16_t)pl.f[j];
        m.inv_bw[j] = 1.0 / pl.bw[j]; m.copies[j] = (uint32_t)copies;
        m.inside |= (uint32_t)inside << (4 * j);
    }
}
// Room for the states of a structure (see above), first guess; a structure that has more is met with four times as much.
uint32_t graph_room(const p2::Plan& pl) {
    static const uint32_t levels[5][P2_MAX_LEN + 1] = {{0, 96, 96, 96, 96, 96, 96, 96},
                                                       {0, 64, 64, 256, 640, 1024, 1280, 1536},
                                                       {0, 64, 128, 768, 3072, 10240, 20480, 32768},
                                                       {0, 64, 256, 1536, 12288, 57344, 57344, 57344},
                                                       {0, 64, 256, 3072, 32768, 32768, 32768, 32768}};
    const size_t n = pl.patterns.size();
    return levels[n <= 4 ? 0 : n <= 9 ? 1 : n <= 16 ? 2 : n <= 25 ? 3 : 4][pl.max_len];
}
// Queries and room of a graph of five or six levels of two devices up to which, and from which, its edges are costed from bandwidth
// rows.  Whole calls, us, from the sizes / from the rows: five levels, five instructions: one query 1 254 / 1 199, eight 1 284 / 1 242,
// sixteen 1 306 / 1 322, 64 1 525 / 1 738; six levels, four: one 853 / 825, eight 885 / 876, 32 948 / 993; five levels, four: one
// 378 / 371, eight 402 / 407; three: 108 / 116.
constexpr size_t kQueriesByRows = 8;
constexpr uint32_t kRoomByRows = 32768;
bool same_graph(const p2::Plan& a, const p2::Plan& b) {
    if (a.R != b.R || graph_rows(a) != graph_rows(b) || a.max_len != b.max_len || a.alphabet != b.alphabet || a.n_ops != b.n_ops ||
        a.patterns.size() != b.patterns.size())
        return false;
    for (int t = 0; t < a.n_ops; ++t)
        if (a.ops[t] != b.ops[t]) return false;
    for (size_t t = 0; t < a.patterns.size(); ++t)
        if (a.patterns[t].g != b.patterns[t].g || a.patterns[t].s != b.patterns[t].s || a.patterns[t].master != b.patterns[t].master)
            return false;
    return true;
}
// Lists of the state-graph engine beyond this size are left to the other engines (a batch that asks for every query to be
// evaluated by itself can have hundreds of large structures), and so are lists that would take more than half of the device
// memory that is free or held by them: their room is made for every state that there can be, the other engines' and the other
// queries' lists come later and are made for what there is.
constexpr size_t kGraphBytesMax = (size_t)32 << 30;
bool graph_has_room(size_t needed, size_t held, size_t free_bytes) { return needed <= (held + free_bytes) / 2; }

// What decides about validity is the same for both: group, chunks, patterns, alphabet and size limit.
bool same_structure(const p2::Plan& a, const p2::Plan& b) {
    if (a.R != b.R || a.k != b.k || a.max_len != b.max_len || a.alphabet != b.alphabet || a.n_ops != b.n_ops ||
        a.patterns.size() != b.patterns.size() || a.n_candidates != b.n_candidates)
        return false;
    for (int t = 0; t < a.n_ops; ++t)
        if (a.ops[t] != b.ops[t]) return false;
    for (size_t t = 0; t < a.patterns.size(); ++t)
        if (a.patterns[t].g != b.patterns[t].g || a.patterns[t].s != b.patterns[t].s || a.patterns[t].master != b.patterns[t].master ||
            a.patterns[t].n_groups != b.patterns[t].n_groups)
            return false;
    return true;
}

// Engine AUTO, several groups of more than 64 devices that differ in structure (`plans`, one of each): the walk takes all
// of them in a launch, the enumerations run four at a time.  Up to four enumerations cost no more than one, and each is
// faster than its walk; beyond, the walks of small groups with few candidates are done first.  Both sides as they
// were measured, in us (groups of 65 to 512 devices, one to three levels, 155 to 168 420 candidates, one to 32 of them):
// a walk 2.5 per device of the largest group, for a candidate's chain of steps, and 2.6 per 10^6 candidates x devices x
// devices (which a step visits, and whose masks are that long, or the chunk sets: the mean of the two counts stands for
// both); an enumeration 20 and 22 a level, of which the programs of a single level, one pattern, use two.  Thirty-two groups of 65 to 128 devices: 420 candidates 0.69 ms walked, 1.90
// enumerated; 2 070: 1.45 and 2.17; 8 420: 7.98 and 2.65.  Of 129 to 256: 155: 1.05 and 1.90; 780: 3.09 and 1.88.
bool walks_together(const std::vector<const p2::Plan*>& plans) {
    if (plans.size() <= (size_t)kFrontSlots) return false;
    double walk = 0.0, pruned = 100.0, devices = 0.0;
    for (const p2::Plan* pl : plans) {
        if (p2::compact_lanes(pl->R, pl->k) == 0) return false;
        const double wide = 0.5 * (pl->R + pl->k);
        devices = std::max(devices, wide);
        walk += 2.6e-6 * (double)pl->n_candidates * pl->R * wide;
        pruned += 20.0 + 22.0 * (pl->patterns.size() == 1 ? std::min(pl->max_len, 2) : pl->max_len);
    }
    return walk + 2.5 * devices < pruned;
}

// A call that enumerates some of its structures in any case (E: past the graphs' size limits, or asked for) may do better to
// enumerate the large groups beside them (L) than to build their graphs first, since the enumerations run kFrontSlots side by
// side and wait for the graphs.  What an enumeration takes by itself, us, within some 40 % for groups from 36 to 512 devices:
// its levels' waits and what its states add; a graph takes 0.55 of that; side by side the enumerations take the longest or
// 1 / 3.6 of their sum, the graphs 1 / 2.4.  Both ways measured: [3 4 6], seven instructions (E), and three groups of 72 to 128
// devices, four: 1 328 us enumerated, 1 660 with graphs; [3 4 6], four (E), and eight groups: 1 315 and 1 517; [100], three (E), and
// five groups: 765 and 938, and 13: 1 845 and 1 848; and [2 4 8 8], five: 2 864 and 1 760.
double enumerated_us(const p2::Plan& pl) {
    int levels = 0;
    for (int j = 0; j < pl.n; ++j) levels += pl.f[j] > 1 ? 1 : 0;
    return 115.0 * std::min(pl.max_len, 2 * levels) + 0.62e-3 * (double)graph_room(pl) * pl.R;
}
bool enumerates_beside(const std::vector<const p2::Plan*>& enumerated, const std::vector<const p2::Plan*>& graphs) {
    if (enumerated.empty() || graphs.empty()) return false;
    double longest[2] = {0.0, 0.0}, sum[2] = {0.0, 0.0};
    for (int which = 0; which < 2; ++which)
        for (const p2::Plan* pl : which == 0 ? enumerated : graphs) {
            const double t = enumerated_us(*pl);
            longest[which] = std::max(longest[which], t);
            sum[which] += t;
        }
    const double after = 0.55 * std::max(longest[1], sum[1] / 2.4) + std::max(longest[0], sum[0] / 3.6);
    return std::max({longest[0], longest[1], (sum[0] + sum[1]) / 3.6}) < 0.97 * after;
}

struct QueryRun {
    p2::Plan plan;
    int engine = P2_ENGINE_LITERAL;       // engine evaluating the bulk (LITERAL or COMPACT)
    bool frontier = false;                // enumeration by size with pruning instead of index by index
    bool flat_counts = false;             // ... in place of a walk (engine AUTO): the stats count what a walk executes
    bool regs = false;                    // per-candidate small-group engine (steps computed in registers)
    bool shared = false;                  // shared-prefix engine (the common instructions of a group applied once)
    bool auto_groups = false;             // its handed-over groups are picked up by the device-driven literal launch
    bool graph = false;                   // evaluated by the state-graph engine (AUTO), reported as the engine it stands in for
    bool graph_frontier = false;          // ... the frontier engine, whose stats count the prefixes' instructions
    bool graph_flat = false;              // ... (or, where it stands in for a walk, the walk's)
    bool graph_large = false;             // its states are worked on by the frontier's kernels
    int graph_id = -1, graph_pos = 0;     // ... its graph, and its place among the graph's queries
    bool wave_cost = false;               // valid programs costed by the wavefront-per-program kernel
    int enum_id = -1, share_pos = 0;      // frontier: its enumeration, and its place among the enumeration's queries
    int topk = 0;
    size_t off_query = 0, off_rowptr = 0, off_rowlevel = 0, off_entries = 0;
    int rows_at = 0;                      // its bandwidth rows' place among the distinct ones
    size_t off_goal = 0, off_rank = 0;    // hierarchies other than the collapsed one: goal masks, ranks of members
    int same_as = -1;                     // an earlier query of the batch with the same reduction group, chunks, patterns,
                                          // alphabet and size limit: its valid programs are this query's too
    uint32_t valid_cap = 0, rerun_cap = 0;
    size_t off_valid = 0, off_rerun = 0;  // element offsets into the valid / rerun buffers
    uint32_t n_valid = 0, n_rerun = 0, n_rerun_groups = 0;
    unsigned long long steps = 0, members = 0;
    unsigned long long evaluated = 0, evaluated_members = 0;   // instruction applications carried out where they differ from steps
    size_t out_first = 0;                 // first row of this query in the sorted/prog/cost buffers
};

constexpr int32_t kWithoutGraphs = 1;      // (internal) the call is to be repeated without the state graphs that `left` names now
// left: per query, whether a state graph was given up for it (the other engines evaluate it).
int32_t run_batch_on(const p2_query* queries, int32_t n_queries, const double* msg_bytes, int32_t n_msg,
                     p2_program* out_prog, double* out_cost, int64_t cap, int64_t* out_offset, p2_stats* stats, std::vector<char>& left) {
    using namespace p2;
    if (!queries || n_queries < 1 || !out_offset) return fail(P2_EINVAL, "null or empty query list");
    if (n_msg < 0 || (n_msg > 0 && !msg_bytes)) return fail(P2_EINVAL, "bad message size list");
    if (n_msg > kMaxMsg) return fail(P2_EUNSUPPORTED, "more than 64 message sizes");
    if (cap < 0 || (cap > 0 && (!out_prog || (n_msg > 0 && !out_cost)))) return fail(P2_EINVAL, "bad output buffers");
    for (int m = 0; m < n_msg; ++m)
        if (!(msg_bytes[m] >= 0.0)) return fail(P2_EINVAL, "message size must be >= 0");
    hipStream_t stream = (queries[0].opt) ? (hipStream_t)queries[0].opt->hip_stream : nullptr;
    Ctx& C = g_ctx;
    CallScope scope(stream);

    // ---- plan every query on the host
    const auto t_begin = std::chrono::steady_clock::now();
    std::vector<QueryRun> runs(n_queries);
    {
        // (the bandwidth rows of the cost model are built later, while the GPU evaluates; large batches: the queries' plans are
        //  independent, and host threads share them, one per 64: a plan takes 1 to 2 us, to start a thread some 30)
        std::vector<int32_t> plan_st((size_t)n_queries, P2_OK);
        std::vector<std::string> plan_err((size_t)n_queries);
        auto plan_one = [&](int i) {
            const p2_query& Q = queries[i];
            plan_st[i] = make_plan(Q.h, Q.axes, Q.n_axes, Q.placement, Q.reduce_axes, Q.n_reduce, Q.max_len, Q.opt, n_msg > 0,
                                   runs[i].plan, plan_err[i], false);
        };
        const unsigned hw = std::thread::hardware_concurrency();
        const int n_threads = (int)std::min<unsigned>({std::max(hw, 1u), 8u, (unsigned)n_queries / 64u + 1u});
        if (n_threads <= 1) {
            for (int i = 0; i < n_queries; ++i) plan_one(i);
        } else {
            std::atomic<int> next{0};
            auto work = [&]() { for (int i = next.fetch_add(1); i < n_queries; i = next.fetch_add(1)) plan_one(i); };
            std::vector<std::thread> pool;
            for (int t = 1; t < n_threads; ++t) pool.emplace_back(work);
            work();
            for (auto& th : pool) th.join();
        }
        for (int i = 0; i < n_queries; ++i)
            if (plan_st[i] != P2_OK) return fail(plan_st[i], "query " + std::to_string(i) + ": " + plan_err[i]);
    }
    bool share_validity = true;              // (see below)
    for (int i = 0; i < n_queries; ++i)
        if (queries[i].opt && (queries[i].opt->flags & P2_FLAG_EVALUATE_EVERY_QUERY)) share_validity = false;
    for (int i = 0; i < n_queries; ++i) {
        const p2_query& Q = queries[i];
        runs[i].topk = Q.opt ? Q.opt->topk : 0;
        if (runs[i].topk < 0) return fail(P2_EINVAL, "topk < 0");
        if (runs[i].topk > kMaxTopK) return fail(P2_EUNSUPPORTED, "topk > 1024");
        if (runs[i].topk > 0 && n_msg == 0) return fail(P2_EINVAL, "topk needs at least one message size");
        const int want = Q.opt ? Q.opt->engine : P2_ENGINE_AUTO;
        const Plan& pl = runs[i].plan;
        const bool lit_ok = true;        // the literal engine falls back to a global state buffer
        const bool cmp_ok = compact_lanes(pl.R, pl.k) != 0;
        if (pl.hierarchy != P2_HIERARCHY_COLLAPSED) {
            // ranks inside a group and per-device goals are known to the literal engine only
            if (want != P2_ENGINE_LITERAL && want != P2_ENGINE_AUTO)
                return fail(P2_EUNSUPPORTED, "query " + std::to_string(i) + ": this synthesis hierarchy runs on the literal engine only");
            if (pl.n_candidates > (1ull << 30))
                return fail(P2_EUNSUPPORTED, "query " + std::to_string(i) + ": more than 2^30 candidates under this synthesis hierarchy");
            runs[i].engine = P2_ENGINE_LITERAL;
        } else if (want == P2_ENGINE_LITERAL) {
            if (!lit_ok) return fail(P2_EUNSUPPORTED, "state too large for the literal engine");
            runs[i].engine = P2_ENGINE_LITERAL;
        } else if (want == P2_ENGINE_FRONTIER || (want == P2_ENGINE_AUTO && pl.n_candidates > kWalkMax)) {
            runs[i].engine = P2_ENGINE_COMPACT;      // its programs are costed like the compact engine's
            runs[i].frontier = true;
        } else if (want == P2_ENGINE_AUTO && pruned_is_faster(pl)) {
            runs[i].engine = P2_ENGINE_COMPACT;
            runs[i].frontier = runs[i].flat_counts = true;
        } else if (want == P2_ENGINE_COMPACT || want == P2_ENGINE_AUTO || want == P2_ENGINE_SMALL || want == P2_ENGINE_SHARED) {
            // power-of-two patterns: the shared-prefix engine holds up to 64 devices, the per-candidate
            // small-group engine up to 32 devices and 32 chunks
            bool shared_ok = pl.R <= 64, regs_ok = pl.R <= 32 && pl.k <= 32;
            for (const Pattern& p : pl.patterns) {
                shared_ok = shared_ok && reg_shape_of(p.g, p.s, p.master, 6) >= 0;
                regs_ok = regs_ok && reg_shape_of(p.g, p.s, p.master, 5) >= 0;
            }
            if (want == P2_ENGINE_SMALL && !regs_ok)
                return fail(P2_EUNSUPPORTED, "the small-group engine needs R <= 32, k <= 32 and power-of-two patterns");
            if (want == P2_ENGINE_SHARED && !shared_ok)
                return fail(P2_EUNSUPPORTED, "the shared-prefix engine needs R <= 64 and power-of-two patterns");
            runs[i].regs = want == P2_ENGINE_SMALL;
            runs[i].shared = shared_ok && (want == P2_ENGINE_SHARED || want == P2_ENGINE_AUTO);
            if (cmp_ok) runs[i].engine = P2_ENGINE_COMPACT;
            else if (lit_ok && want == P2_ENGINE_AUTO) runs[i].engine = P2_ENGINE_LITERAL;
            else return fail(P2_EUNSUPPORTED, "state too large for the available engines");
        } else return fail(P2_EINVAL, "unknown engine");
        if ((size_t)pl.patterns.size() > (size_t)kMaxPatterns) return fail(P2_EUNSUPPORTED, "more than 64 patterns");
        // valid programs of these queries are costed one per wavefront, lanes as devices
        runs[i].wave_cost = runs[i].engine == P2_ENGINE_COMPACT && pl.R <= 64;
        for (const Pattern& p : pl.patterns) runs[i].wave_cost = runs[i].wave_cost && reg_shape_of(p.g, p.s, p.master, 6) >= 0;
        if (!left[i] && want == P2_ENGINE_AUTO && graph_applies(pl)) {
            runs[i].graph = true;
            runs[i].graph_frontier = runs[i].frontier;
            runs[i].frontier = runs[i].flat_counts = false;
        }
    }
    // (once it is settled which groups are enumerated: see below)
    auto take_large_graphs = [&]() {
        for (int i = 0; i < n_queries; ++i) {
            QueryRun& r = runs[i];
            const int want = queries[i].opt ? queries[i].opt->engine : P2_ENGINE_AUTO;
            if (left[i] || want != P2_ENGINE_AUTO || !r.frontier || r.graph || !large_graph_applies(r.plan)) continue;
            r.graph = r.graph_large = true;
            r.graph_frontier = true; r.graph_flat = r.flat_counts;
            r.frontier = r.flat_counts = false;
        }
    };
    {
        std::vector<const Plan*> large;              // groups of more than 64 devices that AUTO would enumerate, one of each structure
        for (const QueryRun& r : runs) {
            if (!r.flat_counts || r.plan.R <= 64) continue;
            bool seen = false;
            for (size_t t = 0; t < large.size() && !seen && share_validity; ++t) seen = same_structure(*large[t], r.plan);
            if (!seen) large.push_back(&r.plan);
        }
        if (walks_together(large))
            for (QueryRun& r : runs)
                if (r.flat_counts && r.plan.R > 64) r.frontier = r.flat_counts = false;
    }

    take_large_graphs();
    {
        std::vector<const Plan*> enumerated, large;      // one of each structure
        for (const QueryRun& r : runs) {
            if (!(r.frontier || r.graph_large) || r.plan.n_candidates == 0) continue;
            std::vector<const Plan*>& list = r.frontier ? enumerated : large;
            bool seen = false;
            for (size_t t = 0; t < list.size() && !seen && share_validity; ++t) seen = same_structure(*list[t], r.plan);
            if (!seen) list.push_back(&r.plan);
        }
        if (enumerates_beside(enumerated, large))
            for (QueryRun& r : runs)
                if (r.graph_large) { r.frontier = true; r.flat_counts = r.graph_flat; r.graph = r.graph_large = r.graph_frontier = r.graph_flat = false; }
    }
    {
        bool walks = false, few = true;
        for (const QueryRun& r : runs) {
            walks |= !r.graph && !r.frontier && r.plan.n_candidates != 0;
            few &= !r.graph || (!r.graph_large && !r.graph_frontier && walks_beside(r.plan));
        }
        if (walks && few)
            for (QueryRun& r : runs) r.graph = false;
    }
    // queries of one reduction structure are answered from one graph, and so are the structures of one skeleton
    struct Graph { int leader = -1; std::vector<int32_t> members; uint32_t n_blocks = 0; bool small = false, large = false, skeleton = false, narrow = false;
                   int R = 0, rows = 0; size_t off_members = 0, off_query = 0, off_sizes = 0; };
    std::vector<Graph> graphs;
    bool any_whole = false;              // some skeleton is there in any case
    for (const QueryRun& r : runs) any_whole |= r.graph && whole_alphabet(r.plan) && has_skeleton(r.plan);
    auto fused_sums = [](const QueryRun& r) { return r.graph_frontier && !r.graph_flat ? 0u : 1u; };
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        if (!r.graph) continue;
        const Plan& pl = r.plan;
        // (else every query's graph is that of its own devices; single instructions of a narrowed alphabet are no reason for skeletons'
        //  launches beside those of small groups)
        const bool skeleton = share_validity && has_skeleton(pl) && (whole_alphabet(pl) || r.graph_large || any_whole);
        const int R = skeleton ? 1 << group_levels(pl) : pl.R;
        const bool split = pl.k % pl.R != 0;             // (how far rows can be cut is the group's own)
        auto same_group = [&](const QueryRun& o) {
            return o.graph_frontier == r.graph_frontier && o.graph_flat == r.graph_flat && o.graph_large == r.graph_large && same_graph(o.plan, pl);
        };
        for (size_t g = 0; g < graphs.size() && r.graph_id < 0 && share_validity; ++g) {
            const Graph& G = graphs[g];
            if (G.skeleton != skeleton || G.R != R) continue;
            const Plan& lead = runs[G.leader].plan;
            if (skeleton && !split ? lead.k % lead.R == 0 && lead.max_len == pl.max_len && lead.op_mask == pl.op_mask && lead.form_mask == pl.form_mask : same_group(runs[G.leader]))
                r.graph_id = (int)g;
        }
        if (r.graph_id < 0) {
            r.graph_id = (int)graphs.size();
            graphs.emplace_back();
            Graph& G = graphs.back();
            G.leader = i; G.skeleton = skeleton; G.narrow = skeleton && group_levels(pl) <= kNarrowLevels; G.large = r.graph_large && !skeleton; G.R = R; G.rows = skeleton ? R : graph_rows(pl);
        }
        Graph& G = graphs[r.graph_id];
        r.graph_pos = (int)G.members.size();
        G.members.push_back(i);
    }
    // (a skeleton of five or six levels whose queries' groups all have two devices a level is their own graph: where it has many edges
    //  and few queries these are costed from the bandwidth rows, a wavefront's lanes the devices, instead of a lane to a query)
    for (Graph& G : graphs) {
        bool own = G.skeleton && !G.narrow && G.members.size() <= kQueriesByRows && graph_room(runs[G.leader].plan) >= kRoomByRows;
        for (size_t t = 0; t < G.members.size() && own; ++t) own = runs[G.members[t]].plan.R == G.R;
        if (own) G.skeleton = false;
    }
    // those that p2_skeleton.hip works on come first, by levels; of one and two levels a block each, unless there are larger ones, whose
    // launches they ride along in
    uint32_t n_narrow[3] = {0, 0, 0};
    bool alone_skeletons = false;
    {
        auto class_of = [](const Graph& G) { return !G.narrow ? 3 : G.R <= 4 ? 0 : G.R == 8 ? 1 : 2; };
        std::vector<int> at(graphs.size());
        std::vector<Graph> in_order;
        in_order.reserve(graphs.size());
        for (int c = 0; c <= 3; ++c)
            for (size_t g = 0; g < graphs.size(); ++g)
                if (class_of(graphs[g]) == c) { at[g] = (int)in_order.size(); in_order.push_back(graphs[g]); if (c < 3) ++n_narrow[c]; }
        graphs.swap(in_order);
        for (QueryRun& r : runs) if (r.graph_id >= 0) r.graph_id = at[r.graph_id];
        alone_skeletons = n_narrow[0] > 0 && n_narrow[1] + n_narrow[2] == 0;
    }
    const uint32_t n_skeletons = n_narrow[0] + n_narrow[1] + n_narrow[2];
    size_t n_others = 0;                 // queries that other engines evaluate
    bool any_topk = false;
    for (const QueryRun& r : runs) { n_others += r.graph || r.plan.n_candidates == 0 ? 0 : 1; any_topk |= r.topk > 0; }
    // Every query answered from a graph: the whole call is one stream of kernels, tables and results travel by kernels that
    // read and write pinned host memory, and where no shortlist is asked for the rows go straight there.
    const bool only_graphs = n_others == 0 && !graphs.empty();
    // (rows are dealt out 256 to a block query by query: as many rows as there is room for, however the queries share them, take
    //  a block per 256 and at most one more per query)
    size_t rows_room = 0, emit_blocks = 0;
    if (only_graphs && !any_topk) {
        for (const QueryRun& r : runs)
            if (r.graph) { rows_room += most_valid(r.plan); ++emit_blocks; }
        rows_room = rows_at_once(rows_room, cap, n_msg);
        emit_blocks += rows_room / 256;
    }
    bool direct = rows_room > 0;
    const bool wanted_direct = direct;
    // Shortlists of every query, answered from graphs: the rows and the selections are queued for as many programs as there can be,
    // each takes their number from the graph's counts, and the rows that are picked are written to the host by the selections:
    // one wait instead of two, and four launches fewer ([3 4 6], ten of 571: 147 us, and 118 so).
    size_t shortlist_rows = 0, narrowed_rows = 0, shortlist_out = 0;
    bool shortlists = only_graphs && n_msg > 0;
    int shortlist_k = 0;
    size_t shortlist_most = 0;
    for (const QueryRun& r : runs) {
        if (!r.graph) continue;
        const size_t most = most_valid(r.plan);
        shortlists = shortlists && r.topk > 0 && most <= kTopkJobMax;
        shortlist_rows += most;
        narrowed_rows += whole_alphabet(r.plan) ? 0 : most;
        shortlist_out += shortlist_rows_of(r.plan, r.topk, n_msg);
        shortlist_k = std::max(shortlist_k, r.topk);
        shortlist_most = std::max(shortlist_most, most);
    }
    // (the rows that are picked go to pinned memory, which is bounded as for lists)
    const size_t row_bytes = sizeof(p2_program) + 8 + 8 * (size_t)std::max(n_msg, 1);
    shortlists = shortlists && cap > 0 && shortlist_out <= (size_t)cap && rows_at_once(shortlist_out, cap, n_msg) > 0 &&
                 shortlist_rows <= kShortlistBytes / row_bytes && narrowed_rows <= kNarrowedShortlistBytes / row_bytes;
    // (the shortlist of what has one program at most is its list, unless a cost may be no number, which a list takes and a shortlist does
    //  not: less to select and to gather.  Walked searches ask for as many of these as for others: on 3 x 6, 215 us a call with, 195 without)
    const bool costs_are_numbers = n_msg == 1 && msg_bytes[0] > 0.0 && std::isfinite(msg_bytes[0]);
    for (QueryRun& r : runs)
        if (!shortlists && costs_are_numbers && r.topk > 0 && r.plan.hierarchy == P2_HIERARCHY_COLLAPSED && most_valid(r.plan) == 1) r.topk = 0;
    // Of a graph with several queries the rows are written once, and their costs worked out for all of them side by side (k_graph_sums).
    auto shares_rows = [&](const Graph& G) {
        return G.narrow && G.members.size() >= kSharedQueries && runs[G.leader].plan.n_ops == 5;
    };
    size_t off_jobs = 0, off_rows = 0, off_sums = 0, off_columns = 0;
    size_t n_jobs = 0, n_segs = 0, n_sums = 0, n_columns = 0;
    size_t shared_rows = 0, listed_rows = 0;             // rows of graphs that share them; those and the other queries'
    size_t shared_costs = 0;
    unsigned shortlist_blocks = 0, sums_blocks = 0, most_columns = 0, sum_rows = 64;
    auto add_rows = [&](const Plan& pl) { ++n_segs; listed_rows += most_valid(pl); shortlist_blocks += (unsigned)((most_valid(pl) + 255) / 256); };
    if (shortlists) {
        for (const Graph& G : graphs) {
            n_jobs += (size_t)n_msg * G.members.size();
            if (!shares_rows(G)) continue;
            ++n_sums; n_columns += G.members.size();
            add_rows(runs[G.leader].plan);
            shared_costs += most_valid(runs[G.leader].plan) * G.members.size();
            most_columns = std::max(most_columns, (unsigned)G.members.size());
        }
        shared_rows = listed_rows;
        // (a block sets up tables of its queries first: 64 rows each while the chip is not full, and 512 otherwise)
        if (shared_rows / 64 * ((most_columns + kSumMembers - 1) / kSumMembers) > 1024) sum_rows = 512;
        for (const Graph& G : graphs) if (shares_rows(G)) sums_blocks += (unsigned)((most_valid(runs[G.leader].plan) + sum_rows - 1) / sum_rows);
        for (const QueryRun& r : runs) if (r.graph && !shares_rows(graphs[r.graph_id])) add_rows(r.plan);
    }
    auto leave_graph = [&](const Graph& G) { for (int32_t i : G.members) left[i] = 1; };
    // Validity depends on the reduction group, the chunks, the patterns and the alphabet only (not on the
    // links, nor on where the placement puts the group in the system): a query that equals an earlier one of
    // the batch in these is not evaluated again; it takes over the list of valid programs and the counts, and
    // only its costs are worked out, from its own bandwidth rows.  (The frontier engine does the same further
    // down.)  P2_FLAG_EVALUATE_EVERY_QUERY in any query's options switches this off for the batch.
    {
        for (int i = 0; i < n_queries && share_validity; ++i) {
            QueryRun& r = runs[i];
            const Plan& pl = r.plan;
            if (r.graph || r.frontier || pl.hierarchy != P2_HIERARCHY_COLLAPSED || pl.n_candidates == 0) continue;
            for (int j = 0; j < i && r.same_as < 0; ++j) {
                const QueryRun& c = runs[j];
                if (c.same_as < 0 && !c.graph && !c.frontier && c.plan.hierarchy == P2_HIERARCHY_COLLAPSED && c.engine == r.engine && c.shared == r.shared &&
                    c.regs == r.regs && same_structure(c.plan, pl))
                    r.same_as = j;
            }
        }
    }
    g_prof.last.host_plan_ms = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    // ---- lay out the table blob: queries, message sizes, bandwidth rows
    size_t off = 0;
    for (auto& r : runs) { r.off_query = off; off += sizeof(DevQuery); }      // one contiguous DevQuery array
    off = align_up(off, 256);
    // compact-engine queries are launched together, one launch per (chunk words, mask words) class
    struct Launch {
        int kind;                                   // 0 compact engine (state in LDS), 1 per-candidate small-group, 2 shared-prefix
        int kw, mw, max_R, max_k; std::vector<DevSegment> segs; unsigned blocks; size_t off_segs;
        std::vector<DevShare> shares; unsigned grid = 0; size_t off_shares = 0;     // shared-prefix kernel only
    };
    std::vector<Launch> launches;
    auto word_class = [](int bits) { int w = (bits + 31) / 32; return w <= 1 ? 1 : w <= 2 ? 2 : w <= 4 ? 4 : w <= 8 ? 8 : 16; };
    for (int i = 0; i < n_queries; ++i) {
        if (runs[i].engine != P2_ENGINE_COMPACT || runs[i].graph || runs[i].frontier || runs[i].same_as >= 0 || runs[i].plan.n_candidates == 0) continue;
        const Plan& pl = runs[i].plan;
        const int kind = runs[i].shared ? 2 : runs[i].regs ? 1 : 0;
        const int kw = kind == 1 ? 1 : word_class(pl.k), mw = kind == 1 ? 1 : word_class(pl.R);
        Launch* L = nullptr;
        for (auto& c : launches) if (c.kind == kind && c.kw == kw && c.mw == mw) L = &c;
        if (!L) { launches.push_back(Launch{kind, kw, mw, 0, 0, {}, 0u, 0, {}, 0u, 0}); L = &launches.back(); }
        L->max_R = std::max(L->max_R, pl.R);
        L->max_k = std::max(L->max_k, pl.k);
    }
    // stems (prefixes of len-2 instructions) of all shared-prefix queries of the batch
    unsigned long long shared_stems = 0;
    for (int i = 0; i < n_queries; ++i) {
        const Plan& pl = runs[i].plan;
        if (!runs[i].shared || runs[i].graph || runs[i].frontier || runs[i].same_as >= 0 || pl.n_candidates == 0 || pl.alphabet == 0) continue;
        for (int len = 2; len <= pl.max_len; ++len)
            shared_stems += (pl.base[len + 1] - pl.base[len]) / ((unsigned long long)pl.alphabet * (unsigned long long)pl.alphabet);
    }
    const unsigned long long shared_cut = shared_stems >= (1ull << 17) ? 1 : shared_stems >= (1ull << 15) ? 2 : 4;
    for (auto& L : launches) {
        const int lanes = L.kind != 0 ? 64 : compact_lanes(L.max_R, L.max_k);
        if (lanes == 0) return fail(P2_EUNSUPPORTED, "state too large for the compact engine");
        unsigned long long blocks = 0;
        for (int i = 0; i < n_queries; ++i) {
            const Plan& pl = runs[i].plan;
            if (runs[i].engine != P2_ENGINE_COMPACT || runs[i].graph || runs[i].frontier || runs[i].same_as >= 0 || pl.n_candidates == 0) continue;
            const int kind = runs[i].shared ? 2 : runs[i].regs ? 1 : 0;
            if (kind != L.kind || (kind == 1 ? 1 : word_class(pl.k)) != L.kw || (kind == 1 ? 1 : word_class(pl.R)) != L.mw) continue;
            for (int len = 1; len <= pl.max_len; ++len) {
                const unsigned long long count = pl.base[len + 1] - pl.base[len];
                DevSegment sg;
                sg.first_block = (uint32_t)blocks; sg.query = i; sg.len = len;
                sg.first_index = pl.base[len]; sg.count = count;
                if (L.kind == 2) {
                    // shared-prefix kernel: an item is a run of groups under one stem (the first len-2
                    // instructions).  With few stems a stem is cut into four items, which balances the load
                    // of the fixed grid; with many stems a whole stem is one item, so its state is worked out once
                    const unsigned long long I = (unsigned long long)pl.alphabet;
                    const unsigned long long per_item = len >= 2 ? (I + shared_cut - 1) / shared_cut : 1;
                    sg.iters = (int)per_item;
                    blocks += len >= 2 ? (count / (I * I)) * shared_cut : 1;     // (items past a short stem's groups are empty)
                } else {
                    const unsigned long long chunks = (count + lanes - 1) / lanes;
                    unsigned long long iters = (chunks + 4095) / 4096;
                    iters = std::min<unsigned long long>(std::max<unsigned long long>(iters, 1), 64);
                    sg.iters = (int)iters;
                    blocks += (chunks + iters - 1) / iters;
                }
                L.segs.push_back(sg);
                if (blocks > 0x7fffffffull) return fail(P2_EUNSUPPORTED, "too many candidates for one launch");
            }
        }
        L.blocks = (unsigned)blocks;
        L.off_segs = off;
        off += align_up(sizeof(DevSegment) * L.segs.size(), 256);
        if (L.kind == 2) {
            // divide a grid of about 8192 blocks (32 wavefronts per compute unit) among the queries by their items
            const unsigned long long target = 8192;
            for (size_t a = 0; a < L.segs.size();) {
                size_t b = a;
                while (b < L.segs.size() && L.segs[b].query == L.segs[a].query) ++b;
                DevShare shq;
                shq.first_item = L.segs[a].first_block;
                shq.n_items = (b < L.segs.size() ? L.segs[b].first_block : L.blocks) - shq.first_item;
                unsigned long long nb = (target * shq.n_items + L.blocks / 2) / std::max(1u, L.blocks);
                nb = std::min<unsigned long long>(std::max<unsigned long long>(nb, 1), std::max(1u, shq.n_items));
                shq.first_block = L.grid; shq.n_blocks = (uint32_t)nb;
                shq.query = L.segs[a].query; shq.first_seg = (int32_t)a; shq.n_segs = (int32_t)(b - a);
                shq.cut_log = shared_cut == 4 ? 2 : shared_cut == 2 ? 1 : 0;
                L.grid += (unsigned)nb;
                L.shares.push_back(shq);
                a = b;
            }
            L.off_shares = off;
            off += align_up(sizeof(DevShare) * L.shares.size(), 256);
        }
    }
    // Groups that the shared-prefix engine hands to the literal engine are found on the device, so that kernel
    // is queued right behind the evaluation: one launch per mask width, each with the list of its queries.
    struct AutoGroups { int cls = 0, max_R = 0, max_k = 0, class_cap = 64; std::vector<int32_t> qlist; size_t off = 0; };
    std::vector<AutoGroups> autos;
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        if (!r.shared || r.graph || r.frontier || r.same_as >= 0 || r.plan.n_candidates == 0) continue;
        const int mw = r.plan.R <= 32 ? 1 : 2;
        const int cls = mw;
        AutoGroups* A = nullptr;
        for (auto& a : autos) if (a.cls == cls) A = &a;
        if (!A) { autos.emplace_back(); A = &autos.back(); A->cls = cls; }
        A->max_R = std::max(A->max_R, r.plan.R); A->max_k = std::max(A->max_k, r.plan.k);
        A->class_cap = std::min(A->class_cap, r.plan.max_row_classes);
        A->qlist.push_back(i);
        r.auto_groups = true;
    }
    for (auto& A : autos) { A.off = off; off += align_up(sizeof(int32_t) * A.qlist.size(), 256); }
    for (auto& r : runs) {
        if (r.plan.hierarchy == P2_HIERARCHY_COLLAPSED) continue;
        r.off_goal = off;
        off += align_up(sizeof(uint32_t) * (r.plan.goal.empty() ? 0 : (size_t)r.plan.R * literal_mask_words(r.plan.R)), 256);
        r.off_rank = off;
        size_t n_rank = 0;
        for (const Pattern& p : r.plan.patterns) n_rank += p.rank.size();
        off += align_up(sizeof(int32_t) * n_rank, 256);
    }
    // the state graphs: their descriptions, which blocks work on which, and the queries that share each
    size_t off_gasked = 0, off_graphs = 0, off_glevel = 0, off_gsteps = 0, off_gcosts = 0, off_gsmall = 0, off_glarge = 0;
    std::vector<GraphBlock> glevel, gsteps, gcosts;
    unsigned most_members = 0;
    std::vector<uint32_t> gsmall, glarge;
    int graph_levels = 0, narrow_levels = 0;
    if (!graphs.empty()) {
        uint32_t n_by_size[3] = {0, 0, 0};                // up to two levels, three, more
        auto size_of = [&](const Graph& G) { const size_t n = runs[G.leader].plan.patterns.size(); return n <= 4 ? 0 : n <= 9 ? 1 : 2; };
        for (Graph& G : graphs) if (!G.large) ++n_by_size[size_of(G)];
        const bool alone = n_by_size[1] + n_by_size[2] == 0;      // (beside larger ones the small ones ride along in their launches)
        for (size_t g = 0; g < graphs.size(); ++g) {
            Graph& G = graphs[g];
            const int sz = size_of(G);
            // (blocks per level: three levels have some 280 states in the largest, four some 9 000; a launch of some 2 000
            //  blocks fills the chip)
            G.small = sz == 0 && alone && graph_alone_holds(graph_room(runs[G.leader].plan));
            const uint32_t share = 2048u / std::max(1u, n_by_size[sz]);
            G.n_blocks = G.small ? 1u : sz == 0 ? 12u : sz == 1 ? std::min(std::max(share, 16u), 160u) : std::min(std::max(share, 64u), 768u);
            if (G.narrow) {
                narrow_levels = std::max(narrow_levels, runs[G.leader].plan.max_len);
            } else if (G.large) {
                glarge.push_back((uint32_t)g);
                G.off_query = off;
                off += align_up(sizeof(DevQuery), 256);
            } else if (G.small) gsmall.push_back((uint32_t)g);
            else {
                glarge.push_back((uint32_t)g);
                graph_levels = std::max(graph_levels, runs[G.leader].plan.max_len);
                for (uint32_t b = 0; b < G.n_blocks; ++b) glevel.push_back(GraphBlock{(uint32_t)g, b, G.n_blocks, 0u});
            }
            // (four edges a block at a time; two levels have some 70 edges on the way to a goal, three 900, four 6 300)
            const uint32_t nb = G.large ? 512u : sz == 0 ? 18u : std::min(std::max(share, 16u), sz == 1 ? 160u : 512u);
            const uint32_t nc = 1600u * std::min(((uint32_t)G.members.size() + 63u) / 64u, 4u);
            if (G.narrow) most_members = std::max(most_members, (unsigned)G.members.size());
            else if (G.skeleton) for (uint32_t b = 0; n_msg > 0 && b < nc; ++b) gcosts.push_back(GraphBlock{(uint32_t)g, b, nc, 0u});
            else for (uint32_t b = 0; n_msg > 0 && b < nb; ++b) gsteps.push_back(GraphBlock{(uint32_t)g, b, nb, 0u});
            G.off_members = off;
            off += align_up(sizeof(int32_t) * G.members.size(), 64);
            if (G.skeleton) {
                off = align_up(off, 128);
                G.off_sizes = off;
                off += sizeof(DevMember) * G.members.size();
            }
        }
        off = align_up(off, 256);
        off_gasked = off; off += align_up(sizeof(GraphQuery) * (size_t)n_queries, 256);
        off_graphs = off; off += align_up(sizeof(DevGraph) * graphs.size(), 256);
        off_glevel = off; off += align_up(sizeof(GraphBlock) * glevel.size(), 256);
        off_gsteps = off; off += align_up(sizeof(GraphBlock) * gsteps.size(), 256);
        off_gcosts = off; off += align_up(sizeof(GraphBlock) * gcosts.size(), 256);
        off_gsmall = off; off += align_up(sizeof(uint32_t) * gsmall.size(), 256);
        off_glarge = off; off += align_up(sizeof(uint32_t) * glarge.size(), 256);
    }
    if (shortlists) {
        off_jobs = off; off += align_up(sizeof(DevTopkJob) * n_jobs, 256);
        off_rows = off; off += align_up(sizeof(GraphRows) * n_segs, 256);
        off_sums = off; off += align_up(sizeof(GraphSums) * n_sums, 256);
        off_columns = off; off += align_up(sizeof(GraphColumn) * n_columns, 256);
    }
    const size_t off_msg = off;
    off += align_up(sizeof(double) * (size_t)std::max(n_msg, 1), 256);
    const size_t blob_bytes = off;
    // The bandwidth rows (cost model) live in buffers of their own: the rows, and per distinct set of rows a header
    // (DevRows) that the query descriptors point at.  They are built on the host after the evaluation kernels have been
    // queued and uploaded on a second stream, so both overlap with the evaluation; the call's stream waits
    // for the upload before its first cost kernel.  Queries whose rows are the same share them, and those of the collapsed
    // hierarchy follow from the factors; worked out for every query, from the devices under every unit, the rows were most of
    // a batch's host time (140 queries of [4 8 8]: 1 000 us of a call's 1 590 with eight threads, and 540 for the call so;
    // 512 queries of [2 4 8 8], 96 distinct sets: 5 600 us, and 400 now without a thread).
    // (The rows of the other hierarchies are every query's own and built from its devices; host threads share them, one per
    //  128, as a set takes 1 to 3 us and a thread some 30, twice: 2 000 queries of eight devices take 17.5 ms so, and 20.3 in one
    //  thread; with eight threads from 32 sets on, 48 queries took 635 us, and 510 in one thread.)
    std::vector<int32_t> row_sets;                       // a query of each
    size_t n_built_sets = 0;                             // ... of another hierarchy
    for (int i = 0; i < n_queries; ++i) {
        size_t t = 0;
        if (runs[i].graph && graphs[runs[i].graph_id].skeleton) continue;            // (costed from its sizes)
        if (runs[i].plan.hierarchy != P2_HIERARCHY_COLLAPSED) { t = row_sets.size(); ++n_built_sets; }
        while (t < row_sets.size() && !same_cost_rows(runs[row_sets[t]].plan, runs[i].plan)) ++t;
        if (t == row_sets.size()) row_sets.push_back(i);
        runs[i].rows_at = (int)t;
    }
    bool rows_ready = false;
    P2_HIP(C.rows_hdr.ensure(sizeof(DevRows) * row_sets.size()));
    P2_HIP(C.h_rows_hdr.ensure(sizeof(DevRows) * row_sets.size()));
    if (!C.copy_stream) {
        P2_HIP(hipStreamCreateWithFlags(&C.copy_stream, hipStreamNonBlocking));
        P2_HIP(hipEventCreateWithFlags(&C.copy_done, hipEventDisableTiming));
        P2_HIP(hipEventCreateWithFlags(&C.front_go, hipEventDisableTiming));
    }
    size_t n_large = 0;
    for (const Graph& G : graphs) n_large += G.large ? 1 : 0;
    int large_slots = 1;
    if (n_large > 1) {
        bool one_at_a_time = false;
        for (int i = 0; i < n_queries; ++i)
            one_at_a_time |= queries[i].opt && (queries[i].opt->flags & P2_FLAG_ONE_ENUMERATION_AT_A_TIME) != 0u;
        if (!one_at_a_time) large_slots = (int)std::min<size_t>(kFrontSlots, n_large);
        if (large_slots > 1) {
            if (!C.slots[1].stream) {                    // (first time: the streams are chosen by timing, on a quiet device)
                P2_HIP(hipStreamSynchronize(stream));
                P2_HIP(hipStreamSynchronize(C.copy_stream));
            }
            P2_HIP(C.open_slot_streams(large_slots));
        }
    }
    auto build_and_upload_rows = [&]() -> int32_t {
        if (rows_ready || row_sets.empty()) return P2_OK;
        size_t bytes = 0;
        const unsigned hw = std::thread::hardware_concurrency();
        const int n_threads = (int)std::min<unsigned>({std::max(hw, 1u), 16u, (unsigned)n_built_sets / 128u + 1u});
        auto for_every_set = [&](const auto& f) {
            if (n_threads <= 1) { for (int32_t i : row_sets) f(i); return; }
            std::atomic<size_t> next{0};
            auto work = [&]() { for (size_t t = next.fetch_add(1); t < row_sets.size(); t = next.fetch_add(1)) f(row_sets[t]); };
            std::vector<std::thread> pool;
            for (int t = 1; t < n_threads; ++t) pool.emplace_back(work);
            work();
            for (auto& th : pool) th.join();
        };
        if (n_msg > 0) for_every_set([&](int32_t i) { build_cost_tables(runs[i].plan); });      // without message sizes the tables stay empty
        for (int32_t i : row_sets) {
            QueryRun& r = runs[i];
            size_t n_rows = 0, n_ent = 0;
            for (const Pattern& p : r.plan.patterns) { n_rows += p.row_level.size(); n_ent += p.entries.size(); }
            r.off_rowptr = bytes; bytes += align_up(sizeof(int32_t) * (n_rows + 1), 16);
            r.off_rowlevel = bytes; bytes += align_up(sizeof(int32_t) * std::max<size_t>(n_rows, 1), 16);
            r.off_entries = bytes; bytes += align_up(sizeof(uint32_t) * std::max<size_t>(n_ent, 1), 256);
        }
        P2_HIP(C.rows.ensure(bytes));
        P2_HIP(C.h_rows.ensure(bytes));
        char* hr = static_cast<char*>(C.h_rows.p);
        char* dr = static_cast<char*>(C.rows.p);
        DevRows* hdr = static_cast<DevRows*>(C.h_rows_hdr.p);
        for_every_set([&](int32_t i) {
            const QueryRun& r = runs[i];
            const Plan& pl = r.plan;
            int32_t* rp = reinterpret_cast<int32_t*>(hr + r.off_rowptr);
            int32_t* rl = reinterpret_cast<int32_t*>(hr + r.off_rowlevel);
            uint32_t* en = reinterpret_cast<uint32_t*>(hr + r.off_entries);
            DevRows& H = hdr[r.rows_at];
            std::memset(&H, 0, sizeof H);
            int row = 0, ent = 0;
            rp[0] = 0;
            for (size_t pi = 0; pi < pl.patterns.size(); ++pi) {
                const Pattern& p = pl.patterns[pi];
                H.pat_begin[pi] = row;
                for (size_t t = 0; t < p.row_level.size(); ++t) {
                    uint32_t sum = 0;
                    for (int e = p.row_ptr[t]; e < p.row_ptr[t + 1]; ++e) { en[ent++] = p.entries[e]; sum += entry_cnt(p.entries[e]); }
                    rl[row] = p.row_level[t];
                    rp[++row] = ent;
                    H.level_max[pi][p.row_level[t]] = std::max(H.level_max[pi][p.row_level[t]], sum);
                }
            }
            for (size_t pi = pl.patterns.size(); pi <= (size_t)kMaxPatterns; ++pi) H.pat_begin[pi] = row;
            H.row_ptr = reinterpret_cast<const int32_t*>(dr + r.off_rowptr);
            H.row_level = reinterpret_cast<const int32_t*>(dr + r.off_rowlevel);
            H.entries = reinterpret_cast<const uint32_t*>(dr + r.off_entries);
        });
        rows_ready = true;
        if (only_graphs && large_slots == 1) {           // (else the call's stream has the slots to wait for)
            const CopyPart up[2] = {{C.rows.p, C.h_rows.p, bytes}, {C.rows_hdr.p, C.h_rows_hdr.p, sizeof(DevRows) * row_sets.size()}};
            P2_HIP(launch_copies(up, 2, stream));
            return P2_OK;
        }
        P2_HIP(hipMemcpyAsync(C.rows.p, C.h_rows.p, bytes, hipMemcpyHostToDevice, C.copy_stream));
        P2_HIP(hipMemcpyAsync(C.rows_hdr.p, C.h_rows_hdr.p, sizeof(DevRows) * row_sets.size(), hipMemcpyHostToDevice, C.copy_stream));
        P2_HIP(hipEventRecord(C.copy_done, C.copy_stream));
        P2_HIP(hipStreamWaitEvent(stream, C.copy_done, 0));
        return P2_OK;
    };
    P2_HIP(C.blob.ensure(blob_bytes));
    P2_HIP(C.h_blob.ensure(blob_bytes));
    P2_HIP(C.counters.ensure(sizeof(DevCounters) * (size_t)n_queries));
    P2_HIP(C.h_counters.ensure(sizeof(DevCounters) * (size_t)n_queries));

    // valid / rerun list capacities (grown and retried if a query overflows them)
    auto layout_lists = [&]() {
        size_t v = 0, rr = 0;
        for (auto& r : runs) { r.off_valid = v; v += r.valid_cap; r.off_rerun = rr; rr += r.rerun_cap; }
        return std::make_pair(v, rr);
    };
    for (auto& r : runs) {
        const unsigned long long N = r.plan.n_candidates;
        r.valid_cap = (r.graph || r.frontier || r.same_as >= 0) ? 0u : (uint32_t)std::min<unsigned long long>(N, 1u << 15);
        r.rerun_cap = (r.engine == P2_ENGINE_COMPACT && !r.graph && !r.frontier && r.same_as < 0) ? (uint32_t)std::min<unsigned long long>(N, 1u << 10) : 0u;
    }

    // global state buffer for literal evaluations whose state does not fit in LDS
    auto lit_scratch = [&](const Plan& pl, void** out) -> hipError_t {
        *out = nullptr;
        if (literal_lds_bytes(pl.R, pl.k) != 0) return hipSuccess;
        unsigned nb = 0;
        hipError_t e = C.lit_scratch.ensure(literal_scratch_bytes(pl.R, pl.k, &nb));
        *out = C.lit_scratch.p;
        return e;
    };
    // Segment tables for the kernels that serve many queries per launch.  Tables of one phase are
    // packed into C.post and uploaded with one copy; `PostLaunch` remembers where each one starts.
    struct PostLaunch { int cls = 0; int max_R = 0, max_k = 0; size_t lit_lds = 0; std::vector<DevPostSeg> segs; unsigned blocks = 0; size_t off = 0; };
    auto add_seg = [](std::vector<PostLaunch>& v, int cls, const Plan& pl, int query, uint32_t count, uint32_t per_block,
                      size_t in_off, size_t out_off) {
        PostLaunch* L = nullptr;
        for (auto& c : v) if (c.cls == cls) L = &c;
        if (!L) { v.emplace_back(); L = &v.back(); L->cls = cls; }
        L->max_R = std::max(L->max_R, pl.R); L->max_k = std::max(L->max_k, pl.k);
        L->lit_lds = std::max(L->lit_lds, literal_lds_bytes(pl.R, pl.k));     // what the literal kernels would need
        DevPostSeg sg;
        sg.first_block = L->blocks; sg.query = query; sg.count = count; sg.per_block = per_block;
        sg.in_off = in_off; sg.out_off = out_off;
        L->segs.push_back(sg);
        L->blocks += (count + per_block - 1) / per_block;
    };
    auto upload_segs = [&](std::vector<std::vector<PostLaunch>*> groups) -> hipError_t {
        size_t bytes = 0;
        for (auto* g : groups) for (auto& L : *g) { L.off = bytes; bytes += align_up(sizeof(DevPostSeg) * L.segs.size(), 256); }
        if (bytes == 0) return hipSuccess;
        hipError_t e = C.post.ensure(bytes);
        if (e != hipSuccess) return e;
        e = C.h_post.ensure(bytes);
        if (e != hipSuccess) return e;
        for (auto* g : groups) for (auto& L : *g)
            std::memcpy(static_cast<char*>(C.h_post.p) + L.off, L.segs.data(), sizeof(DevPostSeg) * L.segs.size());
        return hipMemcpyAsync(C.post.p, C.h_post.p, bytes, hipMemcpyHostToDevice, stream);
    };
    auto segs_of = [&](const PostLaunch& L) { return reinterpret_cast<const DevPostSeg*>(static_cast<char*>(C.post.p) + L.off); };
    auto mask_class = [](int R) { return R <= 32 ? 1 : R <= 64 ? 2 : R <= 128 ? 4 : R <= 256 ? 8 : 16; };
    char* hb = static_cast<char*>(C.h_blob.p);
    char* db = static_cast<char*>(C.blob.p);
    // what the frontier's kernels build a large group's graph in
    struct LargeAt {
        FrontCounters* ctr; FrontMarks* marks; unsigned long long* table[2]; uint32_t table_size[2];
        uint32_t* states[2]; unsigned long long* hash[2]; uint32_t* rep[2]; uint32_t* pos[2]; uint32_t* reps[2]; uint32_t* walk[2];
        uint8_t* codes[2]; unsigned long long* row_counts[2]; uint8_t* unknown[2];
        FrontSurvivor* edges; FrontEntry* literal; uint32_t* literal_parent; uint32_t* rest; void* literal_scratch;
        uint32_t cap[2], cap_literal;
    };
    std::vector<LargeAt> large_at;
    // the lists of the state graphs, one graph after the other (grown and repeated like the others)
    uint32_t graph_scale = 1;
    size_t graph_zero = 0;
    const size_t graph_nan = sizeof(GraphCounters) * graphs.size();      // behind the counters: a word per query, set where a cost is NaN
    const size_t graph_back = graph_nan + sizeof(uint32_t) * (size_t)n_queries;
    auto layout_graphs = [&](DevGraph* out) -> int32_t {
        const size_t n_graphs = graphs.size();
        size_t zero = align_up(graph_nan + sizeof(uint32_t) * (size_t)n_queries, 256), mem = 0;
        auto take = [](size_t& at, size_t bytes) { const size_t here = at; at += align_up(bytes, 256); return here; };
        struct Place { size_t table, table_node, planes, state, path, edge_path, narrow, node_edges, nearest, count2, found, links, use_id, first, use_ends, edges, edge_state, best; };
        std::vector<Place> places(n_graphs);
        large_at.assign(n_graphs, LargeAt{});
        size_t states_bytes = 0;
        for (size_t g = 0; g < n_graphs; ++g) {
            const Graph& G = graphs[g];
            const Plan& pl = runs[G.leader].plan;
            DevGraph& D = out[g];
            std::memset(&D, 0, sizeof D);
            D.query = (uint32_t)G.leader;
            D.R = G.R; D.rows_kept = G.rows;
            D.n_pat = (int)pl.patterns.size(); D.n_ops = pl.n_ops; D.alphabet = pl.alphabet; D.max_len = pl.max_len;
            D.digit_words = (pl.alphabet + 63) / 64;
            D.n_members = (int)G.members.size();
            for (int o = 0; o < pl.n_ops; ++o) { D.op_mask |= 1u << pl.ops[o]; D.op_ranks |= (uint32_t)o << (4 * pl.ops[o]); }
            for (int32_t m : G.members) D.split_check |= (G.skeleton ? runs[m].plan.k % runs[m].plan.R != 0 : runs[m].plan.k != D.rows_kept) ? 1u : 0u;
            D.cap_nodes = graph_room(pl) * graph_scale;
            // (some twice as many children as nodes; a wavefront may leave the rest of what it reserved at every level)
            D.cap_planes = D.cap_nodes * 2 + graph_planes_left(G.n_blocks, pl.max_len) + 256u;
            D.cap_found = D.cap_nodes * 3;
            D.cap_edges = D.cap_nodes + 256;
            uint32_t slots = 64;
            while (slots < 2 * D.cap_nodes) slots *= 2;
            D.table_mask = slots - 1;
            if (G.large) {
                D.cap_planes = 0; D.table_mask = 0;
                LargeAt& L = large_at[g];
                L.cap[0] = D.cap_nodes * 2 + 64; L.cap[1] = D.cap_nodes / 2 + 64; L.cap_literal = D.cap_nodes / 8 + 1024;
                const int kk = D.rows_kept;
                const size_t plane = frontier_state_words(pl.R, kk) * 4, codes = front_code_stride(pl.alphabet);
                D.wq = (int)(plane / 16 / (size_t)pl.R); D.qk = (literal_mask_words(kk) + 3) / 4;
                // (offsets first, pointers once the buffers are there)
                auto at = [](size_t v) { return reinterpret_cast<char*>(v); };
                L.ctr = (FrontCounters*)at(take(zero, sizeof(FrontCounters)));
                L.marks = (FrontMarks*)at(take(mem, sizeof(FrontMarks)));
                for (int li = 0; li < 2; ++li) {
                    L.table_size[li] = 1024;
                    while (L.table_size[li] < 2 * L.cap[li]) L.table_size[li] *= 2;
                    L.table[li] = (unsigned long long*)at(take(zero, sizeof(unsigned long long) * L.table_size[li]));
                    L.hash[li] = (unsigned long long*)at(take(mem, sizeof(unsigned long long) * L.cap[li]));
                    for (uint32_t** p : {&L.rep[li], &L.pos[li], &L.reps[li], &L.walk[li]}) *p = (uint32_t*)at(take(mem, sizeof(uint32_t) * L.cap[li]));
                    L.codes[li] = (uint8_t*)at(take(mem, codes * L.cap[li]));
                    L.row_counts[li] = (unsigned long long*)at(take(mem, sizeof(unsigned long long) * L.cap[li]));
                    L.unknown[li] = (uint8_t*)at(take(mem, L.cap[li]));
                }
                L.edges = (FrontSurvivor*)at(take(mem, sizeof(FrontSurvivor) * D.cap_found));
                L.literal = (FrontEntry*)at(take(mem, sizeof(FrontEntry) * L.cap_literal));
                L.literal_parent = (uint32_t*)at(take(mem, sizeof(uint32_t) * L.cap_literal));
                L.rest = (uint32_t*)at(take(mem, sizeof(uint32_t) * L.cap_literal));
                L.literal_scratch = at(take(mem, pl.max_len >= 6 ? front_literal_goals_scratch_bytes(pl.R, kk, L.cap_literal) : 256));
                L.states[0] = (uint32_t*)at(take(states_bytes, (size_t)L.cap[0] * plane));
                L.states[1] = (uint32_t*)at(take(states_bytes, 2 * (size_t)L.cap[1] * plane));
            }
            for (size_t p = 0; p < pl.patterns.size() && !G.large; ++p) {
                const Pattern& pt = pl.patterns[p];
                int lg = 0, ls = 0;                      // (a skeleton's levels have two devices each)
                for (int j = pt.lo; j < pl.n && G.skeleton; ++j) (j <= pt.hi ? lg : ls) += pl.f[j] > 1 ? 1 : 0;
                const int shape = G.skeleton ? lg | ls << 4 : reg_shape_of(pt.g, pt.s, 0, 6);
                D.shape[p] = (uint8_t)shape;
                for (int d = 0; d < G.R; ++d)
                    if (!pt.master || (d & ((1 << (shape >> 4)) - 1)) == 0) D.part[p] |= 1ull << d;
            }
            D.all_rows = D.rows_kept >= 64 ? ~0ull : (1ull << D.rows_kept) - 1ull;
            D.all_cols = G.R >= 64 ? ~0ull : (1ull << G.R) - 1ull;
            if (G.large) { slots = 0; D.all_rows = D.all_cols = 0ull; }
            if (G.narrow) {
                D.cap_planes = 0;
                D.cap_found = std::min(D.cap_found, (1u << 18) - 1u);        // (a node's first edge is kept in 18 bits)
                D.own_chunks = (uint32_t)pl.k;
                for (int j = pl.n - 1, l = 0; j >= 0; --j) if (pl.f[j] > 1) D.own_size[l++] = (uint32_t)pl.f[j];
            }
            Place& P = places[g];
            P.table = take(zero, sizeof(unsigned long long) * slots);
            P.table_node = take(zero, sizeof(uint32_t) * slots);
            P.planes = take(mem, sizeof(ulonglong2) * (size_t)D.cap_planes * G.R);
            P.state = take(mem, sizeof(uint32_t) * D.cap_nodes);
            P.path = take(mem, G.large ? 0 : sizeof(unsigned long long) * D.cap_nodes);
            P.found = take(mem, G.large || G.narrow ? 0 : sizeof(uint4) * D.cap_found);
            P.narrow = take(mem, G.narrow ? sizeof(uint32_t) * (size_t)skeleton_state_words(group_levels(pl)) * D.cap_found : 0);
            P.nearest = take(mem, G.narrow ? D.cap_nodes : 0);
            P.count2 = take(mem, G.narrow ? sizeof(uint2) * D.cap_nodes : 0);
            P.node_edges = take(mem, G.narrow ? sizeof(uint32_t) * D.cap_nodes : 0);
            P.links = take(mem, sizeof(uint2) * D.cap_found);
            P.use_id = take(mem, sizeof(uint32_t) * D.cap_nodes);
            P.first = take(mem, sizeof(uint2) * (size_t)D.cap_nodes);
            P.use_ends = take(mem, sizeof(uint32_t) * 8 * (size_t)D.cap_nodes);
            P.edges = take(mem, sizeof(uint32_t) * D.cap_edges);
            P.edge_state = take(mem, G.skeleton ? 0 : sizeof(uint32_t) * D.cap_edges);
            P.edge_path = take(mem, G.skeleton && !G.narrow ? sizeof(unsigned long long) * D.cap_edges : 0);
            P.best = take(mem, sizeof(double) * (size_t)D.cap_edges * G.members.size());
        }
        // (nothing of the call that uses these is on its way: this attempt has queued nothing, those before were waited for)
        bool room = mem + zero + states_bytes <= kGraphBytesMax;
        if (room && (zero > C.g_zero.cap || mem > C.g_mem.cap || states_bytes > C.g_large.cap)) {
            size_t free_bytes = 0, all = 0;
            P2_HIP(hipMemGetInfo(&free_bytes, &all));
            room = graph_has_room(mem + zero + states_bytes, C.g_zero.cap + C.g_mem.cap + C.g_large.cap, free_bytes) && C.g_zero.ensure(zero) == hipSuccess &&
                   C.g_mem.ensure(mem) == hipSuccess && C.g_large.ensure(states_bytes) == hipSuccess;
        }
        if (!room) {                                     // (the other engines need less, and get what the graphs had)
            (void)hipGetLastError();
            C.g_zero.release(); C.g_mem.release(); C.g_large.release();
            bool any_large = false;                      // (they take the most: without them the others may well have room)
            for (const Graph& G : graphs) any_large |= G.large;
            for (const Graph& G : graphs) if (G.large || !any_large) leave_graph(G);
            return kWithoutGraphs;
        }
        P2_HIP(C.h_gctr.ensure(graph_back + 16));
        graph_zero = zero;
        char* z = static_cast<char*>(C.g_zero.p);
        char* m = static_cast<char*>(C.g_mem.p);
        for (size_t g = 0; g < n_graphs; ++g) {
            DevGraph& D = out[g];
            const Place& P = places[g];
            D.ctr = reinterpret_cast<GraphCounters*>(z) + g;
            D.table = reinterpret_cast<unsigned long long*>(z + P.table); D.table_node = reinterpret_cast<uint32_t*>(z + P.table_node);
            D.planes = reinterpret_cast<ulonglong2*>(m + P.planes); D.node_state = reinterpret_cast<uint32_t*>(m + P.state);
            D.found = reinterpret_cast<uint4*>(m + P.found); D.links = reinterpret_cast<uint2*>(m + P.links);
            D.use_id = reinterpret_cast<uint32_t*>(m + P.use_id); D.first_edge = reinterpret_cast<uint2*>(m + P.first);
            D.use_ends = reinterpret_cast<uint32_t*>(m + P.use_ends);
            D.edges = reinterpret_cast<uint32_t*>(m + P.edges); D.edge_state = reinterpret_cast<uint32_t*>(m + P.edge_state);
            D.best = reinterpret_cast<double*>(m + P.best);
            D.node_path = reinterpret_cast<unsigned long long*>(m + P.path); D.edge_path = reinterpret_cast<unsigned long long*>(m + P.edge_path);
            D.narrow_planes = reinterpret_cast<uint32_t*>(m + P.narrow); D.node_edges = reinterpret_cast<uint32_t*>(m + P.node_edges);
            D.nearest = reinterpret_cast<uint8_t*>(m + P.nearest);
            D.count2 = reinterpret_cast<uint2*>(m + P.count2);
            D.members = reinterpret_cast<const int32_t*>(static_cast<char*>(C.blob.p) + graphs[g].off_members);
            D.sizes = graphs[g].skeleton ? reinterpret_cast<const DevMember*>(static_cast<char*>(C.blob.p) + graphs[g].off_sizes) : nullptr;
            if (!graphs[g].large) continue;
            LargeAt& L = large_at[g];
            auto shift = [](auto*& p, char* base) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + reinterpret_cast<size_t>(p)); };
            shift(L.ctr, z); shift(L.marks, m);
            for (int li = 0; li < 2; ++li) {
                shift(L.states[li], static_cast<char*>(C.g_large.p));
                shift(L.table[li], z); shift(L.hash[li], m);
                shift(L.rep[li], m); shift(L.pos[li], m); shift(L.reps[li], m); shift(L.walk[li], m);
                shift(L.codes[li], m); shift(L.row_counts[li], m); shift(L.unknown[li], m);
                D.large[li] = reinterpret_cast<const uint4*>(L.states[li]);
            }
            shift(L.edges, m); shift(L.literal, m); shift(L.literal_parent, m); shift(L.rest, m);
            L.literal_scratch = m + reinterpret_cast<size_t>(L.literal_scratch);
        }
        return P2_OK;
    };
    // The graph of a large group: its kernels queued level by level, with nothing to wait for.  (More blocks than a level has
    // states end at once; a level's states are some 45, 450, 2 000, 5 400, 8 900 with four levels.)
    auto queue_large = [&](size_t g, hipStream_t on, SpanRec& spans) -> int32_t {
        const Graph& G = graphs[g];
        const Plan& pl = runs[G.leader].plan;
        const LargeAt& L = large_at[g];
        const DevGraph& D = reinterpret_cast<const DevGraph*>(static_cast<char*>(C.h_blob.p) + off_graphs)[g];
        const DevQuery* const dq = reinterpret_cast<const DevQuery*>(static_cast<char*>(C.blob.p) + G.off_query);
        const int kk = D.rows_kept, M = pl.max_len;
        const size_t sw = frontier_state_words(pl.R, kk);
        // (the few states that are judged literally, 350 us of a chain on some 50 compute units with 512 devices, go beside the
        //  last two levels' work where the stream of the uploads has nothing to do: one query of 512 devices 4 125 us in one chain, 3 740 so)
        const bool beside = only_graphs && large_slots == 1;
        const hipStream_t side = beside ? C.copy_stream : on;
        const bool judge_literal = M >= 6;               // (with fewer instructions no child needs a third pair; one that did would be reported)
        P2_HIP(launch_front_init(dq, 0u, pl.R, kk, L.literal, L.states[0], nullptr, L.rest, 0, on));
        P2_HIP(launch_front_root(L.ctr, L.marks, L.rep[0], L.pos[0], L.reps[0], on));
        for (int l = 0; l < M; ++l) {
            const bool last = l + 1 == M;
            const int lists = l < 2 ? 1 : 2;             // (the first AllGather that can leave two pairs is the second instruction)
            const uint32_t most = l == 0 ? 1u : l == 1 ? 160u : l == 2 ? 1024u : 1u << 20;      // (blocks: a bound on the states, for the grid alone)
            if (l > 0) P2_HIP(launch_front_mark(L.ctr, L.marks, l + 1, on));
            const uint32_t* list[2]; const uint32_t* n_list[2]; const uint32_t* from[2];
            for (int li = 0; li < 2; ++li) { list[li] = L.reps[li]; n_list[li] = &L.marks->rep[li][l + 1]; from[li] = &L.marks->rep[li][l]; }
            if (last) {
                P2_HIP(spans.begin(SpanRec::kGroup, on));
                for (int li = 0; li < lists; ++li)
                    P2_HIP(launch_front_goal_filter(dq, pl.R, kk, L.states[li], std::min(most, L.cap[li]), list[li], n_list[li], from[li], li + 1, L.codes[li],
                                                    L.row_counts[li], L.unknown[li], L.walk[li], &L.ctr->n_walk[li], on));
                P2_HIP(spans.end(on));
            }
            P2_HIP(spans.begin(SpanRec::kClassify, on, lists));
            for (int li = 0; li < lists; ++li)
                P2_HIP(launch_front_classify(dq, pl.R, kk, L.states[li], std::min(most, L.cap[li]), last ? L.walk[li] : list[li],
                                             last ? &L.ctr->n_walk[li] : n_list[li], last ? &L.marks->edges[0] : from[li], li + 1, 2, last ? 1 : 0, 0, L.codes[li],
                                             L.row_counts[li], L.unknown[li], L.ctr, on));
            P2_HIP(spans.end(on));
            P2_HIP(spans.begin(SpanRec::kGroup, on));
            FrontEdges E;
            E.edges = L.edges; E.cap_edges = D.cap_found; E.literal = L.literal; E.literal_parent = L.literal_parent; E.cap_literal = L.cap_literal;
            E.ctr = L.ctr; E.max_len = M;
            for (int li = 0; li < lists; ++li)
                P2_HIP(launch_front_edges(dq, list[li], n_list[li], from[li], L.codes[li], L.unknown[li], li + 1, l, l == 0 ? 1u : l == 1 ? 6u : 320u, E, on));
            P2_HIP(spans.end(on));
            if (last) break;
            if (l + 2 == M && judge_literal) {           // (they are judged one instruction later: everything that asks for is there now)
                if (beside) {
                    P2_HIP(hipEventRecord(C.front_go, on));
                    P2_HIP(hipStreamWaitEvent(side, C.front_go, 0));
                }
                P2_HIP(spans.begin(SpanRec::kLiteral, side));
                P2_HIP(launch_front_literal_goals(dq, pl.R, kk, L.literal, L.literal_parent, L.cap_literal, &L.ctr->next_literal, l + 1, L.states[0], L.states[1],
                                                  L.literal_scratch, nullptr, 0, L.ctr, L.rest, side));
                P2_HIP(spans.end(side));
                if (beside) P2_HIP(hipEventRecord(C.copy_done, side));
            }
            FrontLevel lv;
            std::memset(&lv, 0, sizeof lv);
            lv.states1 = L.states[0]; lv.states2 = L.states[1];
            lv.surv = L.edges; lv.n_surv = D.cap_found;
            lv.next_states1 = L.states[0]; lv.next_states2 = L.states[1]; lv.next_hash1 = L.hash[0]; lv.next_hash2 = L.hash[1];
            lv.surv_from = &L.marks->edges[l + 1]; lv.surv_end = &L.ctr->n_ssurv;
            lv.cap1 = L.cap[0]; lv.cap2 = L.cap[1]; lv.blocks = l == 0 ? 128u : l == 1 ? 1024u : 4096u;
            P2_HIP(spans.begin(SpanRec::kMaterialize, on, lists));
            for (int li = 0; li < lists; ++li) {         // (a launch of its own for the parents with two pairs, which need twice the LDS)
                lv.lds_planes = li + 1; lv.only = lists == 1 ? 0 : li + 1;
                P2_HIP(launch_front_materialize(dq, pl.R, kk, lv, on));
            }
            P2_HIP(spans.end(on));
            P2_HIP(spans.begin(SpanRec::kGroup, on));
            for (int li = 0; li < (l == 0 ? 1 : 2); ++li)
                P2_HIP(launch_front_find(L.states[li], sw * (size_t)(li + 1), L.hash[li], &L.marks->child[li][l + 1], &L.ctr->t_next[li], L.cap[li], L.table[li],
                                         L.table_size[li], L.rep[li], L.pos[li], L.reps[li], &L.ctr->n_reps[li], l == 0 ? 32u : l == 1 ? 256u : 2048u, on));
            P2_HIP(spans.end(on));
        }
        if (beside && judge_literal) P2_HIP(hipStreamWaitEvent(on, C.copy_done, 0));
        FrontLinks K;
        std::memset(&K, 0, sizeof K);
        K.ctr = L.ctr; K.marks = L.marks; K.graph = D.ctr; K.edges = L.edges;
        for (int li = 0; li < 2; ++li) { K.rep[li] = L.rep[li]; K.pos[li] = L.pos[li]; K.reps[li] = L.reps[li]; }
        K.links = D.links; K.node_state = D.node_state;
        K.cap_edges = D.cap_found; K.cap1 = L.cap[0]; K.cap2 = L.cap[1]; K.cap_literal = L.cap_literal; K.cap_nodes = D.cap_nodes;
        K.max_len = M; K.literal_judged = judge_literal ? 1 : 0;
        P2_HIP(launch_front_links(K, 64u, on));
        return P2_OK;
    };
    bool repeated = false;
    for (int attempt = 0; attempt < 4; ++attempt) {
        auto tot = layout_lists();
        P2_HIP(C.valid.ensure(sizeof(unsigned long long) * std::max<size_t>(tot.first, 1)));
        P2_HIP(C.rerun.ensure(sizeof(unsigned long long) * std::max<size_t>(tot.second, 1)));
        std::memset(hb, 0, blob_bytes);
        for (int m = 0; m < n_msg; ++m) reinterpret_cast<double*>(hb + off_msg)[m] = msg_bytes[m];
        for (int i = 0; i < n_queries; ++i) {
            QueryRun& r = runs[i];
            const Plan& pl = r.plan;
            DevQuery* dq = reinterpret_cast<DevQuery*>(hb + r.off_query);
            dq->R = pl.R; dq->k = pl.k;
            dq->MW = (pl.R + 31) / 32; dq->KW = (pl.k + 31) / 32;
            dq->n_patterns = (int)pl.patterns.size(); dq->n_ops = pl.n_ops; dq->alphabet = pl.alphabet; dq->algo = pl.algo;
            dq->max_len = pl.max_len; dq->n_levels = pl.n; dq->n_msg = n_msg;
            dq->n_candidates = pl.n_candidates;
            for (int l = 0; l <= P2_MAX_LEN + 1; ++l) dq->base[l] = pl.base[l];
            for (int o = 0; o < pl.n_ops; ++o) dq->ops[o] = (uint8_t)pl.ops[o];
            dq->magic_alphabet = pl.alphabet <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (unsigned)pl.alphabet + 1ull);
            for (int d = 0; d < pl.alphabet; ++d)
                dq->instr_of_digit[d] = (uint16_t)(((d / pl.n_ops) << 3) | pl.ops[d % pl.n_ops]);
            for (int j = 0; j < pl.n; ++j) { dq->alpha[j] = pl.alpha[j]; dq->inv_bw[j] = 1.0 / pl.bw[j]; }
            for (size_t pi = 0; pi < pl.patterns.size(); ++pi) {
                const Pattern& p = pl.patterns[pi];
                DevPattern& dp = dq->pat[pi];
                dp.g = p.g; dp.s = p.s; dp.master = p.master; dp.n_groups = p.n_groups; dp.span_level = p.span;
                dp.reg_shape = reg_shape_of(p.g, p.s, p.master, 5);
                dp.rank_off = 0; dp.pad1 = 0;
            }
            dq->goal_mask = nullptr; dq->rank_tbl = nullptr;
            if (pl.hierarchy != P2_HIERARCHY_COLLAPSED) {
                if (!pl.goal.empty()) {
                    // the plan's rows are ceil(R/32) words long, the kernels' a power of two
                    const int mw = (pl.R + 31) / 32, mwd = literal_mask_words(pl.R);
                    uint32_t* goal = reinterpret_cast<uint32_t*>(hb + r.off_goal);
                    for (int d = 0; d < pl.R; ++d)
                        for (int w = 0; w < mwd; ++w) goal[(size_t)d * mwd + w] = w < mw ? pl.goal[(size_t)d * mw + w] : 0u;
                    dq->goal_mask = reinterpret_cast<const uint32_t*>(db + r.off_goal);
                }
                int32_t* ranks = reinterpret_cast<int32_t*>(hb + r.off_rank);
                int32_t at = 0;
                for (size_t pi = 0; pi < pl.patterns.size(); ++pi) {
                    const Pattern& p = pl.patterns[pi];
                    if (p.rank.empty()) continue;
                    std::memcpy(ranks + at, p.rank.data(), sizeof(int32_t) * p.rank.size());
                    dq->pat[pi].rank_off = at + 1;
                    at += (int32_t)p.rank.size();
                }
                dq->rank_tbl = reinterpret_cast<const int32_t*>(db + r.off_rank);
            }
            dq->rows = static_cast<const DevRows*>(C.rows_hdr.p) + runs[i].rows_at;
            dq->reg_sum_part = 0;
            for (size_t pi = 0; pi < pl.patterns.size(); ++pi) {
                const Pattern& p = pl.patterns[pi];
                const int shape = reg_shape_of(p.g, p.s, p.master, 6);
                unsigned long long part = pl.R >= 64 ? ~0ull : ((1ull << pl.R) - 1ull);
                if (p.master) {
                    unsigned long long every = 0;             // bit d set iff d % s == 0
                    for (int d = 0; d < 64; d += p.s) every |= 1ull << d;
                    part &= every;
                }
                dq->reg_shape[pi] = (shape < 0 ? 0u : (uint32_t)shape) | ((uint32_t)(p.n_groups * p.g) << 16);
                dq->reg_part[pi] = part;
                dq->reg_sum_part += (uint32_t)(p.n_groups * p.g) * (uint32_t)pl.n_ops;
            }
            dq->msg_bytes = reinterpret_cast<const double*>(db + off_msg);
            dq->valid_idx = static_cast<unsigned long long*>(C.valid.p) + r.off_valid;
            dq->rerun_idx = static_cast<unsigned long long*>(C.rerun.p) + r.off_rerun;
            dq->valid_cap = r.valid_cap; dq->rerun_cap = r.rerun_cap;
            dq->counters = static_cast<DevCounters*>(C.counters.p) + i;
        }
        for (auto& L : launches)
        {
            std::memcpy(hb + L.off_segs, L.segs.data(), sizeof(DevSegment) * L.segs.size());
            if (!L.shares.empty()) std::memcpy(hb + L.off_shares, L.shares.data(), sizeof(DevShare) * L.shares.size());
        }
        for (auto& A : autos) std::memcpy(hb + A.off, A.qlist.data(), sizeof(int32_t) * A.qlist.size());
        if (!graphs.empty()) {
            const int32_t rc = layout_graphs(reinterpret_cast<DevGraph*>(hb + off_graphs));
            if (rc != P2_OK) return rc;
            for (size_t g = 0; g < graphs.size(); ++g) {
                if (!graphs[g].large) continue;
                DevQuery* dq = reinterpret_cast<DevQuery*>(hb + graphs[g].off_query);
                std::memcpy(dq, hb + runs[graphs[g].leader].off_query, sizeof(DevQuery));
                const DevGraph& D = reinterpret_cast<const DevGraph*>(hb + off_graphs)[g];
                dq->k = D.rows_kept; dq->KW = (D.rows_kept + 31) / 32; dq->n_msg = 0; dq->rows_split = (int32_t)D.split_check;
            }
            for (int i = 0; i < n_queries; ++i)
                reinterpret_cast<GraphQuery*>(hb + off_gasked)[i] = GraphQuery{runs[i].graph ? (uint32_t)runs[i].graph_id : ~0u, (uint32_t)runs[i].graph_pos, fused_sums(runs[i]), 0u};
            for (const Graph& G : graphs) {
                std::memcpy(hb + G.off_members, G.members.data(), sizeof(int32_t) * G.members.size());
                for (size_t t = 0; t < G.members.size() && G.skeleton; ++t) describe_member(runs[G.members[t]].plan, reinterpret_cast<DevMember*>(hb + G.off_sizes)[t]);
            }
            if (!glevel.empty()) std::memcpy(hb + off_glevel, glevel.data(), sizeof(GraphBlock) * glevel.size());
            if (!gsteps.empty()) std::memcpy(hb + off_gsteps, gsteps.data(), sizeof(GraphBlock) * gsteps.size());
            if (!gcosts.empty()) std::memcpy(hb + off_gcosts, gcosts.data(), sizeof(GraphBlock) * gcosts.size());
            if (!gsmall.empty()) std::memcpy(hb + off_gsmall, gsmall.data(), sizeof(uint32_t) * gsmall.size());
            if (!glarge.empty()) std::memcpy(hb + off_glarge, glarge.data(), sizeof(uint32_t) * glarge.size());
        }
        // (rows: the shared ones, the other queries' own; costs: behind those, the columns of the queries that share.  Without the room,
        //  the programs are counted first, as for other lists: there may be fewer)
        if (shortlists && (C.sorted.ensure(sizeof(unsigned long long) * listed_rows) != hipSuccess ||
                           C.progs.ensure(sizeof(p2_program) * listed_rows) != hipSuccess ||
                           C.walks.ensure(2 * sizeof(uint4) * shared_rows) != hipSuccess ||
                           C.costs.ensure(sizeof(double) * (listed_rows + shared_costs) * (size_t)n_msg) != hipSuccess ||
                           C.topk_pos.ensure(sizeof(long long) * shortlist_out) != hipSuccess ||
                           C.h_progs.ensure(sizeof(p2_program) * shortlist_out) != hipSuccess ||
                           C.h_costs.ensure(sizeof(double) * shortlist_out * (size_t)n_msg) != hipSuccess ||
                           C.h_pos.ensure(sizeof(uint32_t) * n_jobs) != hipSuccess)) {
            (void)hipGetLastError();
            shortlists = false;
        }
        if (shortlists) {
            GraphRows* seg = reinterpret_cast<GraphRows*>(hb + off_rows);
            GraphSums* sum = reinterpret_cast<GraphSums*>(hb + off_sums);
            GraphColumn* const columns = reinterpret_cast<GraphColumn*>(hb + off_columns);
            size_t first = 0, out = 0, own_costs = listed_rows;
            uint32_t block = 0, sum_block = 0, column = 0;
            std::vector<std::pair<size_t, uint32_t>> shared(graphs.size(), {0, 0u});     // a graph's rows, and its first column
            auto queue_rows = [&](const QueryRun& r, int i, uint32_t member) {
                const size_t most = most_valid(r.plan);
                *seg++ = GraphRows{block, (uint32_t)i, (uint32_t)r.graph_id, member, (uint32_t)most, fused_sums(r), (unsigned long long)first};
                block += (uint32_t)((most + 255) / 256);
                first += most;
                return first - most;
            };
            for (size_t g = 0; g < graphs.size(); ++g) {
                const Graph& G = graphs[g];
                if (!shares_rows(G)) continue;
                const size_t most = most_valid(runs[G.leader].plan), at = queue_rows(runs[G.leader], G.leader, ~0u);
                *sum++ = GraphSums{sum_block, (uint32_t)g, (uint32_t)most, (uint32_t)G.members.size(), column, fused_sums(runs[G.leader]), (unsigned long long)at};
                shared[g] = {at, column};
                sum_block += (uint32_t)((most + sum_rows - 1) / sum_rows); column += (uint32_t)G.members.size();
            }
            DevTopkJob* J = reinterpret_cast<DevTopkJob*>(hb + off_jobs);
            uint32_t* own_flag = static_cast<uint32_t*>(C.h_pos.p);
            for (int i = 0; i < n_queries; ++i) {
                const QueryRun& r = runs[i];
                if (!r.graph) continue;
                const size_t most = most_valid(r.plan);
                size_t rows, costs_at;
                if (shares_rows(graphs[r.graph_id])) {
                    rows = shared[r.graph_id].first; costs_at = own_costs;
                    columns[shared[r.graph_id].second + (uint32_t)r.graph_pos] = GraphColumn{(unsigned long long)costs_at, (uint32_t)i, 0u};
                    own_costs += most;
                } else rows = costs_at = queue_rows(r, i, (uint32_t)r.graph_pos);
                for (int m = 0; m < n_msg; ++m, ++J) {
                    J->costs = static_cast<double*>(C.costs.p) + costs_at * (size_t)n_msg;
                    J->cost = J->costs + m; J->index = static_cast<unsigned long long*>(C.sorted.p) + rows; J->progs = static_cast<p2_program*>(C.progs.p) + rows;
                    J->nan_flag = nullptr; J->own_flag = own_flag++;
                    J->n = (long long)most; J->stride = n_msg; J->k = r.topk; J->n_cost = n_msg;
                    J->n_from = &reinterpret_cast<const GraphCounters*>(C.g_zero.p)[r.graph_id].n_total;
                    J->out_pos = static_cast<long long*>(C.topk_pos.p) + out;
                    J->out_progs = static_cast<p2_program*>(C.h_progs.p) + out; J->out_costs = static_cast<double*>(C.h_costs.p) + out * (size_t)n_msg;
                    out += shortlist_rows_of(r.plan, r.topk, 1);
                }
            }
        }
        if (only_graphs) {
            const CopyPart in[2] = {{db, hb, blob_bytes}, {C.g_zero.p, nullptr, graph_zero}};
            P2_HIP(launch_copies(in, 2, stream));
        } else {
            P2_HIP(hipMemcpyAsync(db, hb, blob_bytes, hipMemcpyHostToDevice, stream));
            P2_HIP(hipMemsetAsync(C.counters.p, 0, sizeof(DevCounters) * (size_t)n_queries, stream));
            if (!graphs.empty()) P2_HIP(hipMemsetAsync(C.g_zero.p, 0, graph_zero, stream));
        }
        // ---- evaluate every candidate of every query
        int eval_launches = 0;
        if (g_prof.on) P2_HIP(hipEventRecord(g_prof.ev[0], stream));
        const DevQuery* const dqs = reinterpret_cast<const DevQuery*>(db);
        const DevGraph* const dgs = reinterpret_cast<const DevGraph*>(db + off_graphs);
        if (!gsmall.empty()) {
            ++eval_launches;
            int max_R = 1;
            for (uint32_t g : gsmall) max_R = std::max(max_R, graphs[g].R);
            P2_HIP(launch_graph_alone(dgs, reinterpret_cast<const uint32_t*>(db + off_gsmall), (unsigned)gsmall.size(), max_R, stream));
        }
        if (alone_skeletons) {
            ++eval_launches;
            P2_HIP(launch_skeleton_alone(dgs, n_skeletons, stream));
        }
        // (the blocks of a launch: what a graph of each size can do with, and less to each where there are many.  Three hundred of three
        //  levels, some 1 024 blocks a launch for them: 720 us a call, 2 048: 740, 4 096: 757, 44 to each: 845; for the costs no more than
        //  4 096, where 1 024 to each took 221 us of device time)
        auto skeleton_grid = [&](const uint32_t (&blocks)[3], const uint32_t (&links)[3], uint32_t least, uint32_t all) {
            SkeletonGrid grid;
            for (int c = 0; c < 3; ++c) {
                const uint32_t share = std::max(least, all / std::max(1u, n_narrow[c]));
                grid.graphs[c] = n_narrow[c]; grid.blocks[c] = std::min(blocks[c], share); grid.links[c] = std::min(links[c], share);
            }
            return grid;
        };
        // large groups: one on the call's stream, several on the slots', the largest first, each to the slot with the least to do
        size_t n_slots_used = 0;
        if (n_large > 0) {
            if (g_prof.on) P2_HIP(hipEventRecord(g_prof.ev[3], stream));
            for (FrontSlot& S : C.slots) { S.spans.on = g_prof.on; S.spans.kernels_only = g_prof.kernels_only; S.spans.reset(); }
            std::vector<size_t> order;
            for (size_t g = 0; g < graphs.size(); ++g) if (graphs[g].large) order.push_back(g);
            // (512 devices, four levels, six instructions: 3.3 ms alone; 256: 2.0; 128: 1.5: a chain of launches, and what the devices add)
            auto weight = [&](size_t g) { const Plan& pl = runs[graphs[g].leader].plan; return (96.0 + pl.R) * (1024.0 + graph_room(pl)); };
            std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) { return weight(x) > weight(y); });
            if (large_slots > 1) {
                n_slots_used = (size_t)large_slots;
                P2_HIP(hipEventRecord(C.front_go, stream));
                for (size_t t = 0; t < n_slots_used; ++t) P2_HIP(hipStreamWaitEvent(C.slots[t].stream, C.front_go, 0));
            }
            double load[kFrontSlots] = {};
            for (size_t g : order) {
                size_t t = 0;
                for (size_t u = 1; u < n_slots_used; ++u) if (load[u] < load[t]) t = u;
                load[t] += weight(g);
                const int32_t rc = queue_large(g, n_slots_used > 0 ? C.slots[t].stream : stream, C.slots[t].spans);
                if (rc != P2_OK) return rc;
            }
        }
        if (!glevel.empty()) {
            eval_launches += graph_levels;
            for (int level = 0; level < graph_levels; ++level)
                P2_HIP(launch_graph_level(dgs, reinterpret_cast<const GraphBlock*>(db + off_glevel), (unsigned)glevel.size(), level, graph_levels, stream));
        }
        if (n_large > 0) {
            for (size_t t = 0; t < n_slots_used; ++t) {
                if (!C.slot_done[t]) P2_HIP(hipEventCreateWithFlags(&C.slot_done[t], hipEventDisableTiming));
                P2_HIP(hipEventRecord(C.slot_done[t], C.slots[t].stream));
                P2_HIP(hipStreamWaitEvent(stream, C.slot_done[t], 0));
            }
            if (g_prof.on) P2_HIP(hipEventRecord(g_prof.ev[4], stream));
        }
        if (n_skeletons > 0 && !alone_skeletons) {
            for (int l = 0; l < narrow_levels; ++l) {
                // (blocks: of four states with four levels, which have some 45, 450, 2 000, 5 400 and 8 900, of eight with three, at most
                //  some 330, and one with fewer; a block for every 64 or 128 edges that led there)
                static const uint32_t states[P2_MAX_LEN][3] = {{1, 1, 1}, {1, 4, 12}, {1, 32, 128}, {1, 44, 512}, {1, 44, 768}, {1, 44, 768}, {1, 44, 768}};
                static const uint32_t links[P2_MAX_LEN][3] = {{0, 0, 0}, {1, 1, 2}, {1, 2, 8}, {1, 4, 32}, {1, 8, 96}, {1, 8, 192}, {1, 8, 192}};
                ++eval_launches;
                P2_HIP(launch_skeleton_level(dgs, skeleton_grid(states[l], links[l], 4, 1024), l, stream));
            }
            ++eval_launches;
            uint32_t most_nodes = 0, most_edges = 0;
            int most_len = 0;
            for (uint32_t g = 0; g < n_skeletons; ++g) {
                const DevGraph& D = reinterpret_cast<const DevGraph*>(hb + off_graphs)[g];
                most_nodes = std::max(most_nodes, D.cap_nodes);
                most_edges = std::max(most_edges, D.cap_found);
                most_len = std::max(most_len, (int)D.max_len);
            }
            P2_HIP(launch_skeleton_finish(dgs, skeleton_grid({1, 4, 64}, {0, 0, 0}, 64, 64), most_nodes, most_edges, most_len, stream));
        }
        if (!glarge.empty()) {
            ++eval_launches;
            // (a byte per node, a word for every count of a node inside, two words per digit set of a node on the way to a goal:
            //  less than ten bytes a node together where there are many, three words where there are few)
            uint32_t most = 0;
            for (uint32_t g : glarge) most = std::max(most, reinterpret_cast<const DevGraph*>(hb + off_graphs)[g].cap_nodes);
            P2_HIP(launch_graph_finish(dgs, reinterpret_cast<const uint32_t*>(db + off_glarge), (unsigned)glarge.size(),
                                       most <= 4096 ? (size_t)most * 12 + 4096 : (size_t)160 * 1024, stream));
        }
        for (auto& L : launches) {
            ++eval_launches;
            if (L.kind == 2)
                P2_HIP(launch_eval_shared(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const DevSegment*>(db + L.off_segs),
                                          (int)L.segs.size(), reinterpret_cast<const DevShare*>(db + L.off_shares),
                                          (int)L.shares.size(), L.grid, L.max_R, L.max_k, stream));
            else if (L.kind == 1)
                P2_HIP(launch_eval_regs(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const DevSegment*>(db + L.off_segs),
                                        (int)L.segs.size(), L.blocks, stream));
            else
                P2_HIP(launch_eval_compact(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const DevSegment*>(db + L.off_segs),
                                           (int)L.segs.size(), L.blocks, L.max_R, L.max_k, stream));
        }
        for (int i = 0; i < n_queries; ++i) {
            QueryRun& r = runs[i];
            const DevQuery* dq = reinterpret_cast<const DevQuery*>(db + r.off_query);
            if (r.engine == P2_ENGINE_LITERAL && r.same_as < 0 && r.plan.n_candidates > 0) {
                ++eval_launches;
                void* gs = nullptr;
                P2_HIP(lit_scratch(r.plan, &gs));
                P2_HIP(launch_eval_literal(dq, r.plan.R, r.plan.k, 0ull, r.plan.n_candidates, nullptr, nullptr, gs, stream));
            }
        }
        if (g_prof.on) { P2_HIP(hipEventRecord(g_prof.ev[1], stream)); g_prof.last.eval_launches = eval_launches; }
        for (auto& A : autos) {
            unsigned nb = 0;
            P2_HIP(C.lit_scratch.ensure(literal_group_scratch_bytes(A.max_R, A.max_k, &nb)));
            P2_HIP(launch_eval_literal_groups_auto(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const int32_t*>(db + A.off),
                                                   (int)A.qlist.size(), A.max_R, A.max_k, C.lit_scratch.p, A.class_cap, stream));
        }
        // while the GPU evaluates: the cost model's tables (first attempt only)
        {
            const int32_t rc = build_and_upload_rows();
            if (rc != P2_OK) return rc;
        }
        if (!gsteps.empty())
            P2_HIP(launch_graph_steps(dqs, dgs, reinterpret_cast<const GraphBlock*>(db + off_gsteps), (unsigned)gsteps.size(), stream));
        P2_HIP(launch_graph_costs(dqs, dgs, reinterpret_cast<const GraphBlock*>(db + off_gcosts), (unsigned)gcosts.size(), stream));
        if (n_skeletons > 0) {
            // (a block for every state on the way to a goal)
            static const uint32_t used[P2_MAX_LEN + 1][3] = {{1, 1, 1}, {1, 1, 1}, {5, 7, 9}, {17, 33, 51}, {23, 97, 229}, {24, 171, 662}, {24, 230, 1419}, {24, 230, 1419}};
            P2_HIP(launch_skeleton_costs(dqs, dgs, skeleton_grid(used[narrow_levels], {0, 0, 0}, 16, 4096), most_members, n_msg > 0 ? 1 : 0, stream));
        }
        if (direct && (C.h_progs.ensure(sizeof(p2_program) * rows_room) != hipSuccess ||
                       C.h_costs.ensure(sizeof(double) * rows_room * (size_t)std::max(n_msg, 1)) != hipSuccess)) {
            (void)hipGetLastError();                     // (the rows themselves may well need less)
            direct = false;
        }
        if (shortlists) {
            // (the last block hands the counts to the host)
            P2_HIP(launch_graph_emit(dqs, dgs, static_cast<const GraphCounters*>(C.g_zero.p), nullptr, 0, reinterpret_cast<const GraphRows*>(db + off_rows), (int)n_segs,
                                     shortlist_blocks + 1u, listed_rows, static_cast<unsigned long long*>(C.sorted.p), static_cast<p2_program*>(C.progs.p),
                                     static_cast<double*>(C.costs.p), C.h_gctr.p, (int)graphs.size(), C.walks.p, stream));
            if (sums_blocks > 0)
                P2_HIP(launch_graph_sums(dqs, dgs, reinterpret_cast<const GraphSums*>(db + off_sums), (int)n_sums, reinterpret_cast<const GraphColumn*>(db + off_columns),
                                         sums_blocks, most_columns, sum_rows, C.walks.p, static_cast<double*>(C.costs.p), stream));
            P2_HIP(launch_topk_jobs(reinterpret_cast<const DevTopkJob*>(db + off_jobs), (unsigned)n_jobs, shortlist_k, (long long)shortlist_most, stream));
            if (g_prof.on) { P2_HIP(hipEventRecord(g_prof.ev[2], stream)); g_prof.last.post_launches = sums_blocks > 0 ? 3 : 2; }
        } else if (direct) {
            P2_HIP(launch_graph_emit(dqs, dgs, static_cast<const GraphCounters*>(C.g_zero.p), reinterpret_cast<const GraphQuery*>(db + off_gasked),
                                     n_queries, nullptr, 0, (unsigned)emit_blocks + 1u, rows_room, nullptr, static_cast<p2_program*>(C.h_progs.p),
                                     static_cast<double*>(C.h_costs.p), C.h_gctr.p, (int)graphs.size(), nullptr, stream));
            if (g_prof.on) { P2_HIP(hipEventRecord(g_prof.ev[2], stream)); g_prof.last.post_launches = 2; }
        } else {
            const CopyPart back[2] = {{C.h_counters.p, C.counters.p, n_others > 0 ? sizeof(DevCounters) * (size_t)n_queries : 0},
                                      {C.h_gctr.p, C.g_zero.p, graph_nan}};
            P2_HIP(launch_copies(back, 2, stream));
        }
        P2_HIP(hipStreamSynchronize(stream));
        bool again = false;
        const GraphCounters* const hg = static_cast<const GraphCounters*>(C.h_gctr.p);
        // (a graph that failed costs its own queries their place, not the others': they stay with theirs when the call is repeated)
        bool failed = false;
        for (size_t g = 0; g < graphs.size(); ++g) {
            unsigned long long valid = 0;
            for (int len = 1; len <= P2_MAX_LEN; ++len) valid += hg[g].n_valid[len];
            if ((hg[g].flags & ~kGraphFull) != 0u || (hg[g].flags != 0u && attempt == 3) || valid > 0xffffffffull) {
                leave_graph(graphs[g]);
                failed = true;
            } else again |= hg[g].flags != 0u;
        }
        if (failed) return kWithoutGraphs;
        if (again) graph_scale *= 4;
        const DevCounters* hc = static_cast<const DevCounters*>(C.h_counters.p);
        // candidates whose state the compact engine could not hold go through the literal engine:
        // one launch per mask-width class for the states that fit in LDS, one per query otherwise
        bool reran = false;
        std::vector<PostLaunch> rerun_launches;
        for (int i = 0; i < n_queries; ++i) {
            QueryRun& r = runs[i];
            if (r.graph || hc[i].n_rerun == 0 || hc[i].n_rerun > r.rerun_cap || r.auto_groups) continue;
            reran = true;
            if (literal_lds_bytes(r.plan.R, r.plan.k) != 0) {
                add_seg(rerun_launches, mask_class(r.plan.R), r.plan, i, hc[i].n_rerun, 1, r.off_rerun, 0);
            } else {
                void* gs = nullptr;
                P2_HIP(lit_scratch(r.plan, &gs));
                P2_HIP(launch_eval_literal(reinterpret_cast<const DevQuery*>(db + r.off_query), r.plan.R, r.plan.k, 0ull,
                                           hc[i].n_rerun, static_cast<unsigned long long*>(C.rerun.p) + r.off_rerun, nullptr, gs, stream));
            }
        }
        if (!rerun_launches.empty()) {
            P2_HIP(upload_segs({&rerun_launches}));
            for (auto& L : rerun_launches)
                P2_HIP(launch_eval_literal_list(reinterpret_cast<const DevQuery*>(db), segs_of(L), (int)L.segs.size(), L.blocks,
                                                L.max_R, L.lit_lds, static_cast<unsigned long long*>(C.rerun.p), stream));
        }
        if (reran) {
            P2_HIP(launch_copy_out(C.h_counters.p, C.counters.p, sizeof(DevCounters) * (size_t)n_queries, stream));
            P2_HIP(hipStreamSynchronize(stream));
        }
        for (int i = 0; i < n_queries; ++i) {
            QueryRun& r = runs[i];
            if (r.plan.n_candidates == 0) continue;       // (a reduction over one device: nothing was evaluated)
            if (r.graph) {
                const GraphCounters& gc = hg[r.graph_id];
                const Plan& pl = r.plan;
                // A walk applies, to every candidate that starts with a valid prefix, one more instruction (a program that
                // has reached the goal is not valid with one more: every rule fails there); the enumeration by size applies
                // the alphabet to every prefix.
                unsigned long long walked = 0, listed = 0, valid = 0, per_alphabet = 0;
                for (const Pattern& p : pl.patterns) per_alphabet += (unsigned long long)p.g * p.n_groups * pl.n_ops;
                for (int len = 0; len < pl.max_len; ++len) {
                    unsigned long long behind = 0, power = 1;
                    for (int l = len; l < pl.max_len; ++l) { behind += power; power *= (unsigned long long)pl.alphabet; }
                    const unsigned long long prefixes = len == 0 ? 1ull : gc.n_prefixes[len];
                    walked += behind * (prefixes + (len > 0 ? gc.n_valid[len] : 0u));
                    listed += prefixes;
                }
                for (int len = 1; len <= pl.max_len; ++len) valid += gc.n_valid[len];
                r.n_valid = (uint32_t)valid; r.n_rerun = r.n_rerun_groups = 0;
                const unsigned long long applied = r.graph_frontier && !r.graph_flat ? listed : walked;
                r.steps = applied * (unsigned long long)pl.alphabet; r.members = applied * per_alphabet;
                // (carried out for the graph's first query, on the devices that its states are of)
                const Graph& G = graphs[r.graph_id];
                const DevGraph& D = reinterpret_cast<const DevGraph*>(hb + off_graphs)[r.graph_id];
                unsigned long long judged_on = 0;
                for (size_t p = 0; p < pl.patterns.size(); ++p)
                    judged_on += (unsigned long long)pl.n_ops * (unsigned long long)(G.skeleton ? __builtin_popcountll(D.part[p]) : pl.patterns[p].g * pl.patterns[p].n_groups);
                const unsigned long long judged = G.leader == i ? gc.n_judged : 0u;
                r.evaluated = judged * (unsigned long long)pl.alphabet;
                r.evaluated_members = judged * judged_on;
                continue;
            }
            r.n_valid = hc[i].n_valid; r.n_rerun = hc[i].n_rerun; r.n_rerun_groups = hc[i].n_rerun_groups;
            r.steps = 0; r.members = 0;
            for (int t = 0; t < kCounterStripes; ++t) { r.steps += hc[i].steps[t]; r.members += hc[i].members[t]; }
            r.evaluated = 0; r.evaluated_members = 0;
            for (int t = 0; t < kCounterStripes; ++t) { r.evaluated += hc[i].evaluated[t]; r.evaluated_members += hc[i].evaluated_members[t]; }
            if (r.same_as >= 0) {                       // (the earlier query's figures; nothing was carried out for this one)
                const QueryRun& o = runs[r.same_as];
                r.n_valid = o.n_valid; r.n_rerun = o.n_rerun; r.n_rerun_groups = o.n_rerun_groups;
                r.steps = o.steps; r.members = o.members; r.off_valid = o.off_valid;
                continue;
            }
            if (r.n_valid > r.valid_cap || r.n_rerun > r.rerun_cap) {
                again = true;
                r.valid_cap = std::max(r.valid_cap, r.n_valid);
                r.rerun_cap = std::max(r.rerun_cap, r.n_rerun);
            }
        }
        if (!again) break;
        repeated = true;
        if (attempt == 3) return fail(P2_EDEVICE, "result lists kept overflowing");
    }

    // ---- frontier queries: enumeration by program size (Sec. 3.5).  Queries that agree in everything validity
    //      depends on form one enumeration; its prefixes carry the running cost sums of every member query.
    struct Enum {
        int leader = -1, id = 0;
        std::vector<int32_t> members;
        size_t off_valid = 0, off_share = 0;     // element offsets into f_rank, f_share
        uint32_t n_valid = 0, n_goal_literal = 0;
        unsigned long long flat_instr = 0;       // instructions that a walk of every candidate applies, over the alphabet's size
    };
    std::vector<Enum> enums;
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        if (!r.frontier) continue;
        const Plan& pl = r.plan;
        r.n_valid = 0; r.n_rerun = 0; r.steps = 0; r.members = 0;
        if (pl.n_candidates == 0) continue;
        int found = -1;
        for (size_t e = 0; e < enums.size() && found < 0 && share_validity; ++e) {
            const Plan& o = runs[enums[e].leader].plan;
            if (o.max_row_classes == pl.max_row_classes && o.frontier_pairs == pl.frontier_pairs &&
                runs[enums[e].leader].flat_counts == r.flat_counts && same_structure(o, pl))
                found = (int)e;
        }
        if (found < 0) { enums.emplace_back(); found = (int)enums.size() - 1; enums[found].leader = i; }
        r.enum_id = found;
        r.share_pos = (int)enums[found].members.size();
        enums[found].members.push_back(i);
    }
    if (!enums.empty()) {
        size_t n_share_all = 0;
        for (auto& E : enums) { E.off_share = n_share_all; n_share_all += E.members.size(); }
        P2_HIP(C.f_share.ensure(sizeof(int32_t) * n_share_all));
        P2_HIP(C.h_fshare.ensure(sizeof(int32_t) * n_share_all));
        for (auto& E : enums) std::memcpy(static_cast<int32_t*>(C.h_fshare.p) + E.off_share, E.members.data(), sizeof(int32_t) * E.members.size());
        P2_HIP(hipMemcpyAsync(C.f_share.p, C.h_fshare.p, sizeof(int32_t) * n_share_all, hipMemcpyHostToDevice, stream));
    }
    // ---- the enumerations, up to kFrontSlots of them side by side (a host thread and a stream each); they start
    //      once the call's stream has got here, and the call's stream goes on when they are all through
    auto run_enum = [&](Enum& E, FrontSlot& S) -> int32_t {
        const int i = E.leader;
        DevBuf& EV = C.f_evalid[E.id];
        DevBuf& EG = C.f_egsums[E.id];
        QueryRun& r = runs[i];
        const Plan& pl = r.plan;
        const int n_share = (int)E.members.size();
        const size_t sum_doubles = n_msg > 0 ? (size_t)2 * n_share : 0;      // per prefix / per goal
        const size_t step_doubles = r.flat_counts ? 2 * sum_doubles : sum_doubles;      // per child: what its step adds
        const DevQuery* dq = reinterpret_cast<const DevQuery*>(db + r.off_query);
        const size_t sw = frontier_state_words(pl.R, pl.k);
        // words of a device's (chunk set, mask) pair, and the devices that the alphabet's patterns visit per prefix
        const double pair_words = (double)((pl.k + 31) / 32 + (pl.R + 31) / 32);
        double pattern_members = 0.0;
        for (const auto& pt : pl.patterns) pattern_members += (double)pt.g * pt.n_groups;
        // state pairs per device: 2 where two planes fit in LDS; the option can lower it (1: as the compact form;
        // 4: no pair states at all, every prefix on the literal list) or, with 3, have every two-pair prefix
        // classified by the literal kernels (the path of prefixes whose groups are not aligned)
        const int fp = pl.frontier_pairs;
        const int max_pairs = fp == P2_FRONTIER_PAIRS_NONE ? 0 : fp == P2_FRONTIER_PAIRS_ONE ? 1 : frontier_max_pairs(pl.R, pl.k);
        P2_HIP(S.f_ctr.ensure(sizeof(FrontCounters)));
        P2_HIP(S.h_fctr.ensure(sizeof(FrontCounters)));
        FrontCounters* dctr = static_cast<FrontCounters*>(S.f_ctr.p);
        const FrontCounters* hctr = static_cast<const FrontCounters*>(S.h_fctr.p);
        P2_HIP(hipMemsetAsync(dctr, 0, sizeof(FrontCounters), S.stream));
        int cur = 0;
        P2_HIP(S.f_entries[cur].ensure(sizeof(FrontEntry)));
        P2_HIP(S.f_states[cur].ensure(sw * 4));
        P2_HIP(S.f_sums[cur].ensure(std::max<size_t>(sum_doubles, 1) * 8));
        P2_HIP(S.f_sid[cur].ensure(sizeof(uint32_t)));
        P2_HIP(S.f_literal[cur].ensure(sizeof(FrontEntry)));
        // A level: two lists of states (one pair per device; up to two) with n_s entries, of which the distinct ones
        // are judged; two lists of prefixes (n_c, n_c2 entries), each prefix with the index of its state; the
        // literal list (n_l prefixes that are judged from their instructions).
        uint32_t n_s[2] = {0, 0}, n_c = 0, n_c2 = 0, n_l = 0, n_l_literal = 0;      // (n_l_literal: of those, children of literal prefixes)
        bool grouped[2] = {false, false};            // the state list has been searched for equal states
        if (max_pairs >= 1) {
            P2_HIP(launch_front_init(dq, (uint32_t)i, pl.R, pl.k, static_cast<FrontEntry*>(S.f_entries[cur].p),
                                     static_cast<uint32_t*>(S.f_states[cur].p), static_cast<double*>(S.f_sums[cur].p),
                                     static_cast<uint32_t*>(S.f_sid[cur].p), (int)sum_doubles / 2, S.stream));
            n_c = 1; n_s[0] = 1;
        } else {
            const FrontEntry root{(uint32_t)i, 0u, 0ull};
            P2_HIP(hipMemcpyAsync(S.f_literal[cur].p, &root, sizeof root, hipMemcpyHostToDevice, S.stream));
            P2_HIP(hipStreamSynchronize(S.stream));
            n_l = 1;
        }
        uint32_t goals_before = 0;                   // programs of the level's length
        auto behind = [&](int len) {                 // candidates behind a prefix of len instructions and one more
            unsigned long long per = 0, power = 1;
            for (int l = len; l < pl.max_len; ++l) { per += power; power *= (unsigned long long)pl.alphabet; }
            return per;
        };
        void* gs = nullptr;
        const int handover = fp == P2_FRONTIER_PAIRS_TWO_HANDOVER ? 1 : 0;
        bool ctr_clean = true;                       // (all of the counters were cleared above)
        int len = 0;
        for (; len < pl.max_len && (n_c > 0 || n_c2 > 0 || n_l > 0); ++len) {
            const int keep = len + 1 < pl.max_len ? 1 : 0;
            size_t cap_c = std::max<size_t>(1024, ((size_t)n_c + n_c2) * pl.alphabet / 8);
            size_t cap_l = std::max<size_t>(1024, ((size_t)n_l + n_c2 / 8) * pl.alphabet / 2);
            uint32_t n_surv_l_first = 0;
            P2_HIP(S.f_unknown.ensure(std::max<size_t>(n_c2, 1) * sizeof(FrontEntry)));
            const DevBuf* list_states[2] = {&S.f_states[cur], &S.f_states2[cur]};
            // ---- one state of every group of equal states is judged against the alphabet, into a row of codes
            for (int li = 0; li < 2; ++li) {
                if (n_s[li] == 0) continue;
                P2_HIP(S.f_codes[li].ensure((size_t)n_s[li] * front_code_stride(pl.alphabet)));
                P2_HIP(S.f_unk[li].ensure(n_s[li]));
                P2_HIP(S.f_rowcnt[li].ensure((size_t)n_s[li] * sizeof(unsigned long long)));
            }
            // The literal prefixes of the level.  (On a second stream of the slot they would overlap with the pair states'
            // kernels only if that stream had a hardware queue to itself, which it would take from another slot.)
            // At the last level the goals behind a prefix that is one AllGather away from a state held in pairs are read off
            // that state (the lists of the level before are still there: the children's kernel writes no state now).
            const bool goals_from_pairs = !keep && max_pairs == 2 && len > 0 && n_l > 0;
            auto literal_prefixes = [&]() -> int32_t {
                if (n_l == 0) return P2_OK;
                P2_HIP(S.f_surv_literal.ensure(cap_l * sizeof(FrontSurvivor)));
                P2_HIP(S.spans.begin(SpanRec::kLiteral, S.stream));
                if (goals_from_pairs) {
                    P2_HIP(S.lit_scratch.ensure(std::max(front_literal_goals_scratch_bytes(pl.R, pl.k, n_l),
                                                         n_l_literal > 0 ? front_literal_scratch_bytes(pl.R, pl.k, std::max(n_l, n_c2)) : 0)));
                    P2_HIP(S.f_rest.ensure((size_t)n_l * sizeof(uint32_t)));
                    P2_HIP(launch_front_literal_goals(dq, pl.R, pl.k, static_cast<const FrontEntry*>(S.f_literal[cur].p),
                                                      static_cast<const uint32_t*>(S.f_lit_parent[cur].p), n_l, nullptr, len,
                                                      static_cast<const uint32_t*>(S.f_states[cur ^ 1].p), static_cast<const uint32_t*>(S.f_states2[cur ^ 1].p),
                                                      S.lit_scratch.p, static_cast<FrontSurvivor*>(S.f_surv_literal.p), (uint32_t)cap_l, dctr,
                                                      static_cast<uint32_t*>(S.f_rest.p), S.stream));
                }
                if (!goals_from_pairs || n_l_literal > 0) {
                    P2_HIP(S.lit_scratch.ensure(front_literal_scratch_bytes(pl.R, pl.k, std::max(n_l, n_c2))));
                    gs = S.lit_scratch.p;
                    P2_HIP(launch_front_classify_literal(dq, pl.R, pl.k, static_cast<const FrontEntry*>(S.f_literal[cur].p), n_l, len, keep ? 0 : 1,
                                                         static_cast<FrontSurvivor*>(S.f_surv_literal.p), (uint32_t)cap_l, dctr, gs,
                                                         pl.max_row_classes, goals_from_pairs ? static_cast<const uint32_t*>(S.f_rest.p) : nullptr,
                                                         goals_from_pairs ? &dctr->n_rest : nullptr, S.stream));
                }
                P2_HIP(S.spans.end(S.stream));
                return P2_OK;
            };
            // (the kernel that built the last level's children has cleared the counters of a level's first half; the
            //  kernel that brings them to the host clears those of its second half)
            if (!ctr_clean) P2_HIP(hipMemsetAsync(dctr, 0, offsetof(FrontCounters, steps), S.stream));
            ctr_clean = false;
            { const int32_t rc = literal_prefixes(); if (rc != P2_OK) return rc; }
            // At the last level only goals count: a filter first leaves the classification the few states from which an
            // instruction can still end at the goal.
            const uint32_t* cls_list[2]; const uint32_t* cls_n[2];
            for (int li = 0; li < 2; ++li) {
                cls_list[li] = grouped[li] ? static_cast<const uint32_t*>(S.f_replist[li].p) : nullptr;
                cls_n[li] = grouped[li] ? &dctr->n_reps[li] : nullptr;
            }
            if (!keep && n_s[0] + n_s[1] > 0) {
                P2_HIP(S.spans.begin(SpanRec::kGroup, S.stream));
                for (int li = 0; li < 2; ++li) {
                    if (n_s[li] == 0) continue;
                    P2_HIP(S.f_walk[li].ensure((size_t)n_s[li] * sizeof(uint32_t)));
                    P2_HIP(launch_front_goal_filter(dq, pl.R, pl.k, static_cast<const uint32_t*>(list_states[li]->p), n_s[li], cls_list[li],
                                                    cls_n[li], nullptr, li + 1, static_cast<uint8_t*>(S.f_codes[li].p), static_cast<unsigned long long*>(S.f_rowcnt[li].p),
                                                    static_cast<uint8_t*>(S.f_unk[li].p), static_cast<uint32_t*>(S.f_walk[li].p),
                                                    &dctr->n_walk[li], S.stream));
                    cls_list[li] = static_cast<const uint32_t*>(S.f_walk[li].p);
                    cls_n[li] = &dctr->n_walk[li];
                }
                P2_HIP(S.spans.end(S.stream));
            }
            if (n_s[0] + n_s[1] > 0) P2_HIP(S.spans.begin(SpanRec::kClassify, S.stream, (n_s[0] > 0) + (n_s[1] > 0)));
            for (int li = 0; li < 2; ++li)
                P2_HIP(launch_front_classify(dq, pl.R, pl.k, static_cast<const uint32_t*>(list_states[li]->p), n_s[li], cls_list[li],
                                             cls_n[li], nullptr, li + 1, max_pairs, keep ? 0 : 1, (li == 1 && handover) ? 0 : 1,
                                             static_cast<uint8_t*>(S.f_codes[li].p), static_cast<unsigned long long*>(S.f_rowcnt[li].p),
                                             static_cast<uint8_t*>(S.f_unk[li].p), dctr, S.stream));
            if (n_s[0] + n_s[1] > 0) P2_HIP(S.spans.end(S.stream));
            uint32_t walked_planes = 0, kids[3] = {0u, 0u, 0u};
            for (int attempt = 0;; ++attempt) {     // list the survivors of the prefixes; repeat with larger lists if they overflow
                P2_HIP(S.f_surv.ensure(cap_c * sizeof(FrontSurvivor)));
                if (attempt > 0) {
                    P2_HIP(hipMemsetAsync(dctr, 0, offsetof(FrontCounters, steps), S.stream));
                    // (the classification is not repeated: what it counted goes back in)
                    P2_HIP(hipMemcpyAsync(&dctr->t_count[0], kids, sizeof kids, hipMemcpyHostToDevice, S.stream));
                    const int32_t rc = literal_prefixes();
                    if (rc != P2_OK) return rc;
                }
                if (n_c + n_c2 > 0) P2_HIP(S.spans.begin(SpanRec::kGroup, S.stream));
                P2_HIP(launch_front_expand(dq, static_cast<const FrontEntry*>(S.f_entries[cur].p), n_c,
                                           static_cast<const uint32_t*>(S.f_sid[cur].p),
                                           static_cast<const uint8_t*>(S.f_codes[0].p), static_cast<const unsigned long long*>(S.f_rowcnt[0].p),
                                           static_cast<const uint8_t*>(S.f_unk[0].p), 1, 0,
                                           static_cast<FrontSurvivor*>(S.f_surv.p), (uint32_t)cap_c, nullptr, dctr, S.stream));
                P2_HIP(launch_front_expand(dq, static_cast<const FrontEntry*>(S.f_entries2[cur].p), n_c2,
                                           static_cast<const uint32_t*>(S.f_sid2[cur].p),
                                           static_cast<const uint8_t*>(S.f_codes[1].p), static_cast<const unsigned long long*>(S.f_rowcnt[1].p),
                                           static_cast<const uint8_t*>(S.f_unk[1].p), 2, handover,
                                           static_cast<FrontSurvivor*>(S.f_surv.p), (uint32_t)cap_c,
                                           static_cast<FrontEntry*>(S.f_unknown.p), dctr, S.stream));
                // (how many children the judged states have, by kind, the classification has counted)
                if (n_c + n_c2 > 0) P2_HIP(S.spans.end(S.stream));
                P2_HIP(launch_front_counters_out(static_cast<FrontCounters*>(S.h_fctr.p), dctr, S.stream));
                P2_HIP(hipStreamSynchronize(S.stream));
                if (attempt == 0) {                  // (a repeat clears the level's counters)
                    walked_planes = hctr->n_walked_planes;
                    for (int kd = 0; kd < 3; ++kd) kids[kd] = hctr->t_count[kd];
                }
                n_surv_l_first = hctr->n_surv_literal;
                if (hctr->n_unknown > 0 && hctr->n_surv_literal <= cap_l) {
                    // two-pair prefixes that this form could not judge: the literal kernels classify them from their
                    // instructions; their survivors follow those of the literal list
                    const uint32_t n_u = hctr->n_unknown;
                    P2_HIP(hipMemsetAsync(&dctr->n_overflow, 0, sizeof(uint32_t), S.stream));
                    P2_HIP(S.lit_scratch.ensure(front_literal_scratch_bytes(pl.R, pl.k, std::max(std::max(n_l, n_c2), n_u))));
                    gs = S.lit_scratch.p;
                    P2_HIP(S.spans.begin(SpanRec::kLiteral, S.stream));
                    P2_HIP(launch_front_classify_literal(dq, pl.R, pl.k, static_cast<const FrontEntry*>(S.f_unknown.p), n_u, len, keep ? 0 : 1,
                                                         static_cast<FrontSurvivor*>(S.f_surv_literal.p), (uint32_t)cap_l, dctr, gs,
                                                         pl.max_row_classes, nullptr, nullptr, S.stream));
                    P2_HIP(S.spans.end(S.stream));
                    P2_HIP(launch_front_counters_out(static_cast<FrontCounters*>(S.h_fctr.p), dctr, S.stream));
                    P2_HIP(hipStreamSynchronize(S.stream));
                }
                if ((uint32_t)hctr->surv_goal <= cap_c && hctr->n_surv_literal <= cap_l) break;
                // the repeated listing counts its steps again: take them back
                cap_c = std::max<size_t>(cap_c, (uint32_t)hctr->surv_goal); cap_l = std::max<size_t>(cap_l, (size_t)hctr->n_surv_literal * 2);
                FrontCounters fix = *hctr;
                fix.steps = r.steps; fix.members = r.members;
                P2_HIP(hipMemcpyAsync(dctr, &fix, sizeof(FrontCounters), hipMemcpyHostToDevice, S.stream));
                P2_HIP(hipStreamSynchronize(S.stream));
            }
            // The goals kernel and this function tell by rules of their own which literal prefixes are left to the literal
            // kernels; where the rules part, some are judged by neither.
            if (goals_from_pairs && hctr->n_rest != n_l_literal)
                return fail(P2_EDEVICE, "internal: " + std::to_string(hctr->n_rest) + " literal prefixes left over at the last level, " +
                                            std::to_string(n_l_literal) + " expected");
            {   // what the classification launches of this level worked on
                const double j1 = grouped[0] ? (double)hctr->n_reps[0] : (double)n_s[0], j2 = grouped[1] ? (double)hctr->n_reps[1] : (double)n_s[1];
                // (at the last level only the states from which an instruction can still end at the goal are walked)
                const double planes = keep ? j1 + 2.0 * j2 : (double)walked_planes;
                S.prof_entries += (double)n_c + n_c2;
                S.prof_prefixes += j1 + j2;
                S.prof_state_bytes += planes * pl.R * pair_words * 4.0;
                S.prof_lane_ops += planes * pattern_members * pair_words * 4.0;
            }
            // A walk applies, to every candidate that starts with a valid prefix of this length, one more instruction
            // (a program that has reached the goal is not valid with one more: every rule fails there).
            E.flat_instr += behind(len) * ((unsigned long long)n_c + n_c2 + n_l + goals_before);
            const uint32_t n_surv = (uint32_t)hctr->surv_goal, n_surv_l = hctr->n_surv_literal;
            const uint32_t n_goal_pair = (uint32_t)(hctr->surv_goal >> 32), n_goal_lit = hctr->n_goal, n_goal = n_goal_pair + n_goal_lit;
            const uint32_t n_prefix = (uint32_t)hctr->pref_pref2, n_prefix2 = (uint32_t)(hctr->pref_pref2 >> 32), n_plit = hctr->n_prefix_literal;
            const uint32_t t1 = hctr->t_count[0], t2 = hctr->t_count[1], tg = hctr->t_count[2], n_ss = t1 + t2 + tg;
            r.steps = hctr->steps; r.members = hctr->members;
            r.n_rerun += n_plit + hctr->n_unknown;
            E.n_goal_literal += n_goal_lit;
            P2_HIP(grow_keep(EV, ((size_t)E.n_valid + n_goal + 1) * sizeof(unsigned long long), (size_t)E.n_valid * sizeof(unsigned long long), S.stream));
            P2_HIP(grow_keep(EG, (((size_t)E.n_valid + n_goal) * sum_doubles + 1) * sizeof(double), (size_t)E.n_valid * sum_doubles * sizeof(double), S.stream));
            const int nxt = cur ^ 1;
            // the next level's prefixes ...
            P2_HIP(S.f_entries[nxt].ensure(std::max<size_t>(n_prefix, 1) * sizeof(FrontEntry)));
            P2_HIP(S.f_sums[nxt].ensure(std::max<size_t>((size_t)n_prefix * sum_doubles, 1) * 8));
            P2_HIP(S.f_sid[nxt].ensure(std::max<size_t>(n_prefix, 1) * sizeof(uint32_t)));
            P2_HIP(S.f_entries2[nxt].ensure(std::max<size_t>(n_prefix2, 1) * sizeof(FrontEntry)));
            P2_HIP(S.f_sums2[nxt].ensure(std::max<size_t>((size_t)n_prefix2 * sum_doubles, 1) * 8));
            P2_HIP(S.f_sid2[nxt].ensure(std::max<size_t>(n_prefix2, 1) * sizeof(uint32_t)));
            P2_HIP(S.f_literal[nxt].ensure(std::max<size_t>(n_plit, 1) * sizeof(FrontEntry)));
            P2_HIP(S.f_lit_parent[nxt].ensure(std::max<size_t>(n_plit, 1) * sizeof(uint32_t)));
            // ... and states: a child per (judged state, valid instruction), its hash, what the step
            // adds to the cost sums; where a state's children are
            P2_HIP(S.f_states[nxt].ensure(std::max<size_t>(t1, 1) * sw * 4));
            P2_HIP(S.f_states2[nxt].ensure(std::max<size_t>(t2, 1) * sw * 8));
            P2_HIP(S.f_hash[nxt].ensure(std::max<size_t>(t1, 1) * sizeof(unsigned long long)));
            P2_HIP(S.f_hash2[nxt].ensure(std::max<size_t>(t2, 1) * sizeof(unsigned long long)));
            P2_HIP(S.f_delta[0].ensure(std::max<size_t>((size_t)t1 * step_doubles, 1) * 8));
            P2_HIP(S.f_delta[1].ensure(std::max<size_t>((size_t)t2 * step_doubles, 1) * 8));
            P2_HIP(S.f_delta[2].ensure(std::max<size_t>((size_t)tg * step_doubles, 1) * 8));
            P2_HIP(S.f_ssurv.ensure(std::max<size_t>(n_ss, 1) * sizeof(FrontSurvivor)));
            for (int li = 0; li < 2; ++li) P2_HIP(S.f_childof[li].ensure(std::max<size_t>((size_t)n_s[li] * pl.alphabet, 1) * sizeof(uint32_t)));
            if (n_ss > 0) P2_HIP(S.spans.begin(SpanRec::kGroup, S.stream));
            for (int li = 0; li < 2; ++li) {
                if (li == 1 && handover) continue;
                P2_HIP(launch_front_children(dq, n_s[li], grouped[li] ? static_cast<const uint32_t*>(S.f_replist[li].p) : nullptr,
                                             grouped[li] ? &dctr->n_reps[li] : nullptr, static_cast<const uint8_t*>(S.f_codes[li].p),
                                             static_cast<const uint8_t*>(S.f_unk[li].p), li + 1, keep, 1, static_cast<uint32_t*>(S.f_childof[li].p),
                                             static_cast<FrontSurvivor*>(S.f_ssurv.p), dctr, S.stream));
            }
            if (n_ss > 0) P2_HIP(S.spans.end(S.stream));
            FrontLevel lv;
            std::memset(&lv, 0, sizeof lv);
            lv.query = (uint32_t)i;
            lv.share = static_cast<const int32_t*>(C.f_share.p) + E.off_share;
            lv.n_share = n_share; lv.n_msg = n_msg;
            lv.states1 = static_cast<const uint32_t*>(S.f_states[cur].p); lv.states2 = static_cast<const uint32_t*>(S.f_states2[cur].p);
            lv.surv = static_cast<const FrontSurvivor*>(S.f_ssurv.p); lv.n_surv = n_ss;
            lv.lds_planes = n_s[1] > 0 ? 2 : 1;
            lv.only = 0;
            lv.n_reps = &dctr->n_reps[0];
            lv.ctr = dctr;
            ctr_clean = n_ss > 0;                    // (the kernel is launched only if there are children)
            lv.next_states1 = static_cast<uint32_t*>(S.f_states[nxt].p); lv.next_states2 = static_cast<uint32_t*>(S.f_states2[nxt].p);
            lv.next_hash1 = static_cast<unsigned long long*>(S.f_hash[nxt].p); lv.next_hash2 = static_cast<unsigned long long*>(S.f_hash2[nxt].p);
            lv.delta1 = static_cast<double*>(S.f_delta[0].p); lv.delta2 = static_cast<double*>(S.f_delta[1].p);
            lv.delta_goal = static_cast<double*>(S.f_delta[2].p);
            lv.factors = r.flat_counts ? 1 : 0;
            if (n_ss > 0) P2_HIP(S.spans.begin(SpanRec::kMaterialize, S.stream));
            P2_HIP(launch_front_materialize(reinterpret_cast<const DevQuery*>(db), pl.R, pl.k, lv, S.stream));
            if (n_ss > 0) {
                P2_HIP(S.spans.end(S.stream));
                // every child reads its parent (one plane at least) and is written: state and what the step costs
                S.prof_children += (double)n_ss;
                S.prof_mat_bytes += ((double)n_ss + (double)t1 + 2.0 * t2) * pl.R * pair_words * 4.0 + (double)n_ss * (double)sum_doubles * 8.0;
            }
            // ---- the next state lists searched for equal states (hashes propose, a word-by-word comparison decides)
            const uint32_t n_next[2] = {t1, t2};
            const DevBuf* next_states[2] = {&S.f_states[nxt], &S.f_states2[nxt]};
            const DevBuf* next_hash[2] = {&S.f_hash[nxt], &S.f_hash2[nxt]};
            bool grouped_next[2] = {false, false};
            for (int li = 0; li < 2; ++li) grouped_next[li] = n_next[li] >= kGroupMin && n_next[li] < (1u << 24);
            for (int li = 0; li < 2; ++li) {
                const uint32_t n = n_next[li];
                if (!grouped_next[li]) continue;
                size_t table = 1024;
                while (table < (size_t)n * 2) table *= 2;
                P2_HIP(S.f_table.ensure(table * sizeof(unsigned long long)));
                P2_HIP(S.f_rep[li].ensure((size_t)n * sizeof(uint32_t)));
                P2_HIP(S.f_replist[li].ensure((size_t)n * sizeof(uint32_t)));
                P2_HIP(S.spans.begin(SpanRec::kGroup, S.stream));
                P2_HIP(hipMemsetAsync(S.f_table.p, 0xff, table * sizeof(unsigned long long), S.stream));
                P2_HIP(launch_front_dedup(static_cast<const uint32_t*>(next_states[li]->p), sw * (li + 1),
                                          static_cast<const unsigned long long*>(next_hash[li]->p), n,
                                          static_cast<unsigned long long*>(S.f_table.p), (uint32_t)table,
                                          static_cast<uint32_t*>(S.f_rep[li].p), static_cast<uint32_t*>(S.f_replist[li].p),
                                          &dctr->n_reps[li], S.stream));
                P2_HIP(S.spans.end(S.stream));
            }
            // ---- the next level's prefixes and this level's goals: those of the pair kernels at the places the listing
            //      gave them, then those of literal prefixes
            unsigned long long* vout = static_cast<unsigned long long*>(EV.p) + E.n_valid;
            double* gsums = static_cast<double*>(EG.p) + (size_t)E.n_valid * sum_doubles;
            unsigned long long* vout_lit = vout + n_goal_pair;
            double* gsums_lit = gsums + (size_t)n_goal_pair * sum_doubles;
            FrontPrefixes px;
            std::memset(&px, 0, sizeof px);
            px.query = (uint32_t)i; px.n_share = n_share; px.n_msg = n_msg;
            px.surv = static_cast<const FrontSurvivor*>(S.f_surv.p); px.n_surv = n_surv;
            px.parent_len = len; px.keep_prefixes = keep;
            px.entries1 = static_cast<const FrontEntry*>(S.f_entries[cur].p); px.sid1 = static_cast<const uint32_t*>(S.f_sid[cur].p);
            px.sums1 = static_cast<const double*>(S.f_sums[cur].p);
            px.entries2 = static_cast<const FrontEntry*>(S.f_entries2[cur].p); px.sid2 = static_cast<const uint32_t*>(S.f_sid2[cur].p);
            px.sums2 = static_cast<const double*>(S.f_sums2[cur].p);
            px.child_of1 = static_cast<const uint32_t*>(S.f_childof[0].p); px.child_of2 = static_cast<const uint32_t*>(S.f_childof[1].p);
            px.rep1 = grouped_next[0] ? static_cast<const uint32_t*>(S.f_rep[0].p) : nullptr;
            px.rep2 = grouped_next[1] ? static_cast<const uint32_t*>(S.f_rep[1].p) : nullptr;
            px.delta1 = lv.delta1; px.delta2 = lv.delta2; px.delta_goal = lv.delta_goal; px.factors = lv.factors;
            px.next_entries1 = static_cast<FrontEntry*>(S.f_entries[nxt].p); px.next_sid1 = static_cast<uint32_t*>(S.f_sid[nxt].p);
            px.next_sums1 = static_cast<double*>(S.f_sums[nxt].p);
            px.next_entries2 = static_cast<FrontEntry*>(S.f_entries2[nxt].p); px.next_sid2 = static_cast<uint32_t*>(S.f_sid2[nxt].p);
            px.next_sums2 = static_cast<double*>(S.f_sums2[nxt].p);
            px.next_literal = static_cast<FrontEntry*>(S.f_literal[nxt].p);
            px.next_literal_parent = static_cast<uint32_t*>(S.f_lit_parent[nxt].p);
            px.valid_out = vout; px.goal_sums = gsums; px.ctr = dctr;
            if (n_surv > 0) P2_HIP(S.spans.begin(SpanRec::kGroup, S.stream));
            P2_HIP(launch_front_prefixes(reinterpret_cast<const DevQuery*>(db), px, S.stream));
            if (n_surv > 0) P2_HIP(S.spans.end(S.stream));
            P2_HIP(launch_front_emit(dq, (uint32_t)i, static_cast<const FrontEntry*>(S.f_literal[cur].p),
                                     static_cast<const FrontSurvivor*>(S.f_surv_literal.p), n_surv_l_first, len, keep,
                                     static_cast<FrontEntry*>(S.f_literal[nxt].p), static_cast<uint32_t*>(S.f_lit_parent[nxt].p), vout_lit, gsums_lit, (int)sum_doubles / 2, dctr, S.stream));
            P2_HIP(launch_front_emit(dq, (uint32_t)i, static_cast<const FrontEntry*>(S.f_unknown.p),
                                     static_cast<const FrontSurvivor*>(S.f_surv_literal.p) + n_surv_l_first, n_surv_l - n_surv_l_first, len, keep,
                                     static_cast<FrontEntry*>(S.f_literal[nxt].p), static_cast<uint32_t*>(S.f_lit_parent[nxt].p), vout_lit, gsums_lit, (int)sum_doubles / 2, dctr, S.stream));
            E.n_valid += n_goal;
            goals_before = n_goal;
            n_c = keep ? n_prefix : 0;
            n_c2 = keep ? n_prefix2 : 0;
            n_l = keep ? n_plit : 0;
            n_l_literal = keep ? n_surv_l - n_goal_lit : 0;
            n_s[0] = keep ? t1 : 0; n_s[1] = keep ? t2 : 0;
            grouped[0] = grouped_next[0]; grouped[1] = grouped_next[1];
            cur = nxt;
        }
        E.flat_instr += behind(len) * goals_before;
        // steps of the last level
        P2_HIP(launch_copy_out(S.h_fctr.p, dctr, sizeof(FrontCounters), S.stream));
        P2_HIP(hipStreamSynchronize(S.stream));
        r.steps = hctr->steps; r.members = hctr->members;
        for (int32_t m : E.members) {        // every query of the enumeration reports its counts
            QueryRun& o = runs[m];
            o.n_valid = E.n_valid; o.n_rerun = r.n_rerun; o.steps = r.steps; o.members = r.members;
        }
        return P2_OK;
    };
    for (FrontSlot& S : C.slots) {       // (also the slots that this call leaves idle: their figures are summed below)
        S.prof_prefixes = S.prof_state_bytes = S.prof_lane_ops = S.prof_children = S.prof_mat_bytes = S.prof_entries = 0.0;
        if (n_large == 0) S.spans.reset();
    }
    for (size_t g = 0; g < graphs.size() && g_prof.on; ++g) {
        if (!graphs[g].large) continue;
        const GraphCounters& gc = static_cast<const GraphCounters*>(C.h_gctr.p)[g];
        const Plan& pl = runs[graphs[g].leader].plan;
        FrontSlot& S = C.slots[0];
        const double words = (double)((graph_rows(pl) + 31) / 32 + (pl.R + 31) / 32);
        double visited = 0.0;
        for (const Pattern& p : pl.patterns) visited += (double)p.g * p.n_groups;
        S.prof_prefixes += gc.n_judged; S.prof_entries += 1.0;
        for (int len = 1; len < pl.max_len; ++len) S.prof_entries += (double)gc.n_prefixes[len];
        S.prof_state_bytes += (double)gc.walked_planes * pl.R * words * 4.0;
        S.prof_lane_ops += (double)gc.walked_planes * visited * words * 4.0;
        S.prof_children += gc.n_children;
        S.prof_mat_bytes += ((double)gc.n_children + gc.n_child_planes) * pl.R * words * 4.0;
    }
    if (g_prof.on && n_large == 0) P2_HIP(hipEventRecord(g_prof.ev[3], stream));
    if (!enums.empty()) {
        for (size_t e = 0; e < enums.size(); ++e) enums[e].id = (int)e;
        if (C.f_evalid.size() < enums.size()) { C.f_evalid.resize(enums.size()); C.f_egsums.resize(enums.size()); }
        bool one_at_a_time = false;
        for (int i = 0; i < n_queries; ++i)
            one_at_a_time |= queries[i].opt && (queries[i].opt->flags & P2_FLAG_ONE_ENUMERATION_AT_A_TIME) != 0u;
        const int n_slots = one_at_a_time ? 1 : (int)std::min<size_t>(kFrontSlots, enums.size());
        P2_HIP(hipEventRecord(C.front_go, stream));
        if (n_slots > 1 && !C.slots[1].stream) {     // (first time: the streams are chosen by timing, on a quiet device)
            P2_HIP(hipStreamSynchronize(stream));
            P2_HIP(hipStreamSynchronize(C.copy_stream));
        }
        P2_HIP(C.open_slot_streams(n_slots));
        for (int t = 0; t < n_slots; ++t) {
            FrontSlot& S = C.slots[t];
            P2_HIP(hipStreamWaitEvent(S.stream, C.front_go, 0));
            S.spans.on = g_prof.on; S.spans.kernels_only = g_prof.kernels_only;
            S.rc = P2_OK; S.err.clear();
        }
        // the long chains first: large reduction groups, large alphabets
        std::vector<int> order(enums.size());
        for (size_t e = 0; e < enums.size(); ++e) order[e] = (int)e;
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
            const Plan& px = runs[enums[x].leader].plan; const Plan& py = runs[enums[y].leader].plan;
            if (px.R != py.R) return px.R > py.R;
            return px.alphabet > py.alphabet;
        });
        std::atomic<size_t> next{0};
        int device = 0;
        P2_HIP(hipGetDevice(&device));
        auto work = [&](int t, bool own_thread) {
            FrontSlot& S = C.slots[t];
            if (own_thread && hipSetDevice(device) != hipSuccess) { S.rc = P2_EDEVICE; S.err = "hipSetDevice failed in a worker thread"; return; }
            for (size_t at = next.fetch_add(1); at < order.size(); at = next.fetch_add(1)) {
                const int32_t rc = run_enum(enums[order[at]], S);
                if (rc != P2_OK) { S.rc = rc; S.err = g_err; break; }
            }
            // (whatever the slot has queued is waited for, also after a failure: its buffers are reused)
            (void)hipStreamSynchronize(S.stream);
        };
        if (n_slots == 1) {
            work(0, false);
        } else {
            std::vector<std::thread> pool;
            for (int t = 1; t < n_slots; ++t) pool.emplace_back(work, t, true);
            work(0, false);
            for (auto& th : pool) th.join();
        }
        for (int t = 0; t < n_slots; ++t)
            if (C.slots[t].rc != P2_OK) return fail(C.slots[t].rc, C.slots[t].err);
    }

    if (g_prof.on) {
        if (n_large == 0 || !enums.empty()) P2_HIP(hipEventRecord(g_prof.ev[4], stream));
        P2_HIP(hipEventRecord(g_prof.ev[5], stream));
        p2_profile& L = g_prof.last;
        L.front_prefixes = L.front_classify_state_bytes = L.front_classify_lane_ops = L.front_survivors = 0.0;
        L.front_materialize_bytes = L.front_entries = 0.0;
        for (const FrontSlot& S : C.slots) {
            L.front_prefixes += S.prof_prefixes; L.front_classify_state_bytes += S.prof_state_bytes;
            L.front_classify_lane_ops += S.prof_lane_ops; L.front_survivors += S.prof_children;
            L.front_materialize_bytes += S.prof_mat_bytes; L.front_entries += S.prof_entries;
        }
    }

    // ---- order, cost, select
    size_t total_valid = 0;
    for (auto& r : runs) { r.out_first = total_valid; total_valid += r.n_valid; }
    const size_t nm = (size_t)std::max(n_msg, 1);
    // rows the caller gets; without room for them (the sizing call with cap = 0) only the counts are returned,
    // and nothing is ordered, costed or selected
    int64_t need = 0;
    for (auto& r : runs) need += r.topk > 0 ? (int64_t)n_msg * (int64_t)std::min<size_t>(r.topk, r.n_valid) : (int64_t)r.n_valid;
    const bool store = cap >= need && cap > 0;
    // (every query with valid programs asks for a shortlist: only the rows that are picked go back to the host)
    bool only_shortlists = n_msg > 0;
    for (const auto& r : runs) only_shortlists = only_shortlists && (r.n_valid == 0 || r.topk > 0);
    size_t pos_off = 0;
    direct = direct && store && total_valid <= rows_room;       // (the rows are in host memory already)
    for (const QueryRun& r : runs) shortlists = shortlists && (!r.graph || r.n_valid <= most_valid(r.plan));      // (else as if it had not been tried)
    if (shortlists) {
        const uint32_t* trouble = static_cast<const uint32_t*>(C.h_pos.p);
        for (int i = 0; i < n_queries; ++i) {
            uint32_t t = 0;
            for (int m = 0; m < n_msg && runs[i].graph; ++m) t |= *trouble++;
            if (t & 1u) return fail(P2_EINVAL, "query " + std::to_string(i) + ": NaN cost (a message size that is not finite?)");
            if (t != 0u) return fail(P2_EDEVICE, "top-k returned a bad position");
        }
    }
    if (store && !direct && !shortlists) {
    P2_HIP(C.sorted.ensure(sizeof(unsigned long long) * std::max<size_t>(total_valid, 1)));
    P2_HIP(C.progs.ensure(sizeof(p2_program) * std::max<size_t>(total_valid, 1)));
    P2_HIP(C.costs.ensure(sizeof(double) * std::max<size_t>(total_valid, 1) * nm));
    size_t topk_rows = 0, topk_scratch = 0;
    for (auto& r : runs)
        if (r.topk > 0 && r.n_valid > 0) {
            topk_rows += (size_t)n_msg * std::min<size_t>(r.topk, r.n_valid);
            if (r.n_valid > kTopkJobMax) topk_scratch = std::max(topk_scratch, topk_scratch_bytes(r.n_valid, r.topk));
        }
    P2_HIP(C.topk_pos.ensure(sizeof(long long) * std::max<size_t>(topk_rows, 1)));
    P2_HIP(C.topk_scratch.ensure(std::max<size_t>(topk_scratch, 256)));
    int post_launches = 0;
    std::vector<DevTopkJob> topk_jobs, topk_big;          // a block each; long lists, all blocks for one after the other
    int topk_jobs_k = 0;
    long long topk_jobs_n = 0;
    // ordering and costing: one launch per kernel and state-size class
    std::vector<PostLaunch> sort_launches, ccost_launches, scost_launches, lcost_launches;
    std::vector<GraphRows> graph_rows_of;
    unsigned graph_row_blocks = 0;
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        if (r.n_valid == 0) continue;
        if (r.graph && only_graphs) continue;            // (one after the other, as the counts on the device say)
        if (r.graph) {                                   // (the rows come out in order and costed)
            graph_rows_of.push_back(GraphRows{graph_row_blocks, (uint32_t)i, (uint32_t)r.graph_id, (uint32_t)r.graph_pos, r.n_valid, fused_sums(r),
                                              (unsigned long long)r.out_first});
            graph_row_blocks += (r.n_valid + 255u) / 256u;
            continue;
        }
        if (r.frontier) {
            // ordered and costed from the enumeration's sums (below); programs that came from literal prefixes
            // have no sums and are costed by the literal kernel
            const bool lit_cost = enums[r.enum_id].n_goal_literal > 0 && n_msg > 0;
            if (lit_cost && literal_lds_bytes(r.plan.R, r.plan.k) != 0)
                add_seg(lcost_launches, mask_class(r.plan.R) * 2 + 1, r.plan, i, r.n_valid, 1, 0, r.out_first);
            continue;
        }
        const size_t list_at = r.off_valid;
        if (r.wave_cost) {
            // one wavefront per program; it also finds the program's place in the ascending order
            add_seg(scost_launches, word_class(r.plan.k) * 100 + word_class(r.plan.R), r.plan, i, r.n_valid, 1, list_at,
                    r.out_first);
        } else {
            add_seg(sort_launches, 0, r.plan, i, r.n_valid, 256, list_at, r.out_first);
        }
        if (r.wave_cost) {
        } else if (r.engine == P2_ENGINE_COMPACT) {
            const int cls = word_class(r.plan.k) * 100 + word_class(r.plan.R);
            add_seg(ccost_launches, cls, r.plan, i, r.n_valid, 1, 0, r.out_first);     // per_block set below
        }
        const bool lit_cost = r.engine == P2_ENGINE_LITERAL || (r.n_rerun > 0 && n_msg > 0);
        if (lit_cost && literal_lds_bytes(r.plan.R, r.plan.k) != 0)
            add_seg(lcost_launches, mask_class(r.plan.R) * 2 + (r.engine == P2_ENGINE_COMPACT ? 1 : 0), r.plan, i, r.n_valid, 1, 0,
                    r.out_first);
    }
    for (auto& L : ccost_launches) {      // a block of the compact cost kernel takes as many entries as it has lanes
        // (one, with the lanes sharing the work, where only a few states fit in LDS)
        const uint32_t lanes = cost_wide_applies(L.max_R, L.max_k) ? 1u : (uint32_t)compact_lanes(L.max_R, L.max_k);
        L.blocks = 0;
        for (auto& sg : L.segs) { sg.per_block = lanes; sg.first_block = L.blocks; L.blocks += (sg.count + lanes - 1) / lanes; }
    }
    P2_HIP(upload_segs({&sort_launches, &ccost_launches, &scost_launches, &lcost_launches}));
    unsigned long long* sorted_base = static_cast<unsigned long long*>(C.sorted.p);
    p2_program* progs_base = static_cast<p2_program*>(C.progs.p);
    double* costs_base = static_cast<double*>(C.costs.p);
    for (auto& L : sort_launches) {
        ++post_launches;
        P2_HIP(launch_rank_sort(static_cast<unsigned long long*>(C.valid.p), nullptr, sorted_base,
                                segs_of(L), (int)L.segs.size(), L.blocks, stream));
    }
    // the compact engine costs what it can hold and marks the rest with NaN for the literal engine
    for (auto& L : ccost_launches) {
        ++post_launches;
        if (cost_wide_applies(L.max_R, L.max_k))
            P2_HIP(launch_cost_wide_list(reinterpret_cast<const DevQuery*>(db), segs_of(L), (int)L.segs.size(), L.blocks, L.max_R,
                                         L.max_k, sorted_base, progs_base, costs_base, stream));
        else
            P2_HIP(launch_cost_compact_list(reinterpret_cast<const DevQuery*>(db), segs_of(L), (int)L.segs.size(), L.blocks, L.max_R,
                                            L.max_k, sorted_base, progs_base, costs_base, stream));
    }
    for (auto& L : scost_launches) {
        ++post_launches;
        P2_HIP(launch_cost_shared(reinterpret_cast<const DevQuery*>(db), segs_of(L), (int)L.segs.size(), L.blocks, L.max_R,
                                  L.max_k, static_cast<unsigned long long*>(C.valid.p), nullptr,
                                  sorted_base, progs_base, costs_base, stream));
    }
    if (only_graphs && total_valid > 0) {
        size_t blocks = 0;
        for (const QueryRun& r : runs) blocks += (r.n_valid + 255u) / 256u;
        ++post_launches;
        P2_HIP(launch_graph_emit(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const DevGraph*>(db + off_graphs),
                                 static_cast<const GraphCounters*>(C.g_zero.p), reinterpret_cast<const GraphQuery*>(db + off_gasked), n_queries,
                                 nullptr, 0, (unsigned)blocks, total_valid, sorted_base, progs_base, costs_base, nullptr, 0, nullptr, stream));
    }
    if (!graph_rows_of.empty()) {
        const size_t bytes = sizeof(GraphRows) * graph_rows_of.size();
        P2_HIP(C.g_rows.ensure(bytes));
        P2_HIP(C.h_grows.ensure(bytes));
        std::memcpy(C.h_grows.p, graph_rows_of.data(), bytes);
        P2_HIP(hipMemcpyAsync(C.g_rows.p, C.h_grows.p, bytes, hipMemcpyHostToDevice, stream));
        ++post_launches;
        P2_HIP(launch_graph_emit(reinterpret_cast<const DevQuery*>(db), reinterpret_cast<const DevGraph*>(db + off_graphs),
                                 nullptr, nullptr, 0, static_cast<const GraphRows*>(C.g_rows.p), (int)graph_rows_of.size(), graph_row_blocks,
                                 total_valid, sorted_base, progs_base, costs_base, nullptr, 0, nullptr, stream));
    }
    // frontier enumerations: the place of every program in ascending index order, once per enumeration; then
    // every query of the enumeration writes its rows (programs, and costs from its own sums)
    if (!enums.empty()) {
        size_t ranked = 0;
        size_t most = 0;
        for (auto& E : enums) { E.off_valid = ranked; ranked += E.n_valid; most = std::max<size_t>(most, E.n_valid); }
        P2_HIP(C.f_rank.ensure(sizeof(uint32_t) * std::max<size_t>(ranked, 1)));
        P2_HIP(C.f_rank_runs.ensure(sizeof(unsigned long long) * std::max<size_t>(most, 1)));
        std::vector<FrontFinish> jobs;
        uint32_t max_valid = 0;
        for (auto& E : enums) {
            if (E.n_valid == 0) continue;
            const unsigned long long* list = static_cast<const unsigned long long*>(C.f_evalid[E.id].p);
            uint32_t* rank = static_cast<uint32_t*>(C.f_rank.p) + E.off_valid;
            // (a query that asks for the cheapest programs only has them selected by (cost, index): its rows need no order)
            bool ordered = false;
            for (int32_t m : E.members) ordered |= runs[m].topk == 0;
            if (ordered) {
                post_launches += front_rank_launches(E.n_valid);
                P2_HIP(launch_front_rank(list, E.n_valid, static_cast<unsigned long long*>(C.f_rank_runs.p), rank, stream));
            }
            for (size_t m = 0; m < E.members.size(); ++m) {
                FrontFinish F;
                std::memset(&F, 0, sizeof F);
                F.query = (uint32_t)E.members[m]; F.n_share = (int32_t)E.members.size(); F.share_pos = (int32_t)m;
                F.n_valid = E.n_valid; F.valid = list; F.rank = runs[E.members[m]].topk == 0 ? rank : nullptr;
                F.goal_sums = static_cast<const double*>(C.f_egsums[E.id].p);
                F.out_first = runs[E.members[m]].out_first;
                F.sorted = sorted_base; F.progs = progs_base; F.costs = costs_base;
                jobs.push_back(F);
                max_valid = std::max(max_valid, E.n_valid);
            }
        }
        if (!jobs.empty()) {                        // the rows of all of them in one launch
            P2_HIP(C.f_finish.ensure(sizeof(FrontFinish) * jobs.size()));
            P2_HIP(C.h_finish.ensure(sizeof(FrontFinish) * jobs.size()));
            std::memcpy(C.h_finish.p, jobs.data(), sizeof(FrontFinish) * jobs.size());
            P2_HIP(hipMemcpyAsync(C.f_finish.p, C.h_finish.p, sizeof(FrontFinish) * jobs.size(), hipMemcpyHostToDevice, stream));
            ++post_launches;
            P2_HIP(launch_front_finish(reinterpret_cast<const DevQuery*>(db), static_cast<const FrontFinish*>(C.f_finish.p),
                                       (uint32_t)jobs.size(), max_valid, stream));
        }
    }
    for (auto& L : lcost_launches) {
        ++post_launches;
        P2_HIP(launch_cost_literal_list(reinterpret_cast<const DevQuery*>(db), segs_of(L), (int)L.segs.size(), L.blocks, L.max_R,
                                        L.lit_lds, sorted_base, progs_base, costs_base, L.cls & 1, stream));
    }
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        if (r.n_valid == 0) continue;
        const DevQuery* dq = reinterpret_cast<const DevQuery*>(db + r.off_query);
        unsigned long long* sorted = sorted_base + r.out_first;
        p2_program* progs = progs_base + r.out_first;
        double* costs = costs_base + r.out_first * nm;
        const bool lit_cost = r.graph ? false : r.frontier ? (enums[r.enum_id].n_goal_literal > 0 && n_msg > 0)
                                         : (r.engine == P2_ENGINE_LITERAL || (r.n_rerun > 0 && n_msg > 0));
        if (lit_cost && literal_lds_bytes(r.plan.R, r.plan.k) == 0) {      // literal state too large for LDS
            void* gs = nullptr;
            P2_HIP(lit_scratch(r.plan, &gs));
            ++post_launches;
            P2_HIP(launch_cost_literal(dq, r.plan.R, r.plan.k, sorted, r.n_valid, progs, costs,
                                       r.engine == P2_ENGINE_COMPACT ? 1 : 0, gs, stream));
        }
        if (r.topk > 0) {
            const size_t kk = std::min<size_t>(r.topk, r.n_valid);
            for (int m = 0; m < n_msg; ++m) {
                DevTopkJob J;
                std::memset(&J, 0, sizeof J);
                J.cost = costs + m; J.index = sorted; J.out_pos = static_cast<long long*>(C.topk_pos.p) + pos_off;
                J.nan_flag = only_graphs ? reinterpret_cast<uint32_t*>(static_cast<char*>(C.g_zero.p) + graph_nan) + i
                                         : &static_cast<DevCounters*>(C.counters.p)[i].nan_seen;
                J.n = (long long)r.n_valid; J.stride = n_msg; J.k = r.topk;
                pos_off += kk;
                if (r.n_valid <= kTopkJobMax) {            // one launch for all of them, below
                    topk_jobs.push_back(J);
                    topk_jobs_k = std::max(topk_jobs_k, r.topk);
                    topk_jobs_n = std::max(topk_jobs_n, J.n);
                } else {
                    topk_big.push_back(J);
                }
            }
        }
    }
    std::vector<DevGatherSeg> gather_segs;               // (shortlists only: which rows go back)
    if (only_shortlists) {
        size_t at = 0;
        for (int i = 0; i < n_queries; ++i) {
            const QueryRun& r = runs[i];
            if (r.n_valid == 0) continue;
            const size_t rows = (size_t)n_msg * std::min<size_t>(r.topk, r.n_valid);
            gather_segs.push_back(DevGatherSeg{(unsigned long long)r.out_first, (unsigned long long)at, (uint32_t)rows, 0u});
            at += rows;
        }
    }
    {
        const size_t job_bytes = sizeof(DevTopkJob) * topk_jobs.size(), seg_bytes = sizeof(DevGatherSeg) * gather_segs.size();
        P2_HIP(C.topk_jobs.ensure(job_bytes));
        P2_HIP(C.h_topk_jobs.ensure(job_bytes));
        P2_HIP(C.gather.ensure(seg_bytes));
        P2_HIP(C.h_gather.ensure(seg_bytes));
        if (job_bytes > 0) std::memcpy(C.h_topk_jobs.p, topk_jobs.data(), job_bytes);
        if (seg_bytes > 0) std::memcpy(C.h_gather.p, gather_segs.data(), seg_bytes);
        const CopyPart in[2] = {{C.topk_jobs.p, C.h_topk_jobs.p, job_bytes}, {C.gather.p, C.h_gather.p, seg_bytes}};
        P2_HIP(launch_copies(in, 2, stream));
    }
    if (!topk_jobs.empty()) {
        ++post_launches;
        P2_HIP(launch_topk_jobs(static_cast<const DevTopkJob*>(C.topk_jobs.p), (unsigned)topk_jobs.size(), topk_jobs_k, topk_jobs_n, stream));
    }
    if (!topk_big.empty()) {
        P2_HIP(C.open_topk_control(stream));
        C.topk_control_clear = false;
        for (const DevTopkJob& J : topk_big) {
            ++post_launches;
            P2_HIP(launch_topk(J.cost, J.stride, J.index, J.n, J.k, J.out_pos, C.topk_scratch.p, C.topk_control.p, J.nan_flag, stream));
        }
    }
    if (g_prof.on) { P2_HIP(hipEventRecord(g_prof.ev[2], stream)); g_prof.last.post_launches = post_launches; }
    P2_HIP(C.h_pos.ensure(sizeof(long long) * std::max<size_t>(topk_rows, 1)));
    if (only_shortlists) {
        // every query asks for a shortlist: the rows that were picked are gathered on the device, and only they go back
        P2_HIP(C.sel_progs.ensure(sizeof(p2_program) * std::max<size_t>(topk_rows, 1)));
        P2_HIP(C.sel_costs.ensure(sizeof(double) * std::max<size_t>(topk_rows, 1) * nm));
        P2_HIP(C.h_progs.ensure(sizeof(p2_program) * std::max<size_t>(topk_rows, 1)));
        P2_HIP(C.h_costs.ensure(sizeof(double) * std::max<size_t>(topk_rows, 1) * nm));
        if (!gather_segs.empty())
            P2_HIP(launch_gather_rows(static_cast<const DevGatherSeg*>(C.gather.p), (unsigned)gather_segs.size(), progs_base, costs_base, n_msg,
                                      static_cast<const long long*>(C.topk_pos.p), static_cast<p2_program*>(C.sel_progs.p),
                                      static_cast<double*>(C.sel_costs.p), stream));
    } else {
        P2_HIP(C.h_progs.ensure(sizeof(p2_program) * std::max<size_t>(total_valid, 1)));
        P2_HIP(C.h_costs.ensure(sizeof(double) * std::max<size_t>(total_valid, 1) * nm));
    }
    {   // (the selections flag a NaN cost in their query's counters)
        const size_t rows = only_shortlists ? topk_rows : total_valid;
        const CopyPart back[4] = {{C.h_progs.p, only_shortlists ? C.sel_progs.p : C.progs.p, sizeof(p2_program) * rows},
                                 {C.h_costs.p, only_shortlists ? C.sel_costs.p : C.costs.p, n_msg > 0 ? sizeof(double) * rows * nm : 0},
                                 {C.h_pos.p, C.topk_pos.p, sizeof(long long) * topk_rows},
                                 {only_graphs ? C.h_gctr.p : C.h_counters.p, only_graphs ? C.g_zero.p : C.counters.p,
                                  topk_rows == 0 ? 0 : only_graphs ? graph_back : sizeof(DevCounters) * (size_t)n_queries}};
        P2_HIP(launch_copies(back, 4, stream));
    }
    P2_HIP(hipStreamSynchronize(stream));
    if (!topk_big.empty()) C.topk_control_clear = true;      // (only now have the kernels run to their end)
    if (topk_rows > 0) {
        const DevCounters* hc = static_cast<const DevCounters*>(C.h_counters.p);
        const uint32_t* gn = reinterpret_cast<const uint32_t*>(static_cast<const char*>(C.h_gctr.p) + graph_nan);
        for (int i = 0; i < n_queries; ++i)
            if (runs[i].topk > 0 && runs[i].n_valid > 0 && (only_graphs ? gn[i] : hc[i].nan_seen))
                return fail(P2_EINVAL, "query " + std::to_string(i) + ": NaN cost (a message size that is not finite?)");
    }
    }  // store

    if (g_prof.on) {
        P2_HIP(hipEventElapsedTime(&g_prof.last.eval_ms, g_prof.ev[0], g_prof.ev[1]));
        g_prof.last.post_ms = 0.0f;
        if (store) P2_HIP(hipEventElapsedTime(&g_prof.last.post_ms, direct || shortlists ? g_prof.ev[1] : g_prof.ev[5], g_prof.ev[2]));
        P2_HIP(hipEventSynchronize(g_prof.ev[4]));      // (a call that only sizes its result has not waited since)
        P2_HIP(hipEventElapsedTime(&g_prof.last.front_ms, g_prof.ev[3], g_prof.ev[4]));
        float ms[SpanRec::kKinds] = {0.f, 0.f, 0.f, 0.f};
        int32_t launches[SpanRec::kKinds] = {0, 0, 0, 0};
        for (FrontSlot& S : C.slots) P2_HIP(S.spans.collect(ms, launches));
        g_prof.last.front_classify_ms = ms[SpanRec::kClassify]; g_prof.last.front_classify_launches = launches[SpanRec::kClassify];
        g_prof.last.front_literal_ms = ms[SpanRec::kLiteral]; g_prof.last.front_literal_launches = launches[SpanRec::kLiteral];
        g_prof.last.front_materialize_ms = ms[SpanRec::kMaterialize]; g_prof.last.front_materialize_launches = launches[SpanRec::kMaterialize];
        g_prof.last.front_group_ms = ms[SpanRec::kGroup];
    }
    // ---- hand the results over
    const p2_program* hp = static_cast<const p2_program*>(C.h_progs.p);
    const double* hcst = static_cast<const double*>(C.h_costs.p);
    const long long* hpos = static_cast<const long long*>(C.h_pos.p);
    int64_t w = 0;
    pos_off = 0;
    size_t short_at = 0;                                 // (a shortlist has the place of its query's largest)
    for (int i = 0; i < n_queries; ++i) {
        QueryRun& r = runs[i];
        out_offset[i] = w;
        if (r.topk > 0) {
            const size_t kk = std::min<size_t>(r.topk, r.n_valid);
            if (!store) w += (int64_t)n_msg * (int64_t)kk;
            for (int m = 0; m < n_msg && store; ++m, short_at += r.graph ? shortlist_rows_of(r.plan, r.topk, 1) : 0)
                for (size_t t = 0; t < kk; ++t, ++w) {
                    const size_t sel = pos_off;
                    if (shortlists) {
                        out_prog[w] = hp[short_at + t];
                        for (int c = 0; c < n_msg; ++c) out_cost[w * n_msg + c] = hcst[(short_at + t) * nm + c];
                        continue;
                    }
                    const long long pos = hpos[pos_off++];
                    if (pos < 0 || pos >= (long long)r.n_valid) return fail(P2_EDEVICE, "top-k returned a bad position");
                    const size_t row = only_shortlists ? sel : r.out_first + (size_t)pos;
                    out_prog[w] = hp[row];
                    for (int c = 0; c < n_msg; ++c) out_cost[w * n_msg + c] = hcst[row * nm + c];
                }
        } else {
            if (store) {
                std::memcpy(out_prog + w, hp + r.out_first, sizeof(p2_program) * r.n_valid);
                if (n_msg > 0) std::memcpy(out_cost + w * n_msg, hcst + r.out_first * nm, sizeof(double) * r.n_valid * nm);
            }
            w += r.n_valid;
        }
        if (stats) {
            p2_stats& s = stats[i];
            s.candidates = r.plan.n_candidates; s.steps_executed = r.steps; s.member_visits = r.members;
            s.literal_reruns = r.shared ? (uint64_t)r.n_rerun_groups * (uint64_t)r.plan.alphabet : r.n_rerun;
            s.steps_evaluated = r.shared || r.graph ? r.evaluated : r.steps;
            s.members_evaluated = r.shared || r.graph ? r.evaluated_members : r.members;
            if (r.flat_counts && r.enum_id >= 0) {
                unsigned long long per_alphabet = 0;
                for (const Pattern& p : r.plan.patterns) per_alphabet += (unsigned long long)p.g * p.n_groups * r.plan.n_ops;
                s.steps_executed = enums[r.enum_id].flat_instr * (unsigned long long)r.plan.alphabet;
                s.member_visits = enums[r.enum_id].flat_instr * per_alphabet;
            }
            s.valid = r.n_valid; s.group_size = r.plan.R; s.n_patterns = (int32_t)r.plan.patterns.size();
            s.evaluated_with = r.graph ? (graphs[r.graph_id].leader != i ? graphs[r.graph_id].leader : -1) : r.frontier ? (r.enum_id >= 0 && enums[r.enum_id].leader != i ? enums[r.enum_id].leader : -1) : r.same_as;
            s.route = (r.graph ? P2_ROUTE_GRAPH : 0) | (left[i] ? P2_ROUTE_GRAPH_LEFT : 0) | (repeated ? P2_ROUTE_REPEATED : 0) |
                      (wanted_direct && store && !direct ? P2_ROUTE_ROWS_LATER : 0);
            s.alphabet = r.plan.alphabet; s.engine = r.frontier || r.graph_frontier ? P2_ENGINE_FRONTIER : r.shared ? P2_ENGINE_SHARED : r.regs ? P2_ENGINE_SMALL : r.engine;
        }
    }
    out_offset[n_queries] = w;
    g_prof.last.host_total_ms = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    if (!store && need > 0) return fail(P2_ENOSPC, "output buffer too small: " + std::to_string(need) + " rows needed");
    return P2_OK;
}

int32_t run_batch(const p2_query* queries, int32_t n_queries, const double* msg_bytes, int32_t n_msg,
                  p2_program* out_prog, double* out_cost, int64_t cap, int64_t* out_offset, p2_stats* stats) {
    std::vector<char> left((size_t)std::max(n_queries, 0), 0);
    int32_t rc;
    do rc = run_batch_on(queries, n_queries, msg_bytes, n_msg, out_prog, out_cost, cap, out_offset, stats, left);
    while (rc == kWithoutGraphs);                        // (every time without a graph more)
    return rc;
}

}  // namespace

extern "C" {

const char* p2_last_error(void) { return g_err.c_str(); }

int32_t p2_set_profiling(int32_t on) {
    if (on && !g_prof.ev[0])
        for (auto& e : g_prof.ev) P2_HIP(hipEventCreate(&e));
    g_prof.on = on != 0;
    g_prof.kernels_only = on == 2;
    return P2_OK;
}
int32_t p2_get_profile(p2_profile* out) {
    if (!out) return fail(P2_EINVAL, "null argument");
    *out = g_prof.last;
    return P2_OK;
}

int32_t p2_release_thread(void) {
    g_ctx.release();
    g_prof.release();
    return P2_OK;
}

int32_t p2_measure_alu_peak(int32_t reps, double* out_lane_ops_per_s, void* hip_stream) {
    if (!out_lane_ops_per_s || reps < 1 || reps > 100) return fail(P2_EINVAL, "bad arguments");
    P2_HIP(p2::measure_alu_peak(reps, out_lane_ops_per_s, (hipStream_t)hip_stream));
    return P2_OK;
}

int32_t p2_measure_lds_peak(int32_t reps, double* out_bytes_per_s, void* hip_stream) {
    if (!out_bytes_per_s || reps < 1 || reps > 100) return fail(P2_EINVAL, "bad arguments");
    P2_HIP(p2::measure_lds_peak(reps, out_bytes_per_s, (hipStream_t)hip_stream));
    return P2_OK;
}

int32_t p2_enumerate_placements(const p2_hierarchy* h, const int32_t* axes, int32_t n_axes, int32_t* out, int64_t cap,
                                int64_t* out_count) {
    std::string err;
    int32_t st = p2::enumerate_placements(h, axes, n_axes, out, cap, out_count, err);
    if (st != P2_OK) g_err = err;
    return st;
}

int32_t p2_synthesize_batch(const p2_query* queries, int32_t n_queries, const double* msg_bytes, int32_t n_msg,
                            p2_program* out_prog, double* out_cost, int64_t cap, int64_t* out_offset, p2_stats* stats) {
    try {
        return run_batch(queries, n_queries, msg_bytes, n_msg, out_prog, out_cost, cap, out_offset, stats);
    } catch (const std::exception& e) {
        return fail(P2_EDEVICE, std::string("host failure: ") + e.what());
    }
}

int32_t p2_synthesize(const p2_hierarchy* h, const int32_t* axes, int32_t n_axes, const int32_t* placement,
                      const int32_t* reduce_axes, int32_t n_reduce, int32_t max_len, const double* msg_bytes, int32_t n_msg,
                      const p2_options* opt, p2_program* out_prog, double* out_cost, int64_t cap, int64_t* out_count,
                      uint64_t* out_candidates_evaluated, p2_stats* stats) {
    if (!out_count) return fail(P2_EINVAL, "out_count is null");
    p2_query q{h, axes, n_axes, placement, reduce_axes, n_reduce, max_len, opt};
    int64_t offs[2] = {0, 0};
    p2_stats st;
    std::memset(&st, 0, sizeof st);
    int32_t rc = p2_synthesize_batch(&q, 1, msg_bytes, n_msg, out_prog, out_cost, cap, offs, &st);
    if (rc == P2_OK || rc == P2_ENOSPC) {
        *out_count = offs[1];
        if (out_candidates_evaluated) *out_candidates_evaluated = st.candidates;
        if (stats) *stats = st;
    }
    return rc;
}

int32_t p2_search_placements(const p2_hierarchy* h, const int32_t* axes, int32_t n_axes, const int32_t* reduce_sets,
                             const int32_t* reduce_set_len, int32_t n_sets, const double* weights, int32_t max_len,
                             double msg_bytes, const p2_options* opt, int32_t* out_placements, p2_search_row* out_rows,
                             double* out_total, int32_t* out_order, int64_t cap, int64_t* out_count) {
    try {
        if (!h || !axes || !reduce_sets || !reduce_set_len || !out_count) return fail(P2_EINVAL, "null argument");
        if (n_sets < 1) return fail(P2_EINVAL, "no reduction requested");
        if (cap < 0 || (cap > 0 && (!out_placements || !out_rows || !out_total || !out_order)))
            return fail(P2_EINVAL, "bad output buffer");
        if (!(msg_bytes >= 0.0)) return fail(P2_EINVAL, "msg_bytes is negative or NaN");
        if (opt && opt->hierarchy != P2_HIERARCHY_COLLAPSED)
            return fail(P2_EUNSUPPORTED, "the placement search synthesizes on the collapsed hierarchy");
        std::vector<const int32_t*> set_ptr((size_t)n_sets);
        {
            const int32_t* at = reduce_sets;
            for (int s = 0; s < n_sets; ++s) {
                if (reduce_set_len[s] < 1) return fail(P2_EINVAL, "empty set of reduce axes");
                set_ptr[(size_t)s] = at;
                at += reduce_set_len[s];
            }
        }
        int64_t n_pl = 0;
        std::string err;
        int32_t st = p2::enumerate_placements(h, axes, n_axes, nullptr, 0, &n_pl, err);
        if (st != P2_OK) return fail(st, err);
        *out_count = n_pl;
        if (cap == 0) return P2_OK;
        if (cap < n_pl) return fail(P2_ENOSPC, "output buffers too small: " + std::to_string(n_pl) + " placements");
        const size_t per = (size_t)n_axes * (size_t)h->n_levels;
        st = p2::enumerate_placements(h, axes, n_axes, out_placements, n_pl, &n_pl, err);
        if (st != P2_OK) return fail(st, err);
        if (n_pl * (int64_t)n_sets * 2 > 0x7fffffff) return fail(P2_EUNSUPPORTED, "too many (placement, reduction) pairs");

        // two queries per (placement, reduction): the search itself, keeping its cheapest program,
        // and the one-instruction AllReduce over the whole reduction group
        p2_options main_opt;
        std::memset(&main_opt, 0, sizeof main_opt);
        if (opt) main_opt = *opt;
        main_opt.topk = 1;
        p2_options base_opt = main_opt;
        base_opt.form_mask = 1; base_opt.op_mask = 1;
        // (a list of one program, asked for as a shortlist like the others unless its cost may be no number, which a selection refuses: a
        //  size without end over links that take no time, or no bytes over links that take for ever)
        base_opt.topk = msg_bytes > 0.0 && std::isfinite(msg_bytes) ? 1 : 0;
        base_opt.engine = P2_ENGINE_AUTO;
        const int n_q = (int)(n_pl * n_sets * 2);
        std::vector<p2_query> qs((size_t)n_q);
        for (int64_t p = 0; p < n_pl; ++p)
            for (int s = 0; s < n_sets; ++s) {
                const size_t at = ((size_t)p * (size_t)n_sets + (size_t)s) * 2;
                qs[at] = p2_query{h, axes, n_axes, out_placements + (size_t)p * per, set_ptr[(size_t)s], reduce_set_len[s], max_len, &main_opt};
                qs[at + 1] = p2_query{h, axes, n_axes, out_placements + (size_t)p * per, set_ptr[(size_t)s], reduce_set_len[s], 1, &base_opt};
            }
        std::vector<p2_program> progs((size_t)n_q);
        std::vector<double> costs((size_t)n_q);
        std::vector<int64_t> offs((size_t)n_q + 1);
        std::vector<p2_stats> stats((size_t)n_q);
        int32_t rc = run_batch(qs.data(), n_q, &msg_bytes, 1, progs.data(), costs.data(), n_q, offs.data(), stats.data());
        if (rc != P2_OK) return rc;
        const double inf = std::numeric_limits<double>::infinity();
        for (int64_t p = 0; p < n_pl; ++p) {
            double total = 0.0;
            for (int s = 0; s < n_sets; ++s) {
                const size_t at = ((size_t)p * (size_t)n_sets + (size_t)s) * 2;
                p2_search_row& row = out_rows[(size_t)p * (size_t)n_sets + (size_t)s];
                std::memset(&row, 0, sizeof row);
                row.candidates = stats[at].candidates;
                row.valid = stats[at].valid;
                if (stats[at].alphabet == 0) {                  // a reduction over one device: nothing to do
                    row.best_cost = 0.0; row.allreduce_cost = 0.0;
                } else {
                    if (offs[at + 1] > offs[at]) { row.best = progs[(size_t)offs[at]]; row.best_cost = costs[(size_t)offs[at]]; }
                    else row.best_cost = inf;
                    if (offs[at + 2] - offs[at + 1] != 1) return fail(P2_EDEVICE, "the AllReduce baseline did not evaluate to one program");
                    row.allreduce_cost = costs[(size_t)offs[at + 1]];
                }
                total += (weights ? weights[s] : 1.0) * row.best_cost;
            }
            out_total[p] = total;
        }
        for (int64_t p = 0; p < n_pl; ++p) out_order[p] = (int32_t)p;
        std::stable_sort(out_order, out_order + n_pl, [&](int32_t a, int32_t b) { return out_total[a] < out_total[b]; });
        return P2_OK;
    } catch (const std::exception& e) {
        return fail(P2_EDEVICE, std::string("host failure: ") + e.what());
    }
}

int32_t p2_describe_pattern(const p2_hierarchy* h, const int32_t* axes, int32_t n_axes, const int32_t* placement,
                            const int32_t* reduce_axes, int32_t n_reduce, const p2_options* opt, int32_t pattern_id,
                            int32_t* slice_level, int32_t* form, int32_t* form_level, int32_t* group_of_device,
                            int32_t* rank_in_group, int32_t* out_n_patterns) {
    try {
        p2::Plan pl;
        std::string err;
        int32_t st = p2::make_plan(h, axes, n_axes, placement, reduce_axes, n_reduce, 1, opt, false, pl, err);
        if (st != P2_OK) return fail(st, err);
        if (out_n_patterns) *out_n_patterns = (int32_t)pl.patterns.size();
        if (pattern_id < 0 || pattern_id >= (int32_t)pl.patterns.size()) return fail(P2_EINVAL, "pattern id out of range");
        const p2::Pattern& p = pl.patterns[pattern_id];
        if (slice_level) *slice_level = p.slice;
        if (form) *form = p.form;
        if (form_level) *form_level = p.form_level;
        if (group_of_device && rank_in_group) p2::describe_pattern(pl, pattern_id, group_of_device, rank_in_group);
        return P2_OK;
    } catch (const std::exception& e) {
        return fail(P2_EDEVICE, std::string("host failure: ") + e.what());
    }
}

int32_t p2_topk_device(const double* cost, int64_t cost_stride, const uint64_t* index, int64_t n, int32_t k,
                       int64_t* out_pos, void* stream_) {
    using namespace p2;
    if (n < 0 || k < 0 || cost_stride < 1) return fail(P2_EINVAL, "bad n, k or stride");
    if (k > kMaxTopK) return fail(P2_EUNSUPPORTED, "topk > 1024");
    if (n == 0 || k == 0) return P2_OK;
    if (!cost || !index || !out_pos) return fail(P2_EINVAL, "null argument");
    hipStream_t stream = (hipStream_t)stream_;
    Ctx& C = g_ctx;
    P2_HIP(C.topk_scratch.ensure(topk_scratch_bytes(n, k)));
    P2_HIP(C.h_topk_nan.ensure(sizeof(uint32_t)));
    P2_HIP(C.open_topk_control(stream));
    C.topk_control_clear = false;                       // (until the kernels are known to have run to their end)
    uint32_t* nan = static_cast<uint32_t*>(C.h_topk_nan.p);
    *nan = 0u;
    P2_HIP(launch_topk(cost, cost_stride, reinterpret_cast<const unsigned long long*>(index), n, k,
                       reinterpret_cast<long long*>(out_pos), C.topk_scratch.p, C.topk_control.p, nan, stream));
    P2_HIP(hipStreamSynchronize(stream));
    C.topk_control_clear = true;
    if (*static_cast<volatile uint32_t*>(nan)) return fail(P2_EINVAL, "NaN cost");
    return P2_OK;
}

int32_t p2_topk_device_noalloc(const double* cost, int64_t cost_stride, const uint64_t* index, int64_t n, int32_t k,
                               int64_t* out_pos, uint32_t* out_nan, void* stream_) {
    using namespace p2;
    if (n < 0 || k < 0 || cost_stride < 1) return fail(P2_EINVAL, "bad n, k or stride");
    if (k > topk_fixed_max_k()) return fail(P2_EUNSUPPORTED, "topk > 64 without allocation: the fixed scratch holds lists of at most 64 entries");
    if (n == 0 || k == 0) return P2_OK;
    if (!cost || !index || !out_pos) return fail(P2_EINVAL, "null argument");
    P2_HIP(launch_topk_fixed(cost, cost_stride, reinterpret_cast<const unsigned long long*>(index), n, k,
                             reinterpret_cast<long long*>(out_pos), out_nan, (hipStream_t)stream_));
    return P2_OK;
}

int32_t p2_topk(const double* cost, const uint64_t* index, int64_t n, int32_t k, int64_t* out_pos) {
    using namespace p2;
    if (n < 0 || k < 0) return fail(P2_EINVAL, "bad n or k");
    if (k > kMaxTopK) return fail(P2_EUNSUPPORTED, "topk > 1024");
    if (n == 0 || k == 0) return P2_OK;
    if (!cost || !index || !out_pos) return fail(P2_EINVAL, "null argument");
    Ctx& C = g_ctx;
    const size_t kk = (size_t)std::min<int64_t>(k, n);
    P2_HIP(C.topk_in.ensure((size_t)n * 16));
    P2_HIP(C.topk_pos.ensure(kk * sizeof(long long)));
    double* dcost = static_cast<double*>(C.topk_in.p);
    uint64_t* didx = reinterpret_cast<uint64_t*>(dcost + n);
    P2_HIP(hipMemcpy(dcost, cost, (size_t)n * 8, hipMemcpyHostToDevice));
    P2_HIP(hipMemcpy(didx, index, (size_t)n * 8, hipMemcpyHostToDevice));
    int32_t rc = p2_topk_device(dcost, 1, didx, n, k, static_cast<int64_t*>(C.topk_pos.p), nullptr);
    if (rc != P2_OK) return rc;
    P2_HIP(hipMemcpy(out_pos, C.topk_pos.p, kk * sizeof(long long), hipMemcpyDeviceToHost));
    return P2_OK;
}

}  // extern "C"
