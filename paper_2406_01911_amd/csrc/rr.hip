// RR-set generation on gfx950 (Algorithm 3's skeleton with one keyed coin per
// channel), stratified roots, and compaction into the RR-set CSR.
//
// RR sets are very uneven: most cost a few hundred incidences, while a set
// that reaches a hub vertex (a member of ~1e5 hyperedges) or grows into a
// giant component costs millions.  Generation therefore runs in two phases.
//
// Phase A (k_rr_light, persistent): wavefronts steal RR ids from a global
// counter; one wavefront owns one set at a time in a "slot" (member list that
// doubles as the BFS queue, plus a visited bitmap -- in LDS when every graph
// of the launch is small).  Each frontier batch (up to 64 queued vertices) is
// expanded in three load-balanced levels -- vertices -> incidences (v, he) ->
// runs of 4 member positions -- so lanes stay busy under degree and size skew
// and member ids are read contiguously; one Philox4x32-10 block gives the 4
// coins of a run; a live channel from an unvisited member sets its bit
// (atomic OR) and the winner appends it with a ballot-ranked store.  A set
// whose next batch holds a heavy vertex, or that has read its share of
// incidences or member positions, is handed over intact (slot, queue head, size) to phase B and the
// wave takes a fresh slot.  Finished sets are written ascending to a staging
// area.
//
// Phase B (bulk-synchronous over the deferred sets): k_plan cuts every
// deferred set's current frontier into work items of bounded cost --
// segments of consecutive queue entries holding at most a few hundred
// incidences, or one heavy vertex's incidences in chunks -- and k_expand
// spreads the items over every wavefront of the GPU (several wavefronts per
// item when items are fewer than wavefronts), so a single giant set or hub
// expansion uses the whole chip; a wavefront that found only a few light
// members expands them itself right away (continuation) instead of leaving
// one more thin level to the next superstep.  Supersteps repeat until no frontier
// is left; k_finish sorts and stages each set.  No wave ever waits for
// another: items only refer to finished supersteps.
//
// A launch group covers several tasks -- (graph, key, pool, id range) -- back
// to back, described in device memory: both pools of a doubling round, or
// many IM instances on different graphs, share phase A and the supersteps.
//
// The other cascade models reuse this frame: under the gap models the same
// two phases run with level 3 replaced by one geometric-gap stream per
// incidence (expand_gaps); the linear-threshold walk (k_lt_walk) and the
// stratified setting's per-layer draws (k_layered) are one wave per set in
// phase A's slots.  A launch group holds graphs of one kind only.
//
// Compaction turns the per-id sizes into CSR offsets (device scan) and moves
// the staged members into the pools.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "dev_common.h"
#include "internal.h"
#include "plan_layout.h"

namespace hyperim {
namespace {

constexpr int kWG = 256;
constexpr int kWavesPerWG = kWG / kWave;
constexpr uint32_t kSortMax = 1024;          // phase A: sets up to this size are sorted in LDS
constexpr uint32_t kSortMaxWG = 4096;        // phase B: one workgroup sorts up to this size in LDS
constexpr uint32_t kLdsBitmapWords = 1024;   // visited bitmap in LDS when every |V| <= 32768
constexpr uint32_t kBigSet = 4096;           // compaction: one workgroup per larger set
constexpr uint32_t kItemCap = kPlanItemCap;      // phase B: work items per superstep
constexpr uint64_t kSlotBudget = 48ull << 30; // bytes of slot lists + bitmaps
// The remaining execution parameters (heavy-vertex threshold, per-set budget,
// chunk and segment sizes, prefilter threshold, supersteps per sync) are
// runtime values, see hyperim_tuning.

// A set also leaves the per-set phase once it has read this many member
// positions, or the incidence budget where that is larger: hyperedges of
// hundreds of members reach them long before the incidences (sets on hyperedges
// of up to 1000: the per-set phase of a serving session 450 ms without, 23 with).
constexpr uint32_t kReach = 262144;

// Counters (uint64 each) in the workspace counter block.
// kItems and kItems + 1 alternate between supersteps: superstep s plans into
// counter s & 1 while its k_expand clears the other one for superstep s + 1.
// kPlanned counts the frontier entries k_plan has taken (summed queue heads),
// the progress measure of the host loop.
// Counters that waves add to while others are added to lie 128 bytes apart:
// additions to one line are done one after another, about 7.5 ns each.
constexpr uint32_t kCtrLine = 16;
enum Ctr {
    kWork = 0,
    kBump = kCtrLine,
    kBigCount = 2 * kCtrLine,
    kFreeNext = 3 * kCtrLine,
    kDefCount = 4 * kCtrLine,
    kItems = 5 * kCtrLine,
    kItemsOther,
    kPlanned = 6 * kCtrLine,
    kNumCtr = 7 * kCtrLine
};
// Sums that every wave adds to once per launch, in kStatLines copies behind the
// counters, added up on the host.  (6144 waves with two sums each on the
// counters' own line: 0.09 ms of every superstep.)
// kPhiloxA and kPhilox count the Philox4x32-10 blocks k_rr_light and k_expand
// drew (lane blocks whose coins were needed); kBytesMs and kPhiloxMs are
// bundled mode's algorithmic bytes and blocks.
enum Stat { kBytesA = 0, kBytesB, kPhilox, kPhiloxA, kBytesMs, kPhiloxMs };
constexpr uint32_t kStatLines = 64;
constexpr uint32_t kCtrWords = kNumCtr + kStatLines * kCtrLine;

__device__ __forceinline__ void stat_add(unsigned long long *ctr, Stat which, uint64_t x) {
    if (x) atomicAdd(&ctr[kNumCtr + (blockIdx.x % kStatLines) * kCtrLine + which], (unsigned long long)x);
}
uint64_t stat_sum(const unsigned long long *ctr, Stat which) {
    uint64_t x = 0;
    for (uint32_t l = 0; l < kStatLines; ++l) x += ctr[kNumCtr + l * kCtrLine + which];
    return x;
}

// One graph of a launch group.
// vrec[v] = (first incidence, incidences, threshold, Philox blocks) and irec[e]
// = (hyperedge, its first member position, its size, 0): one 16-byte read, and
// one cache line, for all that an expansion needs of a vertex or an incidence.
struct GraphDesc {
    const uint32_t *he_mem, *P;
    const uint4 *vrec, *irec;
    uint32_t n, bm_words;
    // linear-threshold graphs: channels of the incidences before each one
    // (exclusive prefix of |he| - 1 over v_he, nnz + 1 entries); else null
    const unsigned long long *chan;
    // stratified-setting graphs: A(v) by layers and the count tables; else null
    const unsigned long long *lay_nb_off, *lay_ly_off;
    const uint32_t *lay_nb, *lay_ly_end, *l;
    const double *lay_ln, *lay_expm;
    // RR sets divided into R1 / R2 (Section 4.1): pool 0 draws its roots from
    // rP[0 .. rn1), pool 1 from rP[rn1 .. n), and a pool-0 set starts with
    // force[force_off[root] .. force_off[root + 1]) beside its root; else null
    const uint32_t *rP, *force;
    const unsigned long long *force_off;
    uint32_t rn1;
};

// The same arrays as global-memory pointers: descriptors are read from device
// memory, where the compiler cannot tell their address space and would emit
// flat loads.
#define HIM_GLOBAL __attribute__((address_space(1)))
typedef uint32_t Rec __attribute__((ext_vector_type(4)));
struct GraphView {
    const HIM_GLOBAL uint32_t *he_mem, *P, *rP;
    const HIM_GLOBAL Rec *vrec, *irec;
    uint32_t n, bm_words, rn1;
};

// Descriptors are read at wave-uniform indices; their fields go to scalar
// registers.
__device__ __forceinline__ GraphView graph_view(const GraphDesc &d) {
    GraphView v;
    v.he_mem = uni_ptr((const HIM_GLOBAL uint32_t *)d.he_mem);
    v.P = uni_ptr((const HIM_GLOBAL uint32_t *)d.P);
    v.vrec = uni_ptr((const HIM_GLOBAL Rec *)d.vrec);
    v.irec = uni_ptr((const HIM_GLOBAL Rec *)d.irec);
    v.rP = uni_ptr((const HIM_GLOBAL uint32_t *)d.rP);
    v.n = uni(d.n);
    v.bm_words = uni(d.bm_words);
    v.rn1 = uni(d.rn1);
    return v;
}

// One task of a launch group: launch indices [previous end, end) are RR ids
// first_id, first_id + 1, ... of pool `pool` on graph `graph` with Philox key
// (key0, key1).
struct TaskDesc {
    uint64_t end, first_id;
    uint32_t pool, graph, key0, key1;
};

struct RRArgs {
    const GraphDesc *graphs;
    const TaskDesc *tasks;
    uint32_t ntasks, qlog;
    uint32_t heavy, budget, chunk, seg, prefilter_min;   // execution parameters
    uint32_t reach;                  // member positions of a set in the per-set phase
    uint32_t slot_n, slot_words;     // slot list length and bitmap words (largest graph)
    uint32_t take, stage_step;       // launch indices and stage entries a wave reserves at a time (0: a set's)
    uint32_t free0;                  // first slot no wave owns
    uint64_t count;                  // launch indices [0, count)
    uint64_t out_base;               // per-id array index of launch index 0
    unsigned long long *ctr;         // Ctr block
    uint32_t *lists;                 // per slot: slot_n entries
    uint32_t *bitmaps;               // per slot: slot_words (global mode)
    uint32_t slot_total;             // slots available (waves own the first ones)
    uint32_t *stage;
    uint64_t stage_cap;
    uint64_t *stage_off;             // per id
    uint32_t *sizes;                 // per id
    uint32_t *roots;                 // per id
    uint64_t *big_ids;               // per big set: per-id index
    // deferred sets (phase B)
    uint64_t *def_idx;
    uint32_t *def_root, *def_slot, *def_head, *def_size, *def_task;
    uint4 *items;
};

constexpr uint32_t kLiveCap = 256;   // live channels a wave holds before marking them (global marks)
constexpr uint32_t kRunCap = 128;    // runs with a live coin a wave holds before reading their members

struct WaveLdsCore {
    uint32_t fr_scan[kWave];                   // gap models: inclusive scan of the frontier's incidence counts
    uint4 fr[kWave];                           // frontier vertex: id, first incidence - incidences before, thr
    uint4 in[kWave];                           // incidence: hyperedge, first position, size, runs before
    uint2 in_vt[kWave];                        // ... its vertex and threshold
    uint32_t mark[kWave];                      // owners of a window of slots (window_owner)
    uint4 runs[kRunCap];                       // held runs: first member's place, live positions, target
    uint32_t cont_u[kWave], cont_pos[kWave];   // phase B: members this wave appended, and where
};
// With visited bitmaps in global memory a wave also buffers live channels.
struct WaveLds : WaveLdsCore {
    uint32_t live[kLiveCap];                   // sources of live channels waiting to be marked
};

// Four member positions at once, from an address that is a multiple of 4 bytes
// (he_mem is allocated 16 bytes longer than its entries).
typedef uint32_t Quad __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ Quad load_quad(const HIM_GLOBAL uint32_t *p) { return *(const HIM_GLOBAL Quad *)p; }

// The task of launch index idx (first task whose end exceeds idx); idx is
// wave-uniform.
__device__ __forceinline__ uint32_t task_of(const RRArgs &a, uint64_t idx) {
    uint32_t lo = 0, hi = a.ntasks - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (uni64(a.tasks[mid].end) > idx) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// What a set needs to know about where it comes from.
struct SetRef {
    GraphView G;
    uint64_t j;
    uint32_t pool;
    uint2 key;
};

// t and idx are wave-uniform.
__device__ __forceinline__ SetRef set_ref(const RRArgs &a, uint32_t t, uint64_t idx) {
    const TaskDesc &T = a.tasks[t];
    const uint64_t start = t ? uni64(a.tasks[t - 1].end) : 0ull;
    SetRef r;
    r.G = graph_view(a.graphs[uni(T.graph)]);
    r.j = uni64(T.first_id) + (idx - start);
    r.pool = uni(T.pool);
    r.key = make_uint2(uni(T.key0), uni(T.key1));
    return r;
}

// Stratified root of RR id j: block b of the ladder (Q = 2^qlog ids in block
// 0, Q 2^(b-1) in block b >= 1, so block sizes are powers of two), offset
// o_b = floor(x n / 2^64) from the block's Philox draw, root =
// P[floor((t n + o_b) / T_b)] computed in 128-bit arithmetic.  With the RR
// sets divided, P and n are the pool's own root list and its length.
__device__ __forceinline__ uint32_t rr_root(const GraphView &G, uint32_t qlog, uint64_t j, uint32_t pool, uint2 key) {
    const uint64_t Q = 1ull << qlog;
    uint32_t b, s;
    uint64_t J;
    if (j < Q) {
        b = 0;
        J = 0;
        s = qlog;
    } else {
        const uint32_t hb = 63u - (uint32_t)__clzll((long long)j);
        b = hb - qlog + 1u;
        J = 1ull << hb;
        s = hb;
    }
    const HIM_GLOBAL uint32_t *P = G.P;
    uint64_t n = G.n;
    if (G.rP != nullptr) {
        P = pool == 0u ? G.rP : G.rP + G.rn1;
        n = pool == 0u ? G.rn1 : G.n - G.rn1;
    }
    const uint4 r = philox4x32_10(root_counter(b, pool), key);
    const uint64_t x = (uint64_t)r.x | ((uint64_t)r.y << 32);
    const uint64_t o = __umul64hi(x, n);
    const uint64_t t = j - J;
    const uint64_t lo = t * n;
    uint64_t hi = __umul64hi(t, n);
    const uint64_t lo2 = lo + o;
    hi += lo2 < lo ? 1ull : 0ull;
    const uint64_t pos = s == 0 ? lo2 : ((lo2 >> s) | (hi << (64u - s)));
    return P[pos];
}

template <bool kLds>
__device__ __forceinline__ uint32_t bm_load(uint32_t *bm, uint32_t w) {
    if constexpr (kLds) return bm[w];
    else return __hip_atomic_load(bm + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Appends a wave's newly reached members to a list whose size lives in a
// register (phase A: one wave owns the set).
struct LocalAppend {
    uint32_t *list;
    uint32_t size, n;
    // Append the members u[t] of the set bits t of `mask` (this lane's newly
    // reached members), all lanes at once: one wave scan gives each lane its
    // place.  Every lane of the wave calls it.
    __device__ __forceinline__ void push8(uint32_t mask, const uint32_t (&u)[8]) {
        const uint32_t cnt = (uint32_t)__popc(mask);
        const uint32_t incl = wave_incl_scan(cnt);
        const uint32_t total = uni(wave_bcast(incl, kWave - 1));
        if (total == 0) return;
        uint32_t at = size + incl - cnt;
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t)
            if ((mask >> t) & 1u) {
                if (at < n) list[at] = u[t];   // at < n always holds: one bit per vertex
                ++at;
            }
        size = min(size + total, n);
    }
    // One member per lane at most (`fresh`): places from the wave's ballot.
    __device__ __forceinline__ void push1(bool fresh, uint32_t u) {
        const uint64_t bal = __ballot(fresh);
        if (bal == 0ull) return;
        if (fresh) {
            const uint32_t at = size + (uint32_t)__popcll(bal & ((1ull << lane_id()) - 1ull));
            if (at < n) list[at] = u;
        }
        size = min(size + (uint32_t)__popcll(bal), n);
    }
};

// Member positions tested per lane and call: kQ Philox blocks of 4 coins.
// One block per lane and pass keeps every lane's Philox work useful (most
// hyperedges have few members, so the upper half of an 8-position run is
// often empty while its block would still cost the whole wave).
constexpr uint32_t kQ = 1;
constexpr uint32_t kRun = 4 * kQ;

// A queue entry of a deferred set with this bit set was expanded by the wave
// that appended it (continuation, below); readers of the queue mask it.
constexpr uint32_t kExpanded = 0x80000000u;

// Same with the size in global memory (phase B: many waves grow one set); the
// first 64 members this wave appends, and their queue positions, are also kept
// in the wave's LDS.
struct ContAppend {
    uint32_t *list;
    uint32_t *size;
    uint32_t n;
    uint32_t *cu, *cp;
    uint32_t count;   // members appended so far (wave-uniform)
    __device__ __forceinline__ void push8(uint32_t mask, const uint32_t (&u)[8]) {
        const uint32_t cnt = (uint32_t)__popc(mask);
        const uint32_t incl = wave_incl_scan(cnt);
        const uint32_t total = uni(wave_bcast(incl, kWave - 1));
        if (total == 0) return;
        uint32_t base = 0;
        if (lane_id() == kWave - 1) base = atomicAdd(size, total);
        uint32_t at = uni(wave_bcast(base, kWave - 1)) + incl - cnt;
        uint32_t c = count + incl - cnt;
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t)
            if ((mask >> t) & 1u) {
                if (at < n) list[at] = u[t];
                if (c < kWave) {
                    cu[c] = u[t];
                    cp[c] = at;
                }
                ++at;
                ++c;
            }
        count += total;
    }
};

// Marks the wave's buffered live-channel sources in the set's visited
// bitmap (global memory) and appends the ones not marked before.  Each lane
// issues up to four atomics before waiting for any, so a wave pays one
// memory round trip per 256 live channels rather than one per coin batch.
// With kLook the mark is read first and set only where it is missing: sets of the
// gap models reach most members many times over, and atomics go to
// memory every time (large graph, p = 0.01: 555 -> 520 ms; the coins' sets gain
// nothing, their thin supersteps wait for one more round trip).
// Every lane of the wave calls it.
template <bool kLook, class App>
__device__ __forceinline__ void flush_live(uint32_t *bm, WaveLds &L, uint32_t &nlive, App &app) {
    wave_sync();
    const uint32_t lane = lane_id();
    for (uint32_t i0 = 0; i0 < nlive; i0 += 4 * kWave) {
        uint32_t uu[8], old[4];
#pragma unroll
        for (uint32_t r = 0; r < 8; ++r) uu[r] = 0u;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + r * kWave + lane;
            old[r] = ~0u;
            if (i < nlive) {
                uu[r] = L.live[i];
                if constexpr (kLook) old[r] = bm_load<false>(bm, uu[r] >> 5);
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t bit = 1u << (uu[r] & 31);
            if (i0 + r * kWave + lane < nlive && (!kLook || (old[r] & bit) == 0u))
                old[r] = atomicOr(&bm[uu[r] >> 5], bit);
        }
        uint32_t fresh = 0;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) fresh |= ((old[r] >> (uu[r] & 31)) & 1u) ? 0u : 1u << r;
        app.push8(fresh, uu);
    }
    nlive = 0;
    wave_sync();
}

// Reads the members of the wave's held runs, 64 runs at a time, and hands the
// live ones on: to `app` at once when the visited bitmap is in LDS, else to the
// buffer of live channels, marked in batches.  Every lane of the wave calls it.
template <bool kLds, class App, class Lds>
__device__ __forceinline__ void read_runs(const GraphView &G, uint32_t *bm, Lds &L, uint32_t &nrun, uint32_t &nlive,
                                          App &app) {
    wave_sync();
    const uint32_t lane = lane_id();
    for (uint32_t i0 = 0; i0 < nrun; i0 += kWave) {
        uint32_t u[8], lv = 0;
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t) u[t] = 0u;
        if (i0 + lane < nrun) {
            const uint4 r = L.runs[i0 + lane];
            const Quad m = load_quad(G.he_mem + r.x);
            // the target itself is no channel
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t) {
                u[t] = m[t];
                lv |= ((r.y >> t) & 1u) && m[t] != r.z ? 1u << t : 0u;
            }
        }
        if constexpr (kLds) {
            uint32_t fresh = 0;
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t) {
                if ((lv >> t) & 1u) {
                    const uint32_t bit = 1u << (u[t] & 31);
                    if ((atomicOr(&bm[u[t] >> 5], bit) & bit) == 0u) fresh |= 1u << t;
                }
            }
            app.push8(fresh, u);
        } else {
            // placement from one ballot per position
            static_assert(kRun == 4 && kLiveCap >= kRun * kWave, "64 runs fit the buffer");
            uint64_t b[kRun];
            uint32_t tot = 0;
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t) {
                b[t] = __ballot((lv >> t) & 1u);
                tot += (uint32_t)__popcll(b[t]);
            }
            if (nlive + tot > kLiveCap) flush_live<false>(bm, L, nlive, app);
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t) {
                if ((lv >> t) & 1u) L.live[nlive + lane_rank(b[t])] = u[t];
                nlive += (uint32_t)__popcll(b[t]);
            }
        }
    }
    nrun = 0;
    wave_sync();
}

// Test the channels (he, u -> ve) at member positions [p0, p0 + cm) of one
// hyperedge (cm <= kRun, p0 a multiple of 4) in this lane: the coins are the
// words of the Philox block of quad p0/4.  The coins come first, the members
// are read where one is live (with the prefilter, before the coins too): such runs
// are held in L.runs (nrun entries) for read_runs.  Every lane of the wave must
// call it (inactive lanes with active = false).
template <bool kLds, class App, class Lds>
__device__ __forceinline__ void test_run(const GraphView &G, uint64_t j, uint32_t pool, uint2 key, uint32_t *bm,
                                         bool prefilter, bool active, uint32_t he, uint32_t hb, uint32_t p0,
                                         uint32_t cm, uint32_t ve, uint32_t the, App &app, uint64_t &px,
                                         Lds &L, uint32_t &nrun, uint32_t &nlive) {
    static_assert(kRun == 4, "one Philox block and one member load per run");
    uint32_t u[8];
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) u[t] = ve;
    uint32_t cand = active ? (1u << cm) - 1u : 0u;   // positions whose coins count
    if (prefilter) {
        if (active) {
            const Quad m = load_quad(G.he_mem + (hb + p0));
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t) u[t] = t < cm ? m[t] : ve;
        }
        // all mark words in flight together (u[t] is always a vertex id)
        uint32_t seen[kRun];
#pragma unroll
        for (uint32_t t = 0; t < kRun; ++t) seen[t] = bm_load<kLds>(bm, u[t] >> 5);
#pragma unroll
        for (uint32_t t = 0; t < kRun; ++t)
            if (u[t] == ve || (seen[t] & (1u << (u[t] & 31)))) cand &= ~(1u << t);
    }
    if (__ballot(cand != 0u) == 0) return;
    uint4 c = make_uint4(0u, 0u, 0u, 0u);
    if (cand) {
        c = philox4x32_10(coin_counter(j, he, ve, pool, p0 >> 2), key);
        ++px;
    }
    const uint32_t w[kRun] = {c.x, c.y, c.z, c.w};
    uint32_t lv = 0;
#pragma unroll
    for (uint32_t t = 0; t < kRun; ++t) lv |= ((cand >> t) & 1u) && channel_live(w[t], the) ? 1u << t : 0u;
    // with small probabilities most runs have no live channel at all, and
    // their members are never read; the others wait until there are 64 to read
    // at once (a few lanes of a wave find one here)
    const uint64_t hit = __ballot(lv != 0u);
    if (hit == 0ull) return;
    const uint32_t tot = (uint32_t)__popcll(hit);
    if (nrun + tot > kRunCap) read_runs<kLds>(G, bm, L, nrun, nlive, app);
    if (lv) L.runs[nrun + lane_rank(hit)] = make_uint4(hb + p0, lv, ve, 0u);
    nrun += tot;
}

// Independent cascade drawn by geometric gaps (models HYPERIM_MODEL_GAPS_*;
// the subset sampling of Section 2.2.1, Algorithm 2, on the IC channels):
// the stream of (RR id j, hyperedge he, target v) is he's positions in
// stored order, each live with p_v (a live position holding v itself is no
// channel and is dropped); the gaps of dead positions before the next live
// one, Geometric(p_v), come from word r mod 4 of the Philox block at
// counter (j_lo, he, v, pool << 31 | j_hi << 24 | r / 4) for gap r.  A gap
// drawn from word x with G positions left is the largest g <= G with
// Q(g) >= t, t = (2^32 - x) / 2^32: a descent over the bits of G, from the
// top, taking bit i when acc * S_i >= t (then acc = acc * S_i), with
// S_0 = q = 1 - p_v and S_{i+1} = S_i^2 -- IEEE double products in a fixed
// order, no logarithm, so any implementation of the same steps draws the
// same gaps.  g = G: no live position is left in the stream.
__device__ __forceinline__ uint32_t gap_draw(double q, uint32_t x, uint32_t G) {
#pragma clang fp contract(off)
    const double t = (double)((1ull << 32) - (uint64_t)x) * 0x1.0p-32;
    const uint32_t b = G ? 32u - (uint32_t)__clz(G) : 0u;
    uint32_t g = 0;
    double acc = 1.0;
    for (int i = (int)b - 1; i >= 0; --i) {
        double S = q;
        for (int k = 0; k < i; ++k) S = S * S;
        if ((uint64_t)g + (1ull << i) <= (uint64_t)G && acc * S >= t) {
            acc = acc * S;
            g += 1u << i;
        }
    }
    return g;
}

// The same draw from the stream's powers S_i = q^(2^i), i < kGapTab, kept in
// registers (each S_i is q squared i times in sequence, so the values and the
// descent's products are those of gap_draw); for G < 2^kGapTab.
constexpr uint32_t kGapTab = 8;
__device__ __forceinline__ uint32_t gap_draw_tab(const double (&S)[kGapTab], uint32_t x, uint32_t G) {
#pragma clang fp contract(off)
    const double t = (double)((1ull << 32) - (uint64_t)x) * 0x1.0p-32;
    uint32_t g = 0;
    double acc = 1.0;
#pragma unroll
    for (int i = (int)kGapTab - 1; i >= 0; --i) {
        const double a = acc * S[i];
        if (g + (1u << i) <= G && a >= t) {
            acc = a;
            g += 1u << i;
        }
    }
    return g;
}

// One candidate per lane (`live` with member u): marked and appended as in
// test_run.  Every lane of the wave calls it.
template <bool kLds, class App, class Lds>
__device__ __forceinline__ void push_live(uint32_t *bm, Lds &L, uint32_t &nlive, App &app, bool live, uint32_t u) {
    const uint64_t bal = __ballot(live);
    if (bal == 0ull) return;
    if constexpr (kLds) {
        bool fresh = false;
        if (live) {
            const uint32_t bit = 1u << (u & 31);
            fresh = (atomicOr(&bm[u >> 5], bit) & bit) == 0u;
        }
        app.push1(fresh, u);
    } else {
        const uint32_t tot = (uint32_t)__popcll(bal);
        if (nlive + tot > kLiveCap) flush_live<true>(bm, L, nlive, app);
        if (live) L.live[nlive + (uint32_t)__popcll(bal & ((1ull << lane_id()) - 1ull))] = u;
        nlive += tot;
    }
}

// Levels 2 and 3 under the gap models: the call's incidences g in [0, D)
// (wave w of W takes g = w, w + W, ...) go to lanes as a queue -- a lane whose
// stream has ended takes the next incidence -- so lanes stay busy while
// streams of different lengths run (a stream is sequential: gap r + 1 starts
// where gap r ended).  Each step draws one gap per busy lane; a live position
// yields its member (the target itself excepted), which is marked and
// appended as in test_run.  Returns the algorithmic bytes (12 per incidence,
// 4 per member read), wave-uniform after the caller's sum.
template <bool kLds, bool kUniform, class App, class Lds>
__device__ __forceinline__ uint64_t expand_gaps(const GraphView &G, Lds &L, uint64_t j, uint32_t pool, uint2 key,
                                                uint32_t *bm, uint32_t v, uint32_t e0, uint32_t D,
                                                uint32_t th_uniform, App &app, uint64_t &px, uint32_t &nlive,
                                                uint32_t w, uint32_t W) {
#pragma clang fp contract(off)
    const uint32_t lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    uint64_t next = w;   // next incidence of this wave (wave-uniform)
    uint64_t bytes = 0;
    bool more = false;
    uint32_t he = 0, hb = 0, hs = 0, vv = v, cur = 0, r = 0;
    double q = 1.0;
    double S[kGapTab];   // q^(2^i) of the lane's stream, when hs < 2^kGapTab
#pragma unroll
    for (uint32_t i = 0; i < kGapTab; ++i) S[i] = 1.0;
    uint4 blk = make_uint4(0u, 0u, 0u, 0u);
    for (;;) {
        const uint64_t idle = __ballot(!more);
        if (idle != 0ull && next < D) {
            // refill: the idle lanes take the next incidences in lane order
            const uint64_t g = next + (uint64_t)__popcll(idle & below) * W;
            if (!more && g < D) {
                uint32_t e = e0 + (uint32_t)g, th = th_uniform;
                if constexpr (!kUniform) {
                    const uint4 f = L.fr[search64(L.fr_scan, (uint32_t)g)];
                    vv = f.x;
                    e = f.y + (uint32_t)g;
                    th = f.z;
                }
                const Rec ir = G.irec[e];
                he = ir[0];
                hb = ir[1];
                hs = ir[2];
                bytes += 12u;
                more = th != 0u && hs != 0u;   // threshold 0: no channel into vv is live
                cur = 0u;
                r = 0u;
                q = 1.0 - (th == kAlways ? 1.0 : (double)th * 0x1.0p-32);
                if (hs < (1u << kGapTab)) {
                    S[0] = q;
#pragma unroll
                    for (uint32_t i = 1; i < kGapTab; ++i) S[i] = S[i - 1] * S[i - 1];
                }
            }
            next += (uint64_t)__popcll(idle) * W;
        }
        if (__ballot(more) == 0ull) {
            if (next >= D) break;
            continue;
        }
        uint32_t u = vv;
        bool live = false;
        if (more) {
            if ((r & 3u) == 0u) {
                blk = philox4x32_10(coin_counter(j, he, vv, pool, r >> 2), key);
                ++px;
            }
            const uint32_t x = (r & 3u) == 0u ? blk.x : (r & 3u) == 1u ? blk.y : (r & 3u) == 2u ? blk.z : blk.w;
            ++r;
            const uint32_t left = hs - cur;
            const uint32_t gap = hs < (1u << kGapTab) ? gap_draw_tab(S, x, left) : gap_draw(q, x, left);
            if (gap >= left) {
                more = false;
            } else {
                const uint32_t pos = cur + gap;
                u = G.he_mem[hb + pos];
                bytes += 4u;
                live = u != vv;
                cur = pos + 1u;
                more = cur < hs;
            }
        }
        push_live<kLds>(bm, L, nlive, app, live, u);
    }
    return bytes;
}

// Levels 2 and 3 of a frontier expansion.  Each lane brings one vertex v with
// the incidence range [e0, e0 + d) of v_he to expand (d = 0 for none); with
// kUniform all lanes pass the same v and e0 and d is the wave's incidence
// count (one heavy vertex), which needs no owner search.  thr: v's threshold.  Every channel
// (he, u -> v) of those incidences is tested with its coin and newly reached
// members go to `app`.  Level 3 first tests the first run of kRun member
// positions of each lane's own incidence, then spreads the remaining runs of
// the longer hyperedges over the wave.  W waves (a power of two, wave w of them passing
// w) may share one call: they split the batches of 64 incidences between
// them, and when there are fewer batches than waves, each batch's runs too;
// every run is tested by exactly one of them.  Returns the algorithmic bytes of
// the incidences (12 each plus 4 per member position, read or not: members are
// read where a coin is live), each counted by one wave, wave-uniform.
template <bool kLds, bool kUniform, bool kGaps, class App, class Lds>
__device__ __forceinline__ uint64_t expand(const GraphView &G, Lds &L, uint64_t j, uint32_t pool, uint2 key,
                                           uint32_t *bm, bool prefilter, uint32_t v, uint32_t e0, uint32_t d,
                                           uint32_t thr, App &app, uint64_t &px, uint32_t w = 0, uint32_t W = 1) {
    const uint32_t lane = lane_id();
    uint32_t nrun = 0, nlive = 0;   // runs and live channels held in LDS (wave-uniform)
    uint32_t D = d, fstart = 0;
    if constexpr (!kUniform) {
        const uint32_t dscan = wave_incl_scan(d);
        D = wave_bcast(dscan, kWave - 1);
        fstart = dscan - d;
        wave_sync();
        if constexpr (kGaps) L.fr_scan[lane] = dscan;
        L.fr[lane] = make_uint4(v, e0 - fstart, thr, 0u);
        wave_sync();
    }
    if constexpr (kGaps) {
        const uint64_t bytes = expand_gaps<kLds, kUniform>(G, L, j, pool, key, bm, v, e0, D, thr, app, px,
                                                           nlive, w, W);
        if constexpr (!kLds) flush_live<true>(bm, L, nlive, app);
        wave_sync();
        return wave_sum(bytes);
    }
    // batch share: batches b = boff, boff + bstride, ...; within a batch,
    // runs qb = sub_w * 64, (sub_w + sub) * 64, ...  (first runs: sub_w 0)
    const uint32_t nbatch = (D + kWave - 1) / kWave;
    uint32_t bstride = W, sub = 1;
    if (nbatch < W) {
        bstride = 1;
        while (bstride < nbatch) bstride <<= 1;
        sub = W / bstride;
    }
    const uint32_t boff = w & (bstride - 1), sub_w = w / bstride;
    uint64_t bytes = 0;
    for (uint32_t base = boff * kWave; base < D; base += bstride * kWave) {
        // level 2: one incidence (v, he) per lane
        const uint32_t g = base + lane;
        uint32_t he = 0, hb = 0, hs = 0, vv = v, th = thr, no = 0, e = e0 + g;
        if constexpr (!kUniform) {
            const uint4 f = L.fr[window_owner(L.mark, fstart, d, base)];
            vv = f.x;
            e = f.y + g;
            th = f.z;
        }
        if (g < D) {
            const Rec ir = G.irec[e];
            he = ir[0];
            hb = ir[1];
            hs = ir[2];
            no = th ? (hs + kRun - 1u) / kRun : 0u;   // threshold 0: no channel into vv is live
            if (sub_w == 0) bytes += 12u + 4u * hs;
        }
        // level 3, first pass: run 0 of the lane's own incidence
        if (sub_w == 0)
            test_run<kLds>(G, j, pool, key, bm, prefilter, no > 0, he, hb, 0u, min(kRun, hs), vv, th, app, px, L,
                           nrun, nlive);
        // second pass: runs 1.. of the longer hyperedges, flattened over the wave
        const uint32_t rem = no > 1 ? no - 1u : 0u;
        if (__ballot(rem > 0) == 0) continue;
        const uint32_t rscan = wave_incl_scan(rem);
        const uint32_t R = wave_bcast(rscan, kWave - 1);
        wave_sync();
        L.in[lane] = make_uint4(he, hb, hs, rscan - rem);
        if constexpr (!kUniform) L.in_vt[lane] = make_uint2(vv, th);
        wave_sync();
        for (uint32_t qb = sub_w * kWave; qb < R; qb += sub * kWave) {
            const uint32_t qg = qb + lane;
            const bool active = qg < R;
            const uint32_t k = window_owner(L.mark, rscan - rem, rem, qb);
            const uint4 in = L.in[k];
            uint32_t ve = v, the = thr;
            if constexpr (!kUniform) {
                const uint2 vt = L.in_vt[k];
                ve = vt.x;
                the = vt.y;
            }
            const uint32_t p0 = (qg - in.w + 1u) * kRun;
            test_run<kLds>(G, j, pool, key, bm, prefilter, active, in.x, in.y, p0, min(kRun, in.z - p0), ve, the, app,
                           px, L, nrun, nlive);
        }
    }
    read_runs<kLds>(G, bm, L, nrun, nlive, app);
    if constexpr (!kLds) flush_live<false>(bm, L, nlive, app);
    wave_sync();
    return wave_sum(bytes);
}

// A wave's launch indices: kWork hands out a.take at a time, after the first
// ones, which go by wave number.
struct WorkShare {
    uint64_t at = ~0ull, end = 0;
    __device__ __forceinline__ uint64_t next(const RRArgs &a) {
        if (at == ~0ull) {
            at = ((uint64_t)blockIdx.x * kWavesPerWG + uni(threadIdx.x / kWave)) * a.take;
            end = at + a.take;
        } else if (at == end) {
            unsigned long long got = 0;
            if (lane_id() == 0) got = atomicAdd(&a.ctr[kWork], (unsigned long long)a.take);
            at = (uint64_t)gridDim.x * kWavesPerWG * a.take + uni64(wave_bcast64(got, 0));
            end = at + a.take;
        }
        return at++;
    }
};

// A wave's room in the stage: a.stage_step entries at a time for sets of at most
// an eighth of that, so that less than an eighth of a step is left when the next
// one does not fit; larger sets reserve their own.  (Reservations meet at one
// counter, at 7.5 ns each.)
struct StageRoom {
    uint64_t at = 0, end = 0;
    __device__ __forceinline__ uint64_t take(const RRArgs &a, uint32_t size) {
        const bool own = size > a.stage_step / 8u;
        if (own || end - at < size) {
            unsigned long long got = 0;
            if (lane_id() == 0) got = atomicAdd(&a.ctr[kBump], (unsigned long long)(own ? size : a.stage_step));
            got = uni64(wave_bcast64(got, 0));
            if (own) return got;
            at = got;
            end = at + a.stage_step;
        }
        const uint64_t off = at;
        at += size;
        return off;
    }
};

// Record a finished set's per-id outputs.
__device__ __forceinline__ void record_set(const RRArgs &a, uint64_t idx, uint64_t off, uint32_t size, uint32_t root) {
    const uint64_t o = a.out_base + idx;
    a.stage_off[o] = off;
    a.sizes[o] = size;
    a.roots[o] = root;
    if (size > kBigSet) a.big_ids[atomicAdd(&a.ctr[kBigCount], 1ull)] = o;
}

// ---- phase A ---------------------------------------------------------------
// A pool-0 set of a graph whose RR sets are divided (Section 4.1) starts
// with the members of its root's small layers beside the root: they are
// marked and appended before the traversal (every lane of the wave calls it).
__device__ __forceinline__ void seed_forced(const GraphDesc &D, uint32_t root, uint32_t *bm, LocalAppend &app) {
    const HIM_GLOBAL unsigned long long *fo = uni_ptr((const HIM_GLOBAL unsigned long long *)D.force_off);
    if (fo == nullptr) return;
    const HIM_GLOBAL uint32_t *fm = uni_ptr((const HIM_GLOBAL uint32_t *)D.force);
    const uint64_t f0 = uni64(fo[root]), f1 = uni64(fo[root + 1]);
    const uint32_t lane = lane_id();
    for (uint64_t f = f0; f < f1; f += kWave) {
        uint32_t u = 0;
        bool fresh = false;
        if (f + lane < f1) {
            u = fm[f + lane];
            const uint32_t bit = 1u << (u & 31);
            fresh = (atomicOr(&bm[u >> 5], bit) & bit) == 0u;
        }
        app.push1(fresh, u);
    }
}

template <bool kLdsBitmap, bool kGaps>
__global__ __launch_bounds__(kWG) void k_rr_light(RRArgs a) {
    using Lds = typename std::conditional<kLdsBitmap, WaveLdsCore, WaveLds>::type;
    __shared__ Lds lds[kWavesPerWG];
    __shared__ uint32_t lbm[kLdsBitmap ? kWavesPerWG : 1][kLdsBitmap ? kLdsBitmapWords : 1];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    uint32_t slot = blockIdx.x * kWavesPerWG + wv;
    Lds &L = lds[wv];
    // a finished set is sorted where its expansions kept their state
    static_assert(sizeof(Lds) >= sizeof(uint32_t) * kSortMax, "sort buffer");
    uint32_t *sortb = reinterpret_cast<uint32_t *>(&L);
    uint32_t *list = a.lists + (uint64_t)slot * a.slot_n;
    uint32_t *bm;
    if constexpr (kLdsBitmap) {
        bm = lbm[wv];
        for (uint32_t i = lane; i < kLdsBitmapWords; i += kWave) bm[i] = 0u;
    } else {
        bm = a.bitmaps + (uint64_t)slot * a.slot_words;
    }
    wave_sync();
    bool can_defer = true;
    uint64_t bytes_done = 0, px = 0;
    WorkShare work;
    StageRoom room;
    for (;;) {
        const uint64_t idx = work.next(a);
        if (idx >= a.count) break;
        const uint32_t task = task_of(a, idx);
        const SetRef S = set_ref(a, task, idx);
        const GraphView &G = S.G;
        const uint32_t root = rr_root(G, a.qlog, S.j, S.pool, S.key);
        if (lane == 0) {
            list[0] = root;
            atomicOr(&bm[root >> 5], 1u << (root & 31));
        }
        LocalAppend app{list, 1u, G.n};
        if (S.pool == 0u) seed_forced(a.graphs[uni(a.tasks[task].graph)], root, bm, app);
        uint32_t head = 0;
        uint64_t incidences = 0, positions = 0;   // read for this set
        bool deferred = false;

        while (head < app.size) {
            // queue entries were stored by other lanes of this wave: a wave's
            // own accesses stay in order, so there is nothing to wait for (and
            // no L1 line of the graph to drop)
            wave_sync();
            const uint32_t nb = min((uint32_t)kWave, app.size - head);
            uint32_t v = 0, e0 = 0, d = 0, thr = 0;
            if (lane < nb) {
                v = list[head + lane];
                const Rec r = G.vrec[v];
                e0 = r[0];
                d = r[1];
                thr = r[2];
            }
            if (can_defer && (incidences > a.budget || positions > a.reach || __ballot(d > a.heavy) != 0)) {
                // hand the set over to phase B and continue with a fresh slot
                uint32_t fresh_slot = 0;
                if (lane == 0) fresh_slot = (uint32_t)atomicAdd(&a.ctr[kFreeNext], 1ull);
                fresh_slot = wave_bcast(fresh_slot, 0) + a.free0;
                if (fresh_slot < a.slot_total) {
                    if (lane == 0) {
                        const uint32_t dd = (uint32_t)atomicAdd(&a.ctr[kDefCount], 1ull);
                        a.def_idx[dd] = idx;
                        a.def_root[dd] = root;
                        a.def_slot[dd] = slot;
                        a.def_head[dd] = head;
                        a.def_size[dd] = app.size;
                        a.def_task[dd] = task;
                    }
                    if constexpr (kLdsBitmap) {
                        // the marks move to the slot's bitmap (all zero so far)
                        uint32_t *gbm = a.bitmaps + (uint64_t)slot * a.slot_words;
                        wave_sync();
                        for (uint32_t i = lane; i < G.bm_words; i += kWave) {
                            gbm[i] = bm[i];
                            bm[i] = 0u;
                        }
                        wave_sync();
                    } else {
                        bm = a.bitmaps + (uint64_t)fresh_slot * a.slot_words;
                    }
                    slot = fresh_slot;
                    list = a.lists + (uint64_t)slot * a.slot_n;
                    deferred = true;
                    break;
                }
                can_defer = false;   // no spare slot left: this wave finishes its sets itself
            }
            head += nb;
            bytes_done += 20ull * nb;
            const uint64_t bytes =
                expand<kLdsBitmap, false, kGaps>(G, L, S.j, S.pool, S.key, bm, false, v, e0, d, thr, app, px);
            bytes_done += bytes;
            const uint32_t read = wave_sum(d);
            incidences += read;
            positions += bytes / 4u - 3ull * read;   // 12 bytes per incidence, 4 per position
        }
        if (deferred) continue;
        const uint32_t size = app.size;

        // ---- output: ascending members into the stage --------------------
        const uint64_t off = room.take(a, size);
        wave_sync();
        if (off + size <= a.stage_cap) {
            if (size <= kSortMax) {
                uint32_t P2 = kWave;
                while (P2 < size) P2 <<= 1;
                for (uint32_t i = lane; i < P2; i += kWave) sortb[i] = i < size ? list[i] : 0xFFFFFFFFu;
                wave_sync();
                for (uint32_t k = 2; k <= P2; k <<= 1) {
                    for (uint32_t jj = k >> 1; jj > 0; jj >>= 1) {
                        for (uint32_t i = lane; i < P2; i += kWave) {
                            const uint32_t x = i ^ jj;
                            if (x > i) {
                                const uint32_t p = sortb[i], qv = sortb[x];
                                if ((p > qv) == ((i & k) == 0)) {
                                    sortb[i] = qv;
                                    sortb[x] = p;
                                }
                            }
                        }
                        wave_sync();
                    }
                }
                for (uint32_t i = lane; i < size; i += kWave) a.stage[off + i] = sortb[i];
                wave_sync();
            } else {
                uint32_t written = 0;
                for (uint32_t w0 = 0; w0 < G.bm_words; w0 += kWave) {
                    const uint32_t wi = w0 + lane;
                    uint32_t word = wi < G.bm_words ? bm_load<kLdsBitmap>(bm, wi) : 0u;
                    const uint32_t cnt = (uint32_t)__popc(word);
                    const uint32_t incl = wave_incl_scan(cnt);
                    uint64_t pos = off + written + incl - cnt;
                    while (word) {
                        const uint32_t bit = (uint32_t)__ffs(word) - 1u;
                        word &= word - 1u;
                        if (pos < off + size) a.stage[pos] = wi * 32u + bit;
                        ++pos;
                    }
                    written += wave_bcast(incl, kWave - 1);
                }
            }
        }
        if (lane == 0) record_set(a, idx, off, size, root);
        // clear this set's marks (the bitmap is all-zero again afterwards)
        if (kLdsBitmap && size * 4u > G.bm_words) {
            for (uint32_t i = lane; i < G.bm_words; i += kWave) bm[i] = 0u;
        } else {
            for (uint32_t i = lane; i < size; i += kWave) bm[list[i] >> 5] = 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        wave_sync();
    }
    if (lane == 0) stat_add(a.ctr, kBytesA, bytes_done);
    px = wave_sum(px);
    if (lane == 0) stat_add(a.ctr, kPhiloxA, px);
}

// ---- linear-threshold model ------------------------------------------------
// RR sets of the live-edge form of LT (Section 2.1, LT bullet): every vertex v
// keeps at most one of its c(v) channels -- (hyperedge, member) pairs in
// ascending hyperedge order and stored member order, v skipped -- each with
// weight W / 2^32, W = min(thr[v], floor(2^32 / c(v))) (thr = always-live
// counting as 2^32), so the weights into v sum to at most 1.  The Philox word
// at hyperedge slot kLtSlot, position 0, of (RR id, v) picks channel
// floor(x / W) when x < W c(v), none otherwise.  An RR set is the reverse
// walk from its root along kept channels until no channel is kept or the
// walk meets a vertex already in the set.
//
// One wave per set (persistent over the launch group's ids, like phase A).
// c(v) and the incidence holding the picked channel come from the graph's
// channel prefix over v's incidences (a 64-way search: each round the lanes
// probe 64 evenly spaced incidences of the remaining range); the lanes then
// find v's position in that hyperedge.  Lane 0 keeps the walk's list and
// visited bitmap (a slot of the phase-A workspace), so the membership test
// reads what the same lane wrote.  The set leaves ascending through the
// phase-A output path.
constexpr uint32_t kLtSlot = 0xFFFFFFFEu;

template <bool kLdsBitmap>
__global__ __launch_bounds__(kWG) void k_lt_walk(RRArgs a) {
    __shared__ uint32_t sort_s[kWavesPerWG][kSortMax];
    __shared__ uint32_t lbm[kLdsBitmap ? kWavesPerWG : 1][kLdsBitmap ? kLdsBitmapWords : 1];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    const uint32_t slot = blockIdx.x * kWavesPerWG + wv;
    uint32_t *sortb = sort_s[wv];
    uint32_t *list = a.lists + (uint64_t)slot * a.slot_n;
    uint32_t *bm;
    if constexpr (kLdsBitmap) {
        bm = lbm[wv];
        for (uint32_t i = lane; i < kLdsBitmapWords; i += kWave) bm[i] = 0u;
    } else {
        bm = a.bitmaps + (uint64_t)slot * a.slot_words;
    }
    wave_sync();
    uint64_t bytes_done = 0, px = 0;
    WorkShare work;
    StageRoom room;
    for (;;) {
        const uint64_t idx = work.next(a);
        if (idx >= a.count) break;
        const uint32_t task = task_of(a, idx);
        const SetRef S = set_ref(a, task, idx);
        const GraphView &G = S.G;
        const uint32_t root = rr_root(G, a.qlog, S.j, S.pool, S.key);
        const HIM_GLOBAL unsigned long long *chan =
            uni_ptr((const HIM_GLOBAL unsigned long long *)a.graphs[uni(a.tasks[task].graph)].chan);
        if (lane == 0) {
            list[0] = root;
            bm[root >> 5] |= 1u << (root & 31);
        }
        uint32_t size = 1, cur = root;
        for (;;) {
            const Rec vr = G.vrec[cur];
            const uint32_t e0 = uni(vr[0]), e1 = e0 + uni(vr[1]);
            const uint64_t base = uni64(chan[e0]);
            const uint64_t C = uni64(chan[e1]) - base;   // c(v)
            bytes_done += 36ull;
            if (C == 0) break;
            const uint32_t thr = uni(vr[2]);
            const uint64_t cap = (1ull << 32) / C;
            const uint64_t W = min(thr == kAlways ? (1ull << 32) : (uint64_t)thr, cap);
            const uint32_t x = uni(philox4x32_10(coin_counter(S.j, kLtSlot, cur, S.pool, 0u), S.key).x);
            ++px;
            if ((uint64_t)x >= W * C) break;   // W = 0 included: no channel is kept
            // the incidence e holding channel k: the last one in [e0, e1)
            // with chan[e] <= base + k (chan[e0] = base qualifies; the next
            // prefix exceeds it, so e has at least one channel)
            const uint64_t t = base + (uint64_t)x / W;
            uint32_t lo = e0, hi = e1;   // the answer lies in [lo, hi)
            while (hi - lo > (uint32_t)kWave) {
                const uint32_t step = (hi - lo + kWave - 1) / kWave;
                const uint32_t probe = lo + lane * step;
                const uint64_t ok = __ballot(probe < hi && chan[probe] <= t);
                const uint32_t l = 63u - (uint32_t)__clzll((long long)ok);   // lane 0 always qualifies
                lo += l * step;
                hi = min(hi, lo + step);
                bytes_done += 8ull;
            }
            const uint64_t ok = __ballot(lo + lane < hi && chan[lo + lane] <= t);
            const uint32_t e = lo + 63u - (uint32_t)__clzll((long long)ok);
            const Rec ir = G.irec[e];
            const uint64_t k = t - uni64(chan[e]);   // rank among e's channels
            const uint32_t hb = uni(ir[1]), hs = uni(ir[2]);
            // member k of the hyperedge with cur skipped
            uint32_t pc = hs;
            for (uint32_t p0 = 0; p0 < hs; p0 += kWave) {
                const uint64_t hit = __ballot(p0 + lane < hs && G.he_mem[hb + p0 + lane] == cur);
                if (hit) {
                    pc = p0 + (uint32_t)__ffsll((unsigned long long)hit) - 1u;
                    break;
                }
            }
            const uint32_t u = uni(G.he_mem[hb + ((uint32_t)k < pc ? (uint32_t)k : (uint32_t)k + 1u)]);
            bytes_done += 4ull * hs + 24ull;
            uint32_t seen = 0;
            if (lane == 0) {
                const uint32_t bit = 1u << (u & 31);
                seen = (bm_load<kLdsBitmap>(bm, u >> 5) & bit) != 0u;
                if (!seen) {
                    bm[u >> 5] |= bit;
                    list[size] = u;
                }
            }
            if (wave_bcast(seen, 0)) break;
            ++size;
            cur = u;
        }

        // ---- output: ascending members into the stage, as in phase A -----
        const uint64_t off = room.take(a, size);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // lane 0's list and bitmap stores
        if (off + size <= a.stage_cap) {
            if (size <= kSortMax) {
                uint32_t P2 = kWave;
                while (P2 < size) P2 <<= 1;
                for (uint32_t i = lane; i < P2; i += kWave) sortb[i] = i < size ? list[i] : 0xFFFFFFFFu;
                wave_sync();
                for (uint32_t kk = 2; kk <= P2; kk <<= 1) {
                    for (uint32_t jj = kk >> 1; jj > 0; jj >>= 1) {
                        for (uint32_t i = lane; i < P2; i += kWave) {
                            const uint32_t xx = i ^ jj;
                            if (xx > i) {
                                const uint32_t pv = sortb[i], qv = sortb[xx];
                                if ((pv > qv) == ((i & kk) == 0)) {
                                    sortb[i] = qv;
                                    sortb[xx] = pv;
                                }
                            }
                        }
                        wave_sync();
                    }
                }
                for (uint32_t i = lane; i < size; i += kWave) a.stage[off + i] = sortb[i];
                wave_sync();
            } else {
                uint32_t written = 0;
                for (uint32_t w0 = 0; w0 < G.bm_words; w0 += kWave) {
                    const uint32_t wi = w0 + lane;
                    uint32_t word = wi < G.bm_words ? bm_load<kLdsBitmap>(bm, wi) : 0u;
                    const uint32_t cnt = (uint32_t)__popc(word);
                    const uint32_t incl = wave_incl_scan(cnt);
                    uint64_t pos = off + written + incl - cnt;
                    while (word) {
                        const uint32_t bit = (uint32_t)__ffs(word) - 1u;
                        word &= word - 1u;
                        if (pos < off + size) a.stage[pos] = wi * 32u + bit;
                        ++pos;
                    }
                    written += wave_bcast(incl, kWave - 1);
                }
            }
        }
        if (lane == 0) record_set(a, idx, off, size, root);
        for (uint32_t i = lane; i < size; i += kWave) bm[list[i] >> 5] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        wave_sync();
    }
    if (lane == 0) stat_add(a.ctr, kBytesA, bytes_done);
    if (lane == 0) stat_add(a.ctr, kPhiloxA, px);
}

// ---- stratified setting -------------------------------------------------------
// RR sets of the stratified setting (Section 3.1.1, "Activation probability"
// and "Sampling strategy"; Algorithm 3's per-layer draws).  For a popped
// vertex v with l layers and layer i of n members: the layer probability is
// P = 1 / (i ln(l + 1)), a member's p = min(1, P / n); the Philox blocks at
// counter (j_lo, i, v, pool << 31 | j_hi << 24 | r) give U from block 0's
// first two words and the selection draws from its last two and every word
// of the later blocks.  The count h inverts U: Binomial(n, p) for n <= 20,
// else Poisson(P) truncated at min(n, kMaxPick); then h members are picked
// one at a time, draw x picking index floor(x (n - r) / 2^32) among those not
// picked yet (ascending).  ln(l + 1) and e^-P come from the graph's
// host-evaluated tables; the count arithmetic is IEEE double with no fused
// multiply-adds, in the order the recursions state.
//
// One wave per set (persistent, phase A's slots, bitmaps and output path):
// the (vertex, layer) pairs of the set's queued vertices, 64 vertices at a
// time, go to the lanes one pair each -- a hub has over a thousand layers, and
// with one lane per vertex the sets that met one took 9.9 ms a launch (a million
// vertices, 2048 sets a pool) against 0.58; picked members go through the
// visited bitmap (atomic or: the lane that sets the bit appends the member at a
// wave counter in LDS).
// Picks of a layer of at most 32 members live in a bit mask; larger layers
// keep their picked indices, ascending, in a per-lane scratch list.
constexpr uint32_t kMaxPick = 64;

__device__ __forceinline__ uint32_t layer_count(uint32_t n, uint32_t i, uint32_t l, double U,
                                                const HIM_GLOBAL double *ln, const HIM_GLOBAL double *expm) {
#pragma clang fp contract(off)
    const double P = 1.0 / ((double)i * ln[l]);
    const double p = P / (double)n;
    if (n <= 20u) {
        if (p >= 1.0) return n;
        const double q = 1.0 - p;
        double prob = 1.0;
        for (uint32_t t = 0; t < n; ++t) prob = prob * q;
        const double ratio = p / q;
        double cdf = prob;
        uint32_t h = 0;
        while (U >= cdf && h < n) {
            prob = ((prob * (double)(n - h)) / (double)(h + 1)) * ratio;
            ++h;
            cdf = cdf + prob;
        }
        return h;
    }
    double prob = expm[(size_t)l * (l - 1) / 2 + i - 1];
    double cdf = prob;
    const uint32_t hmax = min(n, kMaxPick);
    uint32_t h = 0;
    while (U >= cdf && h < hmax) {
        prob = (prob * P) / (double)(h + 1);
        ++h;
        cdf = cdf + prob;
    }
    return h;
}

// The wave's queued vertices: inclusive scan of their layer counts, id, layers,
// starts of their co-members and of their layer ends.
struct LayerLds {
    uint32_t scan[kWave], v[kWave], l[kWave];
    uint64_t nb[kWave], ly[kWave];
};

template <bool kLdsBitmap>
__global__ __launch_bounds__(kWG) void k_layered(RRArgs a, uint32_t *__restrict__ pick_scratch) {
    __shared__ uint32_t sort_s[kWavesPerWG][kSortMax];
    __shared__ uint32_t lbm[kLdsBitmap ? kWavesPerWG : 1][kLdsBitmap ? kLdsBitmapWords : 1];
    __shared__ uint32_t tail_s[kWavesPerWG];
    __shared__ LayerLds lds[kWavesPerWG];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    const uint32_t slot = blockIdx.x * kWavesPerWG + wv;
    LayerLds &L = lds[wv];
    uint32_t *sortb = sort_s[wv];
    uint32_t *list = a.lists + (uint64_t)slot * a.slot_n;
    uint32_t *picks = pick_scratch + ((uint64_t)slot * kWave + lane) * kMaxPick;
    uint32_t *bm;
    if constexpr (kLdsBitmap) {
        bm = lbm[wv];
        for (uint32_t i = lane; i < kLdsBitmapWords; i += kWave) bm[i] = 0u;
    } else {
        bm = a.bitmaps + (uint64_t)slot * a.slot_words;
    }
    wave_sync();
    uint64_t bytes_done = 0, px = 0;
    WorkShare work;
    StageRoom room;
    for (;;) {
        const uint64_t idx = work.next(a);
        if (idx >= a.count) break;
        const uint32_t task = task_of(a, idx);
        const SetRef S = set_ref(a, task, idx);
        const GraphView &G = S.G;
        const GraphDesc &D = a.graphs[uni(a.tasks[task].graph)];
        const HIM_GLOBAL unsigned long long *nb_off = uni_ptr((const HIM_GLOBAL unsigned long long *)D.lay_nb_off);
        const HIM_GLOBAL unsigned long long *ly_off = uni_ptr((const HIM_GLOBAL unsigned long long *)D.lay_ly_off);
        const HIM_GLOBAL uint32_t *nb = uni_ptr((const HIM_GLOBAL uint32_t *)D.lay_nb);
        const HIM_GLOBAL uint32_t *ly_end = uni_ptr((const HIM_GLOBAL uint32_t *)D.lay_ly_end);
        const HIM_GLOBAL uint32_t *lv_of = uni_ptr((const HIM_GLOBAL uint32_t *)D.l);
        const HIM_GLOBAL double *ln = uni_ptr((const HIM_GLOBAL double *)D.lay_ln);
        const HIM_GLOBAL double *expm = uni_ptr((const HIM_GLOBAL double *)D.lay_expm);
        const uint32_t root = rr_root(G, a.qlog, S.j, S.pool, S.key);
        if (lane == 0) {
            list[0] = root;
            if constexpr (kLdsBitmap) bm[root >> 5] |= 1u << (root & 31);
            else atomicOr(&bm[root >> 5], 1u << (root & 31));
            tail_s[wv] = 1u;
        }
        wave_sync();
        uint32_t head = 0, size = 1;
        while (head < size) {
            // queue entries were stored by other lanes of this wave
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            const uint32_t nbq = min((uint32_t)kWave, size - head);
            uint32_t qv = 0, ql = 0;
            uint64_t qb = 0, qy = 0;
            if (lane < nbq) {
                qv = list[head + lane];
                ql = lv_of[qv];
                qb = nb_off[qv];
                qy = ly_off[qv];
                bytes_done += 20ull + 4ull * ql;
            }
            const uint32_t lscan = wave_incl_scan(ql);
            const uint32_t pairs = wave_bcast(lscan, kWave - 1);
            wave_sync();
            L.scan[lane] = lscan;
            L.v[lane] = qv;
            L.l[lane] = ql;
            L.nb[lane] = qb;
            L.ly[lane] = qy;
            wave_sync();
            for (uint32_t g = lane; g < pairs; g += kWave) {
                const uint32_t k = search64(L.scan, g);
                const uint32_t v = L.v[k], l = L.l[k];
                const uint32_t i = g - (k ? L.scan[k - 1] : 0u) + 1u;   // layer i of v
                const uint64_t base = L.nb[k], lb = L.ly[k];
                const uint32_t lo = i > 1u ? ly_end[lb + i - 2u] : 0u, n = ly_end[lb + i - 1u] - lo;
                uint4 w = philox4x32_10(make_uint4((uint32_t)S.j, i, v,
                                                   (S.pool << 31) | ((uint32_t)(S.j >> 32) << 24)),
                                        S.key);
                ++px;
                const double U = (double)((uint64_t)(w.x >> 11) | ((uint64_t)w.y << 21)) * 0x1.0p-53;
                const uint32_t h = layer_count(n, i, l, U, ln, expm);
                uint32_t mask = 0, np = 0, word = 2, blk = 0;
                for (uint32_t r = 0; r < h; ++r) {
                    if (word == 4) {
                        w = philox4x32_10(make_uint4((uint32_t)S.j, i, v,
                                                     (S.pool << 31) | ((uint32_t)(S.j >> 32) << 24) | ++blk),
                                          S.key);
                        ++px;
                        word = 0;
                    }
                    const uint32_t x = word == 0 ? w.x : word == 1 ? w.y : word == 2 ? w.z : w.w;
                    ++word;
                    const uint32_t aidx = (uint32_t)(((uint64_t)x * (uint64_t)(n - r)) >> 32);
                    uint32_t pi;
                    if (n <= 32u) {
                        // the aidx-th clear bit of the mask
                        uint32_t c = aidx;
                        pi = 0;
                        for (uint32_t t = 0; t < n; ++t) {
                            if ((mask >> t) & 1u) continue;
                            if (c == 0) {
                                pi = t;
                                break;
                            }
                            --c;
                        }
                        mask |= 1u << pi;
                    } else {
                        pi = aidx;
                        uint32_t t = 0;
                        for (; t < np; ++t) {
                            const uint32_t q = picks[t];
                            if (q <= pi) ++pi;
                            else break;
                        }
                        for (uint32_t z = np; z > t; --z) picks[z] = picks[z - 1];
                        picks[t] = pi;
                        ++np;
                    }
                    const uint32_t u = nb[base + lo + pi];
                    const uint32_t bit = 1u << (u & 31);
                    if ((atomicOr(&bm[u >> 5], bit) & bit) == 0u) {
                        const uint32_t pos = atomicAdd(&tail_s[wv], 1u);
                        list[pos] = u;
                    }
                }
                bytes_done += 8ull + 4ull * h;
            }
            wave_sync();
            head += nbq;
            size = uni(tail_s[wv]);
        }

        // ---- output: ascending members into the stage, as in phase A -----
        const uint64_t off = room.take(a, size);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (off + size <= a.stage_cap) {
            if (size <= kSortMax) {
                uint32_t P2 = kWave;
                while (P2 < size) P2 <<= 1;
                for (uint32_t i = lane; i < P2; i += kWave) sortb[i] = i < size ? list[i] : 0xFFFFFFFFu;
                wave_sync();
                for (uint32_t kk = 2; kk <= P2; kk <<= 1) {
                    for (uint32_t jj = kk >> 1; jj > 0; jj >>= 1) {
                        for (uint32_t i = lane; i < P2; i += kWave) {
                            const uint32_t xx = i ^ jj;
                            if (xx > i) {
                                const uint32_t pv = sortb[i], qv = sortb[xx];
                                if ((pv > qv) == ((i & kk) == 0)) {
                                    sortb[i] = qv;
                                    sortb[xx] = pv;
                                }
                            }
                        }
                        wave_sync();
                    }
                }
                for (uint32_t i = lane; i < size; i += kWave) a.stage[off + i] = sortb[i];
                wave_sync();
            } else {
                uint32_t written = 0;
                for (uint32_t w0 = 0; w0 < G.bm_words; w0 += kWave) {
                    const uint32_t wi = w0 + lane;
                    uint32_t wd = wi < G.bm_words ? bm_load<kLdsBitmap>(bm, wi) : 0u;
                    const uint32_t cnt = (uint32_t)__popc(wd);
                    const uint32_t incl = wave_incl_scan(cnt);
                    uint64_t pos = off + written + incl - cnt;
                    while (wd) {
                        const uint32_t bit = (uint32_t)__ffs(wd) - 1u;
                        wd &= wd - 1u;
                        if (pos < off + size) a.stage[pos] = wi * 32u + bit;
                        ++pos;
                    }
                    written += wave_bcast(incl, kWave - 1);
                }
            }
        }
        if (lane == 0) record_set(a, idx, off, size, root);
        for (uint32_t i = lane; i < size; i += kWave) bm[list[i] >> 5] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        wave_sync();
    }
    bytes_done = wave_sum(bytes_done);
    px = wave_sum(px);
    if (lane == 0) stat_add(a.ctr, kBytesA, bytes_done);
    if (lane == 0) stat_add(a.ctr, kPhiloxA, px);
}

// ---- phase B ---------------------------------------------------------------
// Item: x = deferred set d | heavy << 31; light: y = first queue index,
// z = count (<= 64); heavy: y = vertex, z = first incidence, w = end.
// One atomicAdd per planning batch.  A reservation that crosses the cap is
// abandoned: its slots below the cap are filled with skip markers (x = ~0)
// by the reserving wave, so k_expand never reads an unwritten item.
constexpr uint32_t kSkipItem = 0xFFFFFFFFu;

// Owner lane of heavy-chunk slot q: binary search over the wave's inclusive
// scan of per-lane chunk counts, read through lane shuffles (every lane of
// the wave calls it).
__device__ __forceinline__ uint32_t owner_of(uint32_t hscan, uint32_t q) {
    return scan_owner([hscan](uint32_t k) { return (uint32_t)__shfl((int)hscan, (int)k, kWave); }, q);
}
constexpr uint32_t kShareMax = 16;   // waves that may share one item
// Levels a wave may expand past its item: many where other items keep the waves
// busy anyway, few where the superstep waits for its longest chain, up to 4
// items per wave.  8 against 3 there: 777 sets of a 10000-vertex graph 527 and
// 461 us, 4096 of a 1e5-vertex one 1.89 and 1.84 ms, a serving session 236 and
// 225 ms; with 3 everywhere eight mixed instances lost 1.2 %.  The gap models'
// thin supersteps gain nothing from fewer.
constexpr uint32_t kContLevels = 8, kContFew = 3;

// k_plan and k_expand read their arguments from device memory, so that a
// captured batch of supersteps serves every launch group.
__global__ __launch_bounds__(kWG) void k_plan(const RRArgs *__restrict__ ap, uint32_t parity) {
    const RRArgs a = *ap;
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    const uint32_t waves = gridDim.x * kWavesPerWG;
    const uint32_t ndef = uni((uint32_t)a.ctr[kDefCount]);   // sets phase A deferred
    uint64_t taken = 0;   // frontier entries this wave planned (progress count)
    for (uint32_t d = blockIdx.x * kWavesPerWG + wv; d < ndef; d += waves) {
        const uint32_t head0 = uni(a.def_head[d]);
        uint32_t head = head0;
        const uint32_t size = uni(a.def_size[d]);
        const uint32_t *list = a.lists + (uint64_t)uni(a.def_slot[d]) * a.slot_n;
        const GraphView G = graph_view(a.graphs[uni(a.tasks[uni(a.def_task[d])].graph)]);
        uint32_t most = kPlanBatches;   // batches of 64 entries planned at once
        while (head < size) {
            const uint32_t batches = min(most, (size - head + kWave - 1u) / kWave);
            uint32_t v[kPlanBatches], e0[kPlanBatches], deg[kPlanBatches], cv[kPlanBatches], hv[kPlanBatches],
                hscan[kPlanBatches];
            uint64_t firsts[kPlanBatches];
            uint32_t need = 0;
#pragma unroll
            for (uint32_t b = 0; b < kPlanBatches; ++b) {
                v[b] = b < batches && head + b * kWave + lane < size ? list[head + b * kWave + lane] : kExpanded;
            }
#pragma unroll
            for (uint32_t b = 0; b < kPlanBatches; ++b) {
                e0[b] = deg[b] = hv[b] = hscan[b] = 0u;
                firsts[b] = 0ull;
                cv[b] = a.chunk;
                const bool fresh = (v[b] & kExpanded) == 0u;
                if (__ballot(fresh) == 0ull) continue;   // all expanded already, or no such batch
                uint32_t light = 0;
                if (fresh) {
                    const Rec r = G.vrec[v[b]];
                    e0[b] = r[0];
                    deg[b] = r[1];
                    // a heavy vertex is cut into chunks of cv incidences
                    const HeavySplit hs = heavy_split(r[1], weighted_chunk(r[1], r[3], a.chunk));
                    cv[b] = hs.len;
                    hv[b] = hs.count;
                    light = hs.count ? 0u : light_weight(r[1], r[3]);
                }
                // light vertices form segments of consecutive queue entries
                const uint32_t lscan = wave_incl_scan(light);
                const uint32_t seg = segment_of(lscan, light, a.seg);
                const uint32_t prev_seg = __shfl_up(seg, 1, kWave);
                const bool in = head + b * kWave + lane < size;
                firsts[b] = __ballot(in && (lane == 0 || seg != prev_seg));
                hscan[b] = wave_incl_scan(hv[b]);
                need += (uint32_t)__popcll(firsts[b]) + wave_bcast(hscan[b], kWave - 1);
            }
            uint32_t entries = min(batches * kWave, size - head);
            if (const PlanFit fit = plan_fit(need, batches, kItemCap)) {
                if (fit == kPlanOneBatch) {
                    most = 1u;
                    continue;
                }
                entries = 1u;
                if (lane > 0) hv[0] = 0u;
                firsts[0] = 1ull;
                hscan[0] = wave_incl_scan(hv[0]);
                need = 1u + wave_bcast(hscan[0], kWave - 1);
            }
            if (need == 0u) {
                head += entries;
                continue;
            }
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(&a.ctr[kItems + parity], (unsigned long long)need);
            base = wave_bcast64(base, 0);
            if (base + need > kItemCap) {
                for (uint64_t x = base + lane; x < kItemCap; x += kWave) a.items[x].x = kSkipItem;
                break;
            }
#pragma unroll
            for (uint32_t b = 0; b < kPlanBatches; ++b) {
                if (firsts[b] == 0ull) continue;
                const uint32_t at = head + b * kWave, nb = min((uint32_t)kWave, entries - b * kWave);
                if ((firsts[b] >> lane) & 1ull) {
                    // segment = this lane up to the next first lane (or nb)
                    const uint64_t above = lane + 1 < 64 ? (firsts[b] >> (lane + 1)) << (lane + 1) : 0ull;
                    const uint32_t next = above ? (uint32_t)__ffsll((unsigned long long)above) - 1u : nb;
                    a.items[base + lane_rank(firsts[b])] = make_uint4(d, at + lane, min(next, nb) - lane, 0u);
                }
                base += (uint64_t)__popcll(firsts[b]);
                // heavy chunks, spread over the wave (a hub has hundreds)
                const uint32_t H = wave_bcast(hscan[b], kWave - 1);
                for (uint32_t q0 = 0; q0 < H; q0 += kWave) {
                    const uint32_t q = q0 + lane;
                    const uint32_t k = owner_of(hscan[b], min(q, H - 1u));
                    const uint32_t excl = (uint32_t)__shfl((int)(hscan[b] - hv[b]), (int)k, kWave);
                    const uint32_t vk = (uint32_t)__shfl((int)v[b], (int)k, kWave);
                    const uint32_t ek = (uint32_t)__shfl((int)e0[b], (int)k, kWave);
                    const uint32_t ck = (uint32_t)__shfl((int)cv[b], (int)k, kWave);
                    const uint32_t dk = (uint32_t)__shfl((int)deg[b], (int)k, kWave);
                    if (q < H) {
                        const ChunkRange cr = chunk_range(ek, dk, ck, q - excl);
                        a.items[base + q] = make_uint4(d | 0x80000000u, vk, cr.lo, cr.hi);
                    }
                }
                base += H;
            }
            head += entries;
            most = kPlanBatches;
        }
        if (lane == 0) a.def_head[d] = head;
        taken += head - head0;
    }
    if (lane == 0 && taken) atomicAdd(&a.ctr[kPlanned], (unsigned long long)taken);
}

// The counters a batch of supersteps leaves, into pinned host memory: one more
// small kernel of the batch, where a copy engine's transfer kept the next batch
// waiting for 18 us.
__global__ __launch_bounds__(kWG) void k_publish(const unsigned long long *__restrict__ ctr,
                                                  unsigned long long *__restrict__ host) {
    for (uint32_t i = threadIdx.x; i < kNumCtr; i += blockDim.x) host[i] = ctr[i];
    __threadfence_system();
}

template <bool kGaps>
__global__ __launch_bounds__(kWG) void k_expand(const RRArgs *__restrict__ ap, uint32_t parity) {
    const RRArgs a = *ap;
    __shared__ WaveLds lds[kWavesPerWG];
    const uint32_t wv = uni(threadIdx.x / kWave);
    WaveLds &L = lds[wv];
    const uint64_t nitems = min(a.ctr[kItems + parity], (unsigned long long)kItemCap);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr[kItems + (parity ^ 1u)] = 0ull;   // next superstep's counter
    uint64_t bytes_done = 0, px = 0;
    // items cost about seg or chunk incidences (more where one hyperedge alone
    // has more members than that), so a static strided
    // assignment balances well and needs no shared counter.  With fewer items
    // than waves (the thin tail of a traversal), W waves share each item.
    const uint64_t waves = (uint64_t)gridDim.x * kWavesPerWG;
    uint32_t W = 1;
    while (W < kShareMax && 2ull * W * nitems <= waves) W <<= 1;
    const uint32_t levels = kGaps || nitems > 4ull * waves ? kContLevels : kContFew;
    const uint64_t gw = (uint64_t)blockIdx.x * kWavesPerWG + wv, groups = waves / W;
    const uint32_t w = (uint32_t)(gw & (W - 1));
    const uint32_t lane = lane_id();
    // Items of one set lie together, and waves that work on one set at a time
    // queue up at its size counter (a million vertices, gap models: 20 ms a
    // launch against 14): neighbouring waves take items far apart, by an odd
    // multiplier near the golden ratio over the next power of two.
    uint64_t span = 1;
    while (span < nitems) span <<= 1;
    const uint64_t mult = ((span * 0x9E37ull) >> 16) | 1ull;
    for (uint64_t i0 = gw / W; i0 < span && gw < groups * W; i0 += groups) {
        const uint64_t it = (i0 * mult) & (span - 1u);
        if (it >= nitems) continue;
        const uint4 ld = a.items[it];
        const uint4 item = make_uint4(uni(ld.x), uni(ld.y), uni(ld.z), uni(ld.w));
        if (item.x == kSkipItem) continue;
        const uint32_t d = item.x & 0x7FFFFFFFu;
        const bool heavy = (item.x >> 31) != 0u;
        const uint32_t slot = uni(a.def_slot[d]);
        const SetRef S = set_ref(a, uni(a.def_task[d]), uni64(a.def_idx[d]));
        const GraphView &G = S.G;
        uint32_t *list = a.lists + (uint64_t)slot * a.slot_n;
        uint32_t *bm = a.bitmaps + (uint64_t)slot * a.slot_words;
        uint32_t *size_p = &a.def_size[d];
        const bool prefilter =
            uni(__hip_atomic_load(size_p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= a.prefilter_min;
        ContAppend app{list, size_p, G.n, L.cont_u, L.cont_pos, 0u};
        if (!heavy) {
            uint32_t v = 0, e0 = 0, deg = 0, thr = 0;
            const uint32_t raw = lane < item.z ? list[item.y + lane] : kExpanded;
            if ((raw & kExpanded) == 0u) {   // entries marked expanded are done
                v = raw;
                const Rec r = G.vrec[v];
                e0 = r[0];
                deg = r[1];
                thr = r[2];
                if (heavy_split(deg, weighted_chunk(deg, r[3], a.chunk)).count) deg = 0;   // expanded by its heavy items
            }
            if (w == 0) bytes_done += 20ull * (uint64_t)__popcll(__ballot((raw & kExpanded) == 0u));
            bytes_done += expand<false, false, kGaps>(G, L, S.j, S.pool, S.key, bm, prefilter, v, e0, deg, thr, app, px, w,
                                                       W);
        } else {
            // one heavy vertex: incidences [item.z, item.w) of vertex item.y
            bytes_done += expand<false, true, kGaps>(G, L, S.j, S.pool, S.key, bm, prefilter, item.y, item.z,
                                                      item.w - item.z, uni(G.vrec[item.y][2]), app, px, w,
                                                      W);
        }
        // Continuation: when this wave appended at most 64 members, all light
        // and together under seg incidences, it expands them itself (up to
        // kContLevels levels) and marks their queue entries expanded, so the
        // thin tail of a traversal does not take one superstep per level.
        // Nobody else reads those entries before the next superstep.
        for (uint32_t lev = 0; G.n <= kExpanded && lev < levels; ++lev) {
            const uint32_t cn = app.count;
            if (cn == 0 || cn > kWave) break;
            wave_sync();
            uint32_t v = 0, e0 = 0, deg = 0, pos = 0, thr = 0, weight = 0;
            bool heavy_v = false;
            if (lane < cn) {
                v = L.cont_u[lane];
                pos = L.cont_pos[lane];
                const Rec r = G.vrec[v];
                e0 = r[0];
                deg = r[1];
                thr = r[2];
                weight = light_weight(r[1], r[3]);
                heavy_v = deg > weighted_chunk(r[1], r[3], a.chunk);
            }
            const uint64_t tot = wave_sum((uint64_t)weight);
            if (__ballot(heavy_v) != 0 || tot > a.seg) break;   // left to k_plan
            wave_sync();
            if (lane < cn) list[pos] = v | kExpanded;
            app.count = 0;
            bytes_done += 20ull * cn;
            bytes_done += expand<false, false, kGaps>(G, L, S.j, S.pool, S.key, bm, prefilter, v, e0, deg, thr, app, px,
                                                       0u, 1u);
        }
    }
    if (lane == 0) stat_add(a.ctr, kBytesB, bytes_done);
    px = wave_sum(px);
    if (lane == 0) stat_add(a.ctr, kPhilox, px);
}

// One workgroup per deferred set: ascending members into the stage, per-id
// outputs, then the set's marks are cleared.
__global__ __launch_bounds__(kWG) void k_finish(RRArgs a, uint32_t ndef) {
    __shared__ uint32_t buf[kSortMaxWG];
    __shared__ uint32_t wave_tot[kWavesPerWG];
    __shared__ unsigned long long off_s;
    __shared__ uint32_t running;
    const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    for (uint32_t d = blockIdx.x; d < ndef; d += gridDim.x) {
        const uint32_t size = a.def_size[d];
        uint32_t *list = a.lists + (uint64_t)a.def_slot[d] * a.slot_n;
        uint32_t *bm = a.bitmaps + (uint64_t)a.def_slot[d] * a.slot_words;
        const uint32_t words = a.graphs[a.tasks[a.def_task[d]].graph].bm_words;
        if (threadIdx.x == 0) off_s = atomicAdd(&a.ctr[kBump], (unsigned long long)size);
        __syncthreads();
        const uint64_t off = off_s;
        if (off + size <= a.stage_cap) {
            if (size <= kSortMaxWG) {
                uint32_t P2 = kWG;
                while (P2 < size) P2 <<= 1;
                for (uint32_t i = threadIdx.x; i < P2; i += kWG) buf[i] = i < size ? (list[i] & ~kExpanded) : 0xFFFFFFFFu;
                __syncthreads();
                for (uint32_t k = 2; k <= P2; k <<= 1) {
                    for (uint32_t jj = k >> 1; jj > 0; jj >>= 1) {
                        for (uint32_t i = threadIdx.x; i < P2; i += kWG) {
                            const uint32_t x = i ^ jj;
                            if (x > i) {
                                const uint32_t p = buf[i], qv = buf[x];
                                if ((p > qv) == ((i & k) == 0)) {
                                    buf[i] = qv;
                                    buf[x] = p;
                                }
                            }
                        }
                        __syncthreads();
                    }
                }
                for (uint32_t i = threadIdx.x; i < size; i += kWG) a.stage[off + i] = buf[i];
            } else {
                if (threadIdx.x == 0) running = 0;
                __syncthreads();
                for (uint32_t w0 = 0; w0 < words; w0 += kWG) {
                    const uint32_t wi = w0 + threadIdx.x;
                    uint32_t word = wi < words ? bm[wi] : 0u;
                    const uint32_t cnt = (uint32_t)__popc(word);
                    const uint32_t incl = wave_incl_scan(cnt);
                    if (lane == kWave - 1) wave_tot[wv] = incl;
                    __syncthreads();
                    uint32_t before = running;
                    for (uint32_t q = 0; q < wv; ++q) before += wave_tot[q];
                    uint64_t pos = off + before + incl - cnt;
                    while (word) {
                        const uint32_t bit = (uint32_t)__ffs(word) - 1u;
                        word &= word - 1u;
                        if (pos < off + size) a.stage[pos] = wi * 32u + bit;
                        ++pos;
                    }
                    __syncthreads();
                    if (threadIdx.x == kWG - 1) running = before + incl;
                    __syncthreads();
                }
            }
        }
        if (threadIdx.x == 0) record_set(a, a.def_idx[d], off, size, a.def_root[d]);
        __syncthreads();
        if (size > words) {
            for (uint32_t i = threadIdx.x; i < words; i += kWG) bm[i] = 0u;
        } else {
            for (uint32_t i = threadIdx.x; i < size; i += kWG) bm[(list[i] & ~kExpanded) >> 5] = 0u;
        }
        __syncthreads();
    }
}

// ---- bundled mode: 64 sets per bundle, bit-parallel over the sets ----------
// For graphs whose RR sets are large (supercritical cascades), the sets of a
// launch group -- one task, launch indices in bundles of 64 -- grow together,
// level by level.  Per bundle and vertex u, seen[u] has bit s when u is in
// set s of the bundle and nxt[u] the bits found in the current level.  A
// frontier entry (bundle, v, mask) expands v once for every set in mask: v's
// incidences and their members are read once, seen[u] removes the sets that
// already hold u, and only the remaining (set, quad) pairs draw their Philox
// block.  RR sets are reachability closures, so the sets equal those of the
// per-set traversal.
constexpr uint32_t kMsSets = 64;
constexpr uint32_t kMsOutVerts = 4096;   // vertices per output block (16 per thread)

// kMsFetch: next work item of the running expansion (waves fetch items one at
// a time; item costs vary with hyperedge sizes).
enum MsCtr {
    kMsCur = 0,   // the ones that waves add to: a line each
    kMsNext = kCtrLine,
    kMsItems = 2 * kCtrLine,
    kMsPending = 3 * kCtrLine,
    kMsFetch = 4 * kCtrLine,
    kMsLevelDone = 5 * kCtrLine,
    kMsDone,
    kMsEpoch,
    kMsOverflow,
    kMsNumCtr = 6 * kCtrLine
};

struct MsArgs {
    GraphDesc graph;
    const unsigned long long *bytesw;   // algorithmic bytes of each vertex as a member
    uint64_t first_id;                  // RR id of launch index 0
    uint32_t pool, key0, key1, qlog;
    uint32_t nbundles, chunk, seg;
    uint32_t filter;                    // entries with this many sets read seen masks before coins
    uint64_t count;                     // sets: launch indices [0, count)
    uint64_t stride;                    // words per bundle in seen / nxt (>= n)
    unsigned long long *seen, *nxt;
    uint32_t *cur_b, *cur_v;            // frontier entries (bundle, vertex) ...
    unsigned long long *cur_m;          // ... and their set masks
    uint32_t *nx_b, *nx_v;              // vertices reached in the current level
    uint32_t *batch_epoch;              // per 64 frontier entries: level in which they were planned
    uint64_t list_cap;                  // entries of each list
    unsigned long long *ctr;            // MsCtr
    unsigned long long *stats;          // the RR counter block: algorithmic bytes, Philox blocks drawn
    uint4 *items;
    uint32_t *vcnt;                     // output: per (bundle, vertex block, set) counts
    uint32_t nvb;                       // vertex blocks per bundle
};

constexpr uint32_t kMsLiveCap = 256;   // live channels a wave holds before marking them
constexpr uint32_t kMsPend = 128;      // pairs with a live coin a wave holds before looking closer

struct MsLds {
    // level 2: frontier entries of the wave: vertex, first incidence -
    // incidences before, threshold, bundle; and their set masks
    uint4 fr[kWave];
    unsigned long long fr_m[kWave];
    // level 3: one incidence per lane: hyperedge, first position, size, quads
    // before; and its frontier entry's lane
    uint4 in[kWave];
    uint32_t in_k[kWave];
    uint32_t mark[kWave];                // owners of a window of slots (window_owner)
    // pairs with a coin below the threshold: (bundle << 8 | positions - 1 << 6 |
    // set, vertex, first member's place, largest live coin), (hyperedge, quad)
    uint4 pend[kMsPend];
    uint2 pend_q[kMsPend];
    // live channels waiting to be marked: (member, bundle << 6 | set)
    uint2 live[kMsLiveCap];
};

__device__ __forceinline__ void ms_append_next(const MsArgs &m, uint32_t b, uint32_t u) {
    const unsigned long long pos = atomicAdd(&m.ctr[kMsNext], 1ull);
    if (pos < m.list_cap) {
        m.nx_b[pos] = b;
        m.nx_v[pos] = u;
    } else {
        atomicOr(&m.ctr[kMsOverflow], 1ull);
    }
}

// Roots: set s of bundle b is launch index 64 b + s.
__global__ __launch_bounds__(kWG) void k_ms_roots(MsArgs m, RRArgs a) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m.count) return;
    const GraphView G = graph_view(m.graph);
    const uint32_t root = rr_root(G, m.qlog, m.first_id + i, m.pool, make_uint2(m.key0, m.key1));
    a.roots[a.out_base + i] = root;
    const uint32_t b = (uint32_t)(i / kMsSets), s = (uint32_t)(i % kMsSets);
    const unsigned long long old = atomicOr(&m.nxt[(uint64_t)b * m.stride + root], 1ull << s);
    if (old == 0ull) ms_append_next(m, b, root);
    // divided RR sets (Section 4.1): a pool-0 set also starts from the
    // members of its root's small layers
    if (m.pool == 0u && m.graph.force_off != nullptr) {
        for (unsigned long long f = m.graph.force_off[root]; f < m.graph.force_off[root + 1]; ++f) {
            const uint32_t u = m.graph.force[f];
            const unsigned long long o2 = atomicOr(&m.nxt[(uint64_t)b * m.stride + u], 1ull << s);
            if (o2 == 0ull) ms_append_next(m, b, u);
        }
    }
}

// New level: the vertices reached in the last one, with the sets that did not
// hold them yet, become the frontier.  Runs only once the level's frontier
// is fully planned and expanded.
__global__ __launch_bounds__(kWG) void k_ms_advance(MsArgs m) {
    constexpr uint32_t kPer = 4;   // entries per thread and turn: one reservation for all of the workgroup's
    __shared__ uint32_t part[kWavesPerWG];
    __shared__ unsigned long long base_s;
    if (m.ctr[kMsLevelDone] == 0ull) return;
    const uint64_t cnt = min(m.ctr[kMsNext], (unsigned long long)m.list_cap);
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kWG * kPer; i0 < cnt; i0 += (uint64_t)gridDim.x * kWG * kPer) {
        uint32_t b[kPer], u[kPer];
        unsigned long long found[kPer], fresh[kPer];
#pragma unroll
        for (uint32_t r = 0; r < kPer; ++r) {
            const uint64_t i = i0 + r * kWG + threadIdx.x;
            b[r] = u[r] = 0u;
            if (i < cnt) {
                b[r] = m.nx_b[i];
                u[r] = m.nx_v[i];
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kPer; ++r) {
            const uint64_t w = (uint64_t)b[r] * m.stride + u[r];
            found[r] = fresh[r] = 0ull;
            if (i0 + r * kWG + threadIdx.x < cnt) {
                found[r] = m.nxt[w];
                fresh[r] = found[r] & ~m.seen[w];
            }
        }
        uint64_t who[kPer];
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t r = 0; r < kPer; ++r) {
            const uint64_t w = (uint64_t)b[r] * m.stride + u[r];
            if (found[r]) m.nxt[w] = 0ull;
            if (fresh[r]) m.seen[w] |= fresh[r];   // each (bundle, vertex) appears once in the list
            who[r] = __ballot(fresh[r] != 0ull);
            mine += (uint32_t)__popcll(who[r]);
        }
        if (lane == 0) part[wv] = mine;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t all = 0;
            for (uint32_t q = 0; q < kWavesPerWG; ++q) all += part[q];
            base_s = all ? atomicAdd(&m.ctr[kMsCur], (unsigned long long)all) : 0ull;
        }
        __syncthreads();
        unsigned long long pos = base_s;
        for (uint32_t q = 0; q < wv; ++q) pos += part[q];
#pragma unroll
        for (uint32_t r = 0; r < kPer; ++r) {
            if (fresh[r]) {
                const unsigned long long p = pos + lane_rank(who[r]);
                if (p < m.list_cap) {
                    m.cur_b[p] = b[r];
                    m.cur_v[p] = u[r];
                    m.cur_m[p] = fresh[r];
                } else {
                    atomicOr(&m.ctr[kMsOverflow], 1ull);
                }
            }
            pos += (uint64_t)__popcll(who[r]);
        }
        __syncthreads();   // part and base_s are reused
    }
}

// Level bookkeeping between the kernels of one step (a single thread).
// After expansion: the level is done once every frontier batch was planned.
__global__ void k_ms_ctl_expanded(unsigned long long *ctr) {
    if (ctr[kMsPending] == 0ull) {
        ctr[kMsLevelDone] = 1ull;
        ctr[kMsCur] = 0ull;
        ctr[kMsEpoch] += 1ull;
    } else {
        ctr[kMsLevelDone] = 0ull;
    }
    ctr[kMsItems] = 0ull;
    ctr[kMsFetch] = 0ull;
}

// After advancing: the new level's batches are pending; no frontier, done.
__global__ void k_ms_ctl_advanced(unsigned long long *ctr, uint64_t list_cap) {
    if (ctr[kMsLevelDone] != 0ull) {
        ctr[kMsNext] = 0ull;
        const unsigned long long cur = min(ctr[kMsCur], (unsigned long long)list_cap);
        ctr[kMsCur] = cur;
        ctr[kMsPending] = (cur + kWave - 1) / kWave;
        if (cur == 0ull) ctr[kMsDone] = 1ull;
    }
}

// Cut the frontier into work items, 64 entries per wave at a time: light
// vertices in segments of consecutive entries (< seg + chunk incidences),
// heavy ones in chunks of their incidences.  A batch whose items do not fit
// the item buffer stays pending for the next step of the same level.
__global__ __launch_bounds__(kWG) void k_ms_plan(MsArgs m) {
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    const uint64_t ncur = m.ctr[kMsCur];
    const uint32_t epoch = (uint32_t)m.ctr[kMsEpoch] + 1u;   // never 0: fresh entries read 0
    const uint64_t nbatch = (ncur + kWave - 1) / kWave;
    const GraphView G = graph_view(m.graph);
    unsigned long long bytes = 0, planned = 0;
    // kPlanBatches batches per reservation (as in k_plan; one at a time when
    // their items might not fit an empty buffer)
    for (uint64_t b0 = ((uint64_t)blockIdx.x * kWavesPerWG + wv) * kPlanBatches; b0 < nbatch;
         b0 += (uint64_t)gridDim.x * kWavesPerWG * kPlanBatches) {
        uint32_t e0[kPlanBatches], deg[kPlanBatches], cv[kPlanBatches], hv[kPlanBatches], hscan[kPlanBatches],
            batch_need[kPlanBatches];
        uint64_t firsts[kPlanBatches];
        unsigned long long weight[kPlanBatches];   // algorithmic bytes of the lane's entry
        uint32_t todo = 0;
        uint64_t need = 0;
#pragma unroll
        for (uint32_t k = 0; k < kPlanBatches; ++k) {
            e0[k] = deg[k] = hv[k] = hscan[k] = batch_need[k] = 0u;
            cv[k] = m.chunk;
            firsts[k] = weight[k] = 0ull;
            const uint64_t bt = b0 + k;
            if (bt >= nbatch || uni(m.batch_epoch[bt]) == epoch) continue;
            todo |= 1u << k;
            const uint64_t f = bt * kWave + lane;
            const bool in = f < ncur;
            uint32_t light = 0;
            if (in) {
                const uint32_t v = m.cur_v[f], sets = (uint32_t)__popcll(m.cur_m[f]);
                const Rec r = G.vrec[v];
                e0[k] = r[0];
                deg[k] = r[1];
                weight[k] = (unsigned long long)sets * m.bytesw[v];
                // work grows with incidences times sets: heavy entries are cut
                // into chunks of about `chunk` (incidence, set) pairs
                const HeavySplit hs = ms_heavy_split(deg[k], sets, m.chunk);
                cv[k] = hs.len;
                hv[k] = hs.count;
                light = hs.count ? 0u : deg[k] * sets;   // segment weight: (incidence, set) pairs
            }
            const uint32_t lscan = wave_incl_scan(light);
            const uint32_t seg = segment_of(lscan, light, m.seg);
            const uint32_t prev_seg = __shfl_up(seg, 1, kWave);
            firsts[k] = __ballot(in && (lane == 0 || seg != prev_seg));
            hscan[k] = wave_incl_scan(hv[k]);
            batch_need[k] = (uint32_t)__popcll(firsts[k]) + wave_bcast(hscan[k], kWave - 1);
            need += batch_need[k];
        }
        if (todo == 0u) continue;
        const bool together = plan_together(need, kItemCap);
        unsigned long long base = 0;
        if (together) {
            if (lane == 0) base = atomicAdd(&m.ctr[kMsItems], (unsigned long long)need);
            base = uni64(wave_bcast64(base, 0));
            if (base + need > kItemCap) {
                for (uint64_t x = base + lane; x < kItemCap; x += kWave) m.items[x].x = kSkipItem;
                continue;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kPlanBatches; ++k) {
            if (((todo >> k) & 1u) == 0u) continue;
            if (!together) {
                if (lane == 0) base = atomicAdd(&m.ctr[kMsItems], (unsigned long long)batch_need[k]);
                base = uni64(wave_bcast64(base, 0));
                if (base + batch_need[k] > kItemCap) {
                    for (uint64_t x = base + lane; x < kItemCap; x += kWave) m.items[x].x = kSkipItem;
                    continue;
                }
            }
            const uint64_t f = (b0 + k) * kWave + lane;
            const uint32_t nb = (uint32_t)min((uint64_t)kWave, ncur - (b0 + k) * kWave);
            if ((firsts[k] >> lane) & 1ull) {
                const uint64_t above = lane + 1 < 64 ? (firsts[k] >> (lane + 1)) << (lane + 1) : 0ull;
                const uint32_t next = above ? (uint32_t)__ffsll((unsigned long long)above) - 1u : nb;
                m.items[base + lane_rank(firsts[k])] = make_uint4((uint32_t)f, min(next, nb) - lane, 0u, 0u);
            }
            const uint32_t nseg = (uint32_t)__popcll(firsts[k]);
            // heavy chunks, spread over the wave
            const uint32_t H = wave_bcast(hscan[k], kWave - 1);
            for (uint32_t q0 = 0; q0 < H; q0 += kWave) {
                const uint32_t q = q0 + lane;
                const uint32_t o = owner_of(hscan[k], min(q, H - 1u));
                const uint32_t excl = (uint32_t)__shfl((int)(hscan[k] - hv[k]), (int)o, kWave);
                const uint32_t fk = (uint32_t)__shfl((int)(uint32_t)f, (int)o, kWave);
                const uint32_t ek = (uint32_t)__shfl((int)e0[k], (int)o, kWave);
                const uint32_t ck = (uint32_t)__shfl((int)cv[k], (int)o, kWave);
                const uint32_t dk = (uint32_t)__shfl((int)deg[k], (int)o, kWave);
                if (q < H) {
                    const ChunkRange cr = chunk_range(ek, dk, ck, q - excl);
                    m.items[base + nseg + q] = make_uint4(fk | 0x80000000u, cr.lo, cr.hi, 0u);
                }
            }
            base += batch_need[k];
            bytes += weight[k];
            if (lane == 0) m.batch_epoch[b0 + k] = epoch;
            ++planned;
        }
    }
    if (lane == 0 && planned) atomicSub(&m.ctr[kMsPending], planned);
    bytes = wave_sum(bytes);
    if (lane == 0) stat_add(m.stats, kBytesMs, bytes);
}

// Marks the wave's buffered live channels in nxt, those that lead to a member
// the set does not hold yet, and appends the (bundle, member) pairs that got
// their first bit to the next-level list.  A marking needs the old mask back,
// so each lane first issues up to four reads of seen, then up to four atomics,
// and only then waits: two memory round trips per 256 channels.  One
// reservation of places for all of them.  Every lane of the wave calls it.
__device__ __forceinline__ void ms_flush(const MsArgs &m, MsLds &L, uint32_t &nlive) {
    wave_sync();
    const uint32_t lane = lane_id();
    static_assert(kMsLiveCap == 4 * kWave, "four channels per lane");
    unsigned long long old[4], held[4];
    uint32_t bb[4], uu[4], ss[4];
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t i = r * kWave + lane;
        bb[r] = uu[r] = ss[r] = 0;
        held[r] = ~0ull;
        if (i < nlive) {
            const uint2 e = L.live[i];
            uu[r] = e.x;
            bb[r] = e.y >> 6;
            ss[r] = e.y & 63u;
            held[r] = m.seen[(uint64_t)bb[r] * m.stride + uu[r]];
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        old[r] = ~0ull;
        if (((held[r] >> ss[r]) & 1ull) == 0ull)
            old[r] = atomicOr(&m.nxt[(uint64_t)bb[r] * m.stride + uu[r]], 1ull << ss[r]);
    }
    uint64_t who[4];
    uint32_t total = 0;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        who[r] = __ballot(old[r] == 0ull);
        total += (uint32_t)__popcll(who[r]);
    }
    if (total) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&m.ctr[kMsNext], (unsigned long long)total);
        base = wave_bcast64(base, 0);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if (old[r] == 0ull) {
                const unsigned long long pos = base + lane_rank(who[r]);
                if (pos < m.list_cap) {
                    m.nx_b[pos] = bb[r];
                    m.nx_v[pos] = uu[r];
                } else {
                    atomicOr(&m.ctr[kMsOverflow], 1ull);
                }
            }
            base += (uint64_t)__popcll(who[r]);
        }
    }
    nlive = 0;
    wave_sync();
}

// The held pairs' live channels go to the buffer: their block is drawn again
// (64 pairs to a wave here, two or three of its lanes where they were found)
// and their members are read for the first time; the vertex itself is left out.
// Every lane of the wave calls it.
__device__ __forceinline__ void ms_resolve(const MsArgs &m, const GraphView &G, MsLds &L, uint32_t &npend,
                                           uint32_t &nlive) {
    wave_sync();
    const uint32_t lane = lane_id();
    const uint64_t below = (1ull << lane) - 1ull;
    for (uint32_t i0 = 0; i0 < npend; i0 += kWave) {
        uint32_t lv = 0, tag = 0;
        Quad u = {0u, 0u, 0u, 0u};
        if (i0 + lane < npend) {
            const uint4 e = L.pend[i0 + lane];
            const uint2 q = L.pend_q[i0 + lane];
            u = load_quad(G.he_mem + e.z);
            const uint32_t bnd = e.x >> 8, s = e.x & 63u, cnt = ((e.x >> 6) & 3u) + 1u;
            const uint4 w = philox4x32_10(
                coin_counter(m.first_id + (uint64_t)bnd * kMsSets + s, q.x, e.y, m.pool, q.y),
                make_uint2(m.key0, m.key1));
            const uint32_t c[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (uint32_t t = 0; t < 4; ++t) lv |= t < cnt && u[t] != e.y && c[t] <= e.w ? 1u << t : 0u;
            tag = (bnd << 6) | s;
        }
        // placement from one ballot per position: the live channels of
        // position t follow those of positions < t, in lane order
        uint64_t b[4];
        uint32_t tot = 0;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            b[t] = __ballot((lv >> t) & 1u);
            tot += (uint32_t)__popcll(b[t]);
        }
        if (nlive + tot > kMsLiveCap) ms_flush(m, L, nlive);
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            if ((lv >> t) & 1u) L.live[nlive + (uint32_t)__popcll(b[t] & below)] = make_uint2(u[t], tag);
            nlive += (uint32_t)__popcll(b[t]);
        }
    }
    npend = 0;
    wave_sync();
}

// A quad of member positions on its way through the sets of an entry: what of
// its Philox blocks does not depend on the set.  Of the counter's words only
// the set's id j does, so the first round's product of v and one of the second
// round's are the quad's (37 of a block's 40 instructions are left), and M0 j
// is M0 times the bundle's first id plus M0 s.
struct MsQuad {
    uint32_t e, f, cw, mx;           // words of rounds 1 and 2 without the set's part
    uint32_t tag, v, at, most, he, q;
};
__device__ __forceinline__ MsQuad ms_quad(const MsArgs &m, uint32_t bnd, uint32_t v, uint32_t thr, uint32_t he,
                                          uint32_t q, uint32_t cnt, uint32_t at) {
    const uint64_t mv = (uint64_t)kPhiloxM1 * v;
    const uint64_t mx = (uint64_t)kPhiloxM0 * xor3((uint32_t)(mv >> 32), he, m.key0);
    MsQuad o;
    o.e = (uint32_t)mv ^ (m.key0 + kPhiloxW0);
    o.f = (uint32_t)(mx >> 32) ^ (m.key1 + kPhiloxW1);
    o.cw = coin_counter(m.first_id + (uint64_t)bnd * kMsSets, he, v, m.pool, q).w ^ m.key1;
    o.mx = (uint32_t)mx;
    o.tag = (bnd << 8) | (((cnt - 1u) & 3u) << 6);
    o.v = v;
    o.at = at;
    o.most = thr == kAlways ? kAlways : thr - 1u;
    o.he = he;
    o.q = q;
    return o;
}

// One (quad, set) pair per lane: its block, and the pair is held when a coin is
// low enough.  m0 = M0 j; lanes with act = false only join the wave-wide steps.
__device__ __forceinline__ void ms_pair(const MsArgs &m, const GraphView &G, MsLds &L, uint32_t &npend,
                                        uint32_t &nlive, const MsQuad &Q, bool act, uint32_t s, uint64_t m0) {
    const uint64_t m2 = (uint64_t)kPhiloxM1 * ((uint32_t)(m0 >> 32) ^ Q.cw);
    const uint4 w = philox_rounds<2>(make_uint4((uint32_t)(m2 >> 32) ^ Q.e, (uint32_t)m2, (uint32_t)m0 ^ Q.f, Q.mx),
                                     make_uint2(m.key0, m.key1));
    const bool hit = act && min(min(w.x, w.y), min(w.z, w.w)) <= Q.most;
    const uint64_t b = __ballot(hit);
    if (b == 0ull) return;
    const uint32_t tot = (uint32_t)__popcll(b);
    if (npend + tot > kMsPend) ms_resolve(m, G, L, npend, nlive);
    if (hit) {
        const uint32_t i = npend + lane_rank(b);
        L.pend[i] = make_uint4(Q.tag | s, Q.v, Q.at, Q.most);
        L.pend_q[i] = make_uint2(Q.he, Q.q);
    }
    npend += tot;
}

// M0 j of set s of a bundle whose first id is j0, j taken modulo 2^32 as the
// counter does (no bundle passes a multiple of 2^32, where the counter's last
// word would change too: launch groups end there).
__device__ __forceinline__ uint64_t ms_m0(uint64_t j0, uint32_t s) {
    return (uint64_t)kPhiloxM0 * (uint32_t)(j0 + s);
}

// Levels 2-4 for light entries.  Each lane brings a frontier entry (bundle b,
// vertex v, set mask) and the incidence range [e0, e0 + d) of v to expand
// (d = 0 for none).  Level 2 spreads the incidences over the wave, level 3 the
// quads of member positions of those hyperedges, and at level 4 every lane
// walks the sets of its quad.  A quad whose entry carries at least m.filter
// sets first reads its members and their seen masks and keeps only the sets
// that miss one of them; otherwise every set of the mask draws its coins.
__device__ __forceinline__ void ms_expand(const MsArgs &m, const GraphView &G, MsLds &L, uint32_t &npend,
                                          uint32_t &nlive, uint32_t b, uint32_t v, unsigned long long mask,
                                          uint32_t e0, uint32_t d, uint32_t thr, uint64_t &px) {
    const uint32_t lane = lane_id();
    const uint32_t dscan = wave_incl_scan(d);
    const uint32_t D = wave_bcast(dscan, kWave - 1);
    wave_sync();
    L.fr[lane] = make_uint4(v, e0 - (dscan - d), thr, b);
    L.fr_m[lane] = mask;
    wave_sync();
    for (uint32_t base = 0; base < D; base += kWave) {
        // level 2: one incidence (v, he) per lane
        const uint32_t g = base + lane;
        uint32_t he = 0, hb = 0, hs = 0, nq = 0;
        const uint32_t fk = window_owner(L.mark, dscan - d, d, base);
        if (g < D) {
            const uint4 f = L.fr[fk];
            const Rec ir = G.irec[f.y + g];
            he = ir[0];
            hb = ir[1];
            hs = ir[2];
            nq = f.z && hs > 1u ? (hs + 3u) >> 2 : 0u;   // threshold 0: no channel into the vertex is live
        }
        const uint32_t qscan = wave_incl_scan(nq);
        const uint32_t Q = wave_bcast(qscan, kWave - 1);
        if (Q == 0) continue;
        wave_sync();
        L.in[lane] = make_uint4(he, hb, hs, qscan - nq);
        L.in_k[lane] = fk;
        wave_sync();
        for (uint32_t qb = 0; qb < Q; qb += kWave) {
            // level 3: one quad of member positions per lane
            const uint32_t qg = qb + lane;
            const uint32_t k = window_owner(L.mark, qscan - nq, nq, qb);
            const uint4 in = L.in[k];
            const uint32_t fl = L.in_k[k];
            const uint4 f = L.fr[fl];   // vertex, -, threshold, bundle
            const uint32_t qq = qg - in.w, p0 = 4u * qq, at = in.y + p0, cnt = min(4u, in.z - p0);
            unsigned long long un = 0ull;
            if (qg < Q) {
                un = L.fr_m[fl];
                if ((uint32_t)__popcll(un) >= m.filter) {
                    const Quad u = load_quad(G.he_mem + at);
                    const uint64_t row = (uint64_t)f.w * m.stride;
                    unsigned long long sm[4];
#pragma unroll
                    for (uint32_t t = 0; t < 4; ++t) sm[t] = t < cnt && u[t] != f.x ? m.seen[row + u[t]] : ~0ull;
                    un &= ~(sm[0] & sm[1] & sm[2] & sm[3]);
                }
            }
            const uint32_t pc = (uint32_t)__popcll(un), pmax = wave_max(pc);
            if (pmax == 0u) continue;
            px += pc;
            const uint64_t j0 = m.first_id + (uint64_t)f.w * kMsSets;
            const MsQuad mq = ms_quad(m, f.w, f.x, f.z, in.x, qq, cnt, at);
            const uint64_t base0 = ms_m0(j0, 0u);
            unsigned long long rem = un;
            for (uint32_t r = 0; r < pmax; ++r) {
                const bool act = rem != 0ull;
                const uint32_t s = (uint32_t)__ffsll(rem) - 1u;
                rem &= rem - 1ull;
                ms_pair(m, G, L, npend, nlive, mq, act, s & 63u, base0 + (uint64_t)kPhiloxM0 * (s & 63u));
            }
        }
    }
    wave_sync();
}

// Levels 2-4 for a chunk [e0, e1) of a heavy entry's incidences: bundle, vertex
// and sets are the wave's, so every lane draws for the same set at a time, the
// set's part of the block is scalar work, and no lane waits for another.  The
// members' seen masks are not read before the coins: that spares a third of the
// blocks and costs more than those (with them 522 ms of expansion for a
// million vertices at theta = 4096, this form 400).
__device__ __forceinline__ void ms_expand_heavy(const MsArgs &m, const GraphView &G, MsLds &L, uint32_t &npend,
                                                uint32_t &nlive, uint32_t b, uint32_t v, unsigned long long mask,
                                                uint32_t e0, uint32_t e1, uint32_t thr, uint64_t &px) {
    if (thr == 0u) return;   // no channel into the vertex is live
    const uint32_t lane = lane_id(), sets = (uint32_t)__popcll(mask);
    const uint64_t j0 = m.first_id + (uint64_t)b * kMsSets;
    for (uint32_t base = e0; base < e1; base += kWave) {
        uint32_t he = 0, hb = 0, hs = 0, nq = 0;
        if (e1 - base > lane) {
            const Rec ir = G.irec[base + lane];
            he = ir[0];
            hb = ir[1];
            hs = ir[2];
            nq = hs > 1u ? (hs + 3u) >> 2 : 0u;
        }
        const uint32_t qscan = wave_incl_scan(nq);
        const uint32_t Q = wave_bcast(qscan, kWave - 1);
        if (Q == 0) continue;
        wave_sync();
        L.in[lane] = make_uint4(he, hb, hs, qscan - nq);
        wave_sync();
        for (uint32_t qb = 0; qb < Q; qb += kWave) {
            const uint32_t qg = qb + lane;
            const uint4 in = L.in[window_owner(L.mark, qscan - nq, nq, qb)];
            const uint32_t qq = qg - in.w, p0 = 4u * qq;
            const bool act = qg < Q;
            if (act) px += sets;
            const MsQuad mq = ms_quad(m, b, v, thr, in.x, qq, min(4u, in.z - p0), in.y + p0);
            for (unsigned long long rem = mask; rem; rem &= rem - 1ull) {
                const uint32_t s = (uint32_t)__ffsll(rem) - 1u;
                ms_pair(m, G, L, npend, nlive, mq, act, s, ms_m0(j0, s));
            }
        }
    }
    wave_sync();
}

__global__ __launch_bounds__(kWG) void k_ms_expand(MsArgs m) {
    __shared__ MsLds lds[kWavesPerWG];
    const uint32_t wv = uni(threadIdx.x / kWave);
    MsLds &L = lds[wv];
    const GraphView G = graph_view(m.graph);
    const uint64_t nitems = min(m.ctr[kMsItems], (unsigned long long)kItemCap);
    const uint32_t lane = lane_id();
    uint64_t px = 0;
    uint32_t npend = 0, nlive = 0;   // blocks and live channels held in LDS (wave-uniform)
    // items cost up to a few times each other (hyperedge sizes vary inside a
    // chunk), so waves fetch them as they go, a share of 1/16 of a wave's even
    // part at a time (all fetches meet at one counter, 7.5 ns each)
    const uint64_t waves = (uint64_t)gridDim.x * kWavesPerWG;
    const uint64_t share = max((uint64_t)1, min((uint64_t)64, nitems / (16u * waves)));
    for (uint64_t it = 0, end = 0;; ++it) {
        if (it == end) {
            unsigned long long got = 0;
            if (lane == 0) got = atomicAdd(&m.ctr[kMsFetch], (unsigned long long)share);
            it = uni64(wave_bcast64(got, 0));
            end = it + share;
        }
        if (it >= nitems) break;
        const uint4 ld = m.items[it];
        const uint4 item = make_uint4(uni(ld.x), uni(ld.y), uni(ld.z), uni(ld.w));
        if (item.x == kSkipItem) continue;
        if ((item.x >> 31) == 0u) {
            // light segment: entries [item.x, item.x + item.y)
            uint32_t b = 0, v = 0, e0 = 0, d = 0, thr = 0;
            unsigned long long mask = 0;
            if (lane < item.y) {
                const uint32_t f = item.x + lane;
                b = m.cur_b[f];
                v = m.cur_v[f];
                mask = m.cur_m[f];
                const Rec r = G.vrec[v];
                e0 = r[0];
                d = r[1];
                thr = r[2];
                if (ms_heavy_split(d, (uint32_t)__popcll(mask), m.chunk).count) d = 0;   // expanded by its heavy items
            }
            ms_expand(m, G, L, npend, nlive, b, v, mask, e0, d, thr, px);
        } else {
            // one heavy vertex: incidences [item.y, item.z) of entry item.x
            const uint32_t f = item.x & 0x7FFFFFFFu;
            const uint32_t b = uni(m.cur_b[f]), v = uni(m.cur_v[f]);
            const unsigned long long mask = uni64(m.cur_m[f]);
            const uint32_t thr = uni(G.vrec[v][2]);
            ms_expand_heavy(m, G, L, npend, nlive, b, v, mask, item.y, item.z, thr, px);
        }
    }
    ms_resolve(m, G, L, npend, nlive);
    ms_flush(m, L, nlive);
    px = wave_sum(px);
    if (lane == 0) stat_add(m.stats, kPhiloxMs, px);
}

// Output, pass 1: per (bundle, block of kMsOutVerts vertices) member counts
// of every set.
__global__ __launch_bounds__(kWG) void k_ms_count(MsArgs m) {
    __shared__ uint32_t cnt[kMsSets];
    const uint32_t b = blockIdx.x / m.nvb, blk = blockIdx.x % m.nvb;
    const uint32_t n = m.graph.n;
    if (threadIdx.x < kMsSets) cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t row = (uint64_t)b * m.stride;
    for (uint32_t i = 0; i < kMsOutVerts / kWG; ++i) {
        const uint32_t v = blk * kMsOutVerts + i * kWG + threadIdx.x;
        if (v >= n) break;
        unsigned long long w = m.seen[row + v];
        while (w) {
            const uint32_t s = (uint32_t)__ffsll(w) - 1u;
            w &= w - 1ull;
            atomicAdd(&cnt[s], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < kMsSets) m.vcnt[((uint64_t)b * m.nvb + blk) * kMsSets + threadIdx.x] = cnt[threadIdx.x];
}

// Pass 2, one thread per set: block counts become block offsets, the set
// gets its stage range and its per-id outputs.
__global__ __launch_bounds__(kWG) void k_ms_record(MsArgs m, RRArgs a) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m.count) return;
    const uint32_t b = (uint32_t)(i / kMsSets), s = (uint32_t)(i % kMsSets);
    uint32_t total = 0;
    for (uint32_t blk = 0; blk < m.nvb; ++blk) {
        uint32_t *c = &m.vcnt[((uint64_t)b * m.nvb + blk) * kMsSets + s];
        const uint32_t x = *c;
        *c = total;
        total += x;
    }
    const unsigned long long off = atomicAdd(&a.ctr[kBump], (unsigned long long)total);
    record_set(a, i, off, total, a.roots[a.out_base + i]);
}

// Pass 3: members in ascending order.  Each thread owns 16 consecutive
// vertices of the block; per set, a workgroup scan of the threads' counts
// places them.
__global__ __launch_bounds__(kWG) void k_ms_write(MsArgs m, RRArgs a) {
    __shared__ uint32_t wsum[kWavesPerWG];
    constexpr uint32_t kPer = kMsOutVerts / kWG;
    const uint32_t b = blockIdx.x / m.nvb, blk = blockIdx.x % m.nvb;
    const uint32_t n = m.graph.n, lane = lane_id(), wv = threadIdx.x / kWave;
    const uint64_t row = (uint64_t)b * m.stride;
    const uint32_t v0 = blk * kMsOutVerts + threadIdx.x * kPer;
    unsigned long long w[kPer];
    unsigned long long any = 0;
#pragma unroll
    for (uint32_t t = 0; t < kPer; ++t) {
        w[t] = v0 + t < n ? m.seen[row + v0 + t] : 0ull;
        any |= w[t];
    }
    const uint64_t sets = min((uint64_t)kMsSets, m.count - (uint64_t)b * kMsSets);
    for (uint32_t s = 0; s < sets; ++s) {
        const unsigned long long bit = 1ull << s;
        uint32_t c = 0;
        if (any & bit) {
#pragma unroll
            for (uint32_t t = 0; t < kPer; ++t) c += (w[t] & bit) ? 1u : 0u;
        }
        const uint32_t incl = wave_incl_scan(c);
        if (lane == kWave - 1) wsum[wv] = incl;
        __syncthreads();
        uint32_t before = incl - c;
        for (uint32_t q = 0; q < wv; ++q) before += wsum[q];
        const uint64_t id = a.out_base + (uint64_t)b * kMsSets + s;
        const uint64_t off = a.stage_off[id];
        const uint32_t size = a.sizes[id];
        if (c && off + size <= a.stage_cap) {
            uint64_t pos = off + m.vcnt[((uint64_t)b * m.nvb + blk) * kMsSets + s] + before;
#pragma unroll
            for (uint32_t t = 0; t < kPer; ++t)
                if (w[t] & bit) a.stage[pos++] = v0 + t;
        }
        __syncthreads();
    }
}

// ---- compaction ------------------------------------------------------------
// Sets up to kBigSet members, kLanes lanes per set and four members per lane
// and turn: bound by the chain from a set's offsets to its members, so many
// sets at once beat many lanes, until a set takes too many turns.  (A wave that
// moved 64 sets one 64-member window after the other: 209 us for the 320 sets
// of a 1000-vertex query, 5 us now; a serving session 3.4 -> 1.1 ms.)
template <uint32_t kLanes>
__global__ __launch_bounds__(kWG) void k_move_small(const uint64_t *__restrict__ stage_off,
                                                     const uint32_t *__restrict__ sizes,
                                                     const uint64_t *__restrict__ dst_off, uint64_t count,
                                                     const uint32_t *__restrict__ stage, uint32_t *__restrict__ mem) {
    constexpr uint32_t kPerWG = kWG / kLanes, kUnroll = 4;
    for (uint64_t id = (uint64_t)blockIdx.x * kPerWG + threadIdx.x / kLanes; id < count;
         id += (uint64_t)gridDim.x * kPerWG) {
        const uint32_t sz = sizes[id];
        if (sz > kBigSet) continue;
        const uint64_t src = stage_off[id], dst = dst_off[id];
        for (uint32_t e = threadIdx.x % kLanes; e < sz; e += kUnroll * kLanes) {
            uint32_t u[kUnroll];
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) u[t] = e + t * kLanes < sz ? stage[src + e + t * kLanes] : 0u;
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t)
                if (e + t * kLanes < sz) mem[dst + e + t * kLanes] = u[t];
        }
    }
}

// Sets above kBigSet members whose per-id index lies in [first, first + count):
// one workgroup each.
__global__ __launch_bounds__(kWG) void k_move_big(const uint64_t *__restrict__ big_ids,
                                                   const unsigned long long *__restrict__ big_count, uint64_t first,
                                                   uint64_t count, const uint64_t *__restrict__ stage_off,
                                                   const uint32_t *__restrict__ sizes,
                                                   const uint64_t *__restrict__ dst_off,
                                                   const uint32_t *__restrict__ stage, uint32_t *__restrict__ mem) {
    const uint64_t nbig = *big_count;
    for (uint64_t b = blockIdx.x; b < nbig; b += gridDim.x) {
        const uint64_t id = big_ids[b];
        if (id < first || id >= first + count) continue;
        const uint64_t src = stage_off[id], dst = dst_off[id - first];
        const uint32_t sz = sizes[id];
        for (uint32_t i = threadIdx.x; i < sz; i += blockDim.x) mem[dst + i] = stage[src + i];
    }
}

// Sums of four per-vertex weights over the members of a pool prefix.
__global__ __launch_bounds__(kWG) void k_weight_sum(const uint32_t *__restrict__ mem, uint64_t entries,
                                                     const unsigned long long *__restrict__ w0,
                                                     const unsigned long long *__restrict__ w1,
                                                     const unsigned long long *__restrict__ w2,
                                                     const unsigned long long *__restrict__ w3,
                                                     unsigned long long *__restrict__ out) {
    unsigned long long a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < entries;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t v = mem[i];
        a0 += w0[v];
        a1 += w1[v];
        a2 += w2[v];
        a3 += w3[v];
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    a2 = wave_sum(a2);
    a3 = wave_sum(a3);
    if (lane_id() == 0) {
        atomicAdd(out, a0);
        atomicAdd(out + 1, a1);
        atomicAdd(out + 2, a2);
        atomicAdd(out + 3, a3);
    }
}

// ---- host side -------------------------------------------------------------

// The descriptor of one graph in a launch group.
GraphDesc graph_desc(hyperim_graph g) {
    GraphDesc d{};   // fields of other models stay null
    d.he_mem = g->he_mem.as<uint32_t>();
    d.vrec = g->vrec.as<uint4>();
    d.irec = g->irec.as<uint4>();
    d.P = g->P.as<uint32_t>();
    d.n = g->n;
    d.bm_words = (uint32_t)(((uint64_t)g->n + 31u) / 32u);
    if (g->lt()) d.chan = g->chan.as<unsigned long long>();
    if (g->layered()) {
        d.lay_nb_off = g->lay_nb_off.as<unsigned long long>();
        d.lay_ly_off = g->lay_ly_off.as<unsigned long long>();
        d.lay_nb = g->lay_nb.as<uint32_t>();
        d.lay_ly_end = g->lay_ly_end.as<uint32_t>();
        d.l = g->l.as<uint32_t>();
        d.lay_ln = g->lay_ln.as<double>();
        d.lay_expm = g->lay_expm.as<double>();
    }
    if (g->routed) {
        d.rP = g->route_P.as<uint32_t>();
        d.force = g->force.as<uint32_t>();
        d.force_off = g->force_off.as<unsigned long long>();
        d.rn1 = g->route_n1;
    }
    return d;
}
struct LaunchShape {
    uint32_t grid;        // phase A workgroups at full occupancy (one slot per wave)
    uint32_t slots;       // total slots (phase A waves + spare slots for deferred sets)
    uint32_t grid_b;      // phase B workgroups at full occupancy
    uint32_t cus;         // compute units
    uint32_t slot_n, slot_words;
    bool lds;
};

// Slot layout for graphs of up to n_max vertices: phase A grid (from
// occupancy), slots (phase A waves plus spare slots for deferred sets, within
// kSlotBudget bytes) and the phase B grid.  80 slots per compute unit are four
// for each wave of five workgroups there.
// Lean, for graphs whose marks fit LDS: the bytes of 12 lists per compute unit,
// a quarter of the slots spare (a set that finds none stays with its wave).
// 32768 vertices: 2.8 GB of slots, 0.4 GB lean.
constexpr uint32_t kSlotsPerCu = 80, kLeanListsPerCu = 12;
struct SlotLayout {
    uint64_t grid, grid_lds, waves, slots, grid_b, bytes;
    uint32_t cus;
};

int slot_layout(uint32_t n_max, bool lean, SlotLayout *out) {
    int per_cu_lds = 0, per_cu_glb = 0, per_cu_b = 0, cus = 0, dev = 0;
    HIM_HIP(hipGetDevice(&dev));
    HIM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_lds, k_rr_light<true, false>, kWG, 0));
    HIM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_glb, k_rr_light<false, false>, kWG, 0));
    HIM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_b, k_expand<false>, kWG, 0));
    const uint64_t words = ((uint64_t)n_max + 31u) / 32u;
    const uint64_t per_slot = (uint64_t)n_max * 4u + words * 4u;
    const uint64_t max_slots = std::max<uint64_t>(kSlotBudget / std::max<uint64_t>(per_slot, 1), 2 * kWavesPerWG);
    uint64_t grid = (uint64_t)cus * (uint64_t)std::max(per_cu_glb, 1);
    uint64_t slots = std::min<uint64_t>(max_slots, (uint64_t)cus * kSlotsPerCu);
    // phase A keeps at least half of the slots spare for deferred sets
    grid = std::min<uint64_t>(grid, slots / (2 * kWavesPerWG));
    if (lean && n_max <= kLdsBitmapWords * 32u) {
        const uint64_t few = (uint64_t)cus * kLeanListsPerCu * n_max * 4u / std::max<uint64_t>(per_slot, 1);
        slots = std::min(slots, std::max<uint64_t>(few, 2 * kWavesPerWG));
        grid = std::min(grid, slots / 4u * 3u / kWavesPerWG);
    }
    grid = std::max<uint64_t>(grid, 1);
    out->grid_lds = std::min<uint64_t>(grid, (uint64_t)cus * (uint64_t)std::max(per_cu_lds, 1));
    out->grid = grid;
    out->waves = grid * kWavesPerWG;
    out->slots = slots;
    out->grid_b = (uint64_t)cus * (uint64_t)std::max(per_cu_b, 1);
    out->bytes = slots * per_slot;
    out->cus = (uint32_t)cus;
    return HYPERIM_OK;
}

// Allocates what ensure_workspace lays out for graphs of up to n_max vertices;
// the workspace counts as laid out (ws.grid) once everything is there and the
// bitmaps are clear.
int lay_out(RRWorkspace &ws, uint32_t n_max, bool lean, hipStream_t s) {
    const uint32_t words = (uint32_t)(((uint64_t)n_max + 31u) / 32u);
    SlotLayout L;
    HIM_CHECK(slot_layout(n_max, lean, &L));
    HIM_CHECK(ws.lists.reserve(sizeof(uint32_t) * (size_t)L.slots * n_max, s));
    HIM_CHECK(ws.bitmaps.reserve(sizeof(uint32_t) * (size_t)L.slots * words, s));
    HIM_CHECK(ws.counters.reserve(sizeof(unsigned long long) * kCtrWords, s));
    // deferred-set arrays for as many sets as there are slots (phase A may
    // run fewer waves than the occupancy allows, leaving more spare slots)
    const size_t ndef = L.slots;
    HIM_CHECK(ws.def_idx.reserve(sizeof(uint64_t) * ndef, s));
    HIM_CHECK(ws.def_u32.reserve(sizeof(uint32_t) * 5 * ndef, s));
    HIM_CHECK(ws.items.reserve(sizeof(uint4) * (size_t)kItemCap, s));
    HIM_CHECK(ws.args_dev.reserve(sizeof(RRArgs), s));
    HIM_HIP(hipMemsetAsync(ws.bitmaps.ptr, 0, sizeof(uint32_t) * (size_t)L.slots * words, s));
    ws.grid = (uint32_t)L.grid;
    ws.grid_lds = (uint32_t)L.grid_lds;
    ws.waves = (uint32_t)L.waves;
    ws.slots = (uint32_t)L.slots;
    ws.grid_b = (uint32_t)L.grid_b;
    ws.cus = L.cus;
    ws.slot_n = n_max;
    ws.slot_words = words;
    ws.lean = lean && n_max <= kLdsBitmapWords * 32u;
    return HYPERIM_OK;
}

// Slots sized for graphs of up to n_max (at least 1) vertices, re-created when a
// larger graph arrives or a caller that need not save finds a lean layout.  When
// the memory for them is not there, nothing of them stays and the next call
// starts over.
int ensure_workspace(RRWorkspace &ws, uint32_t n_max, bool lean, hipStream_t s, LaunchShape *shape) {
    if (ws.grid != 0 && (ws.slot_n < n_max || (ws.lean && !lean))) {
        HIM_HIP(hipStreamSynchronize(s));
        ws.drop_slots();
    }
    if (ws.grid == 0) {
        const int rc = lay_out(ws, n_max, lean, s);
        if (rc != HYPERIM_OK) {
            ws.drop_slots();
            return rc;
        }
    }
    const bool lds = n_max <= kLdsBitmapWords * 32u;
    shape->grid = lds ? ws.grid_lds : ws.grid;
    shape->slots = ws.slots;
    shape->grid_b = ws.grid_b;
    shape->cus = ws.cus;
    shape->slot_n = ws.slot_n;
    shape->slot_words = ws.slot_words;
    shape->lds = lds;
    return HYPERIM_OK;
}

// Id ranges of every (ladder block, stratum) pair inside [id_begin, id_end).
void stratum_ranges(hyperim_graph g, uint64_t seed, uint32_t instance, uint32_t qlog, uint32_t pool,
                    uint64_t id_begin, uint64_t id_end, std::vector<std::pair<uint64_t, uint64_t>> *out) {
    const uint64_t Q = 1ull << qlog;
    // with the RR sets divided, the pool's own root list and its strata
    const uint32_t n = g->routed ? (pool == 0 ? g->route_n1 : g->n - g->route_n1) : g->n;
    const uint32_t *B = g->routed ? g->route_B[pool ? 1 : 0] : g->info.B;
    uint64_t j = id_begin;
    while (j < id_end) {
        uint32_t b;
        uint64_t J, T;
        if (j < Q) {
            b = 0;
            J = 0;
            T = Q;
        } else {
            uint32_t hb = 63u - (uint32_t)__builtin_clzll(j);
            b = hb - qlog + 1u;
            J = 1ull << hb;
            T = J;
        }
        const uint4 r = philox4x32_10(root_counter(b, pool), make_uint2((uint32_t)seed, instance));
        const uint64_t x = (uint64_t)r.x | ((uint64_t)r.y << 32);
        const uint64_t o = (uint64_t)(((unsigned __int128)x * n) >> 64);
        uint64_t prev = 0;
        for (uint32_t h = 1; h <= kNStrata; ++h) {
            uint64_t th;
            if (h == kNStrata) {
                th = T;
            } else {
                // first t with floor((t n + o) / T) >= B_h
                unsigned __int128 need = (unsigned __int128)B[h] * T;
                th = need <= o ? 0 : (uint64_t)((need - o + n - 1) / n);
                th = std::min<uint64_t>(th, T);
            }
            const uint64_t lo = std::max<uint64_t>(J + prev, id_begin), hi = std::min<uint64_t>(J + th, id_end);
            if (lo < hi) out->push_back({lo, hi});
            prev = th;
        }
        j = J + T;
    }
}

int read_ctr(hipStream_t s, const unsigned long long *dev, int idx, uint64_t *out) {
    unsigned long long v = 0;
    HIM_HIP(hipMemcpyAsync(&v, dev + idx, sizeof(v), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    *out = v;
    return HYPERIM_OK;
}

// Wait for an event of the superstep loops, but not forever: a batch that has
// not finished after HYPERIM_WAIT_LIMIT_S seconds (default 600; a batch of
// the largest workloads takes a few seconds) ends the call with HYPERIM_EHIP
// naming the loop, instead of blocking the caller.  What runs on stream s then
// keeps the workspace until it is done.
int wait_event(RRWorkspace &ws, hipEvent_t e, hipStream_t s, const char *what) {
    static const double limit = [] {
        const char *v = getenv("HYPERIM_WAIT_LIMIT_S");
        const double x = v ? atof(v) : 0.0;
        return x > 0.0 ? x : 600.0;
    }();
    const auto t0 = std::chrono::steady_clock::now();
    for (;;) {
        const hipError_t q = hipEventQuery(e);
        if (q == hipSuccess) return HYPERIM_OK;
        if (q != hipErrorNotReady) {
            set_error_detail(std::string("waiting for ") + what + ": " + hipGetErrorString(q));
            return HYPERIM_EHIP;
        }
        const double el = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        if (el > limit) {
            if (ws.unfinished || hipEventCreate(&ws.unfinished) == hipSuccess)
                ws.left = hipEventRecord(ws.unfinished, s) == hipSuccess;
            set_error_detail(std::string(what) + " did not finish within the wait limit");
            return HYPERIM_EHIP;
        }
        if (el > 2e-3) std::this_thread::sleep_for(std::chrono::microseconds(20));
        else std::this_thread::yield();
    }
}

// Events of the RR workspace: [0], [1] start and end of phase A, [2], [3] of
// the closing k_finish (bundled mode: of the whole group); superstep batch
// slot b (two batches in flight) owns kBatchEv events from 4 + b * kBatchEv:
// batch start (the first batch's only), batch end (after its counter copy), then a start/end pair per
// k_expand launch when kernel times are asked for.  Events that time one
// kernel are stamped by its launch
// (hipExtLaunchKernelGGL): stream markers between dependent kernels would
// stall the device for several microseconds each.
constexpr int kMaxBatch = 64;
constexpr int kBatchEv = 2 + 2 * kMaxBatch;
constexpr int kNumEv = 4 + 2 * kBatchEv;

int event_pair(RRWorkspace &ws) {
    while (ws.events.size() < (size_t)kNumEv) {
        hipEvent_t e;
        HIM_HIP(hipEventCreate(&e));
        ws.events.push_back(e);
    }
    return HYPERIM_OK;
}

hipEvent_t *batch_events(RRWorkspace &ws, uint64_t k) { return &ws.events[4 + (size_t)(k & 1u) * kBatchEv]; }

// Pinned host staging of the RR workspace, in 64-bit words: counter-block
// copies (two superstep batches in flight, the end of a launch group), bundled
// mode's first counter, then per-call regions (graph and task descriptors, the
// pools' new totals).  Copies from and to it are asynchronous; the host
// touches a region only after waiting for the copy that uses it.
constexpr size_t kHostCtr = kNumCtr;
constexpr size_t kHostBatch = 0;   // + (k & 1) * kHostCtr for batch k
constexpr size_t kHostFinal = 2 * kHostCtr;
constexpr size_t kHostMsStart = kHostFinal + kCtrWords;
constexpr size_t kHostArgs = kHostMsStart + kCtrLine;   // the grid-wide phase's RRArgs on their way to the device
constexpr size_t kHostFixed = kHostArgs + (sizeof(RRArgs) + 7) / 8;

int ensure_host(RRWorkspace &ws, size_t words) {
    if (ws.host_words >= words) return HYPERIM_OK;
    const size_t w = std::max<size_t>(words, 2 * ws.host_words);
    if (ws.host) {
        HIM_HIP(hipDeviceSynchronize());   // no copy may still use the old buffer
        HIM_HIP(hipHostFree(ws.host));
    }
    ws.host = nullptr;
    ws.host_words = 0;
    HIM_HIP(hipHostMalloc((void **)&ws.host, w * sizeof(unsigned long long), hipHostMallocDefault));
    ws.host_words = w;
    ws.drop_graphs();   // captured batches copy into the old buffer
    return HYPERIM_OK;
}

// Captures the work `record` issues on the capture stream as one executable
// graph (record returns false when something it calls fails).  A device that
// cannot capture is remembered (graphs_off); *out is null then and the
// caller launches the kernels itself.
template <class Record>
int capture_graph(RRWorkspace &ws, Record &&record, hipGraphExec_t *out) {
    *out = nullptr;
    if (ws.graphs_off) return HYPERIM_OK;
    if (!ws.capture && hipStreamCreateWithFlags(&ws.capture, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        ws.graphs_off = true;
        return HYPERIM_OK;
    }
    hipGraph_t g = nullptr;
    bool ok = hipStreamBeginCapture(ws.capture, hipStreamCaptureModeThreadLocal) == hipSuccess;
    if (ok) {
        ok = record(ws.capture) && hipGetLastError() == hipSuccess;
        ok = hipStreamEndCapture(ws.capture, &g) == hipSuccess && ok && g;
    }
    hipGraphExec_t ex = nullptr;
    if (ok) ok = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess;
    if (g) (void)hipGraphDestroy(g);
    if (!ok) {
        (void)hipGetLastError();
        ws.graphs_off = true;
        return HYPERIM_OK;
    }
    *out = ex;
    return HYPERIM_OK;
}

// The captured superstep batch for `key` (everything the capture bakes in),
// captured on first use and kept in the workspace.
template <class Record>
int captured_batch(RRWorkspace &ws, const uint64_t (&key)[8], Record &&record, hipGraphExec_t *out) {
    *out = nullptr;
    for (const RRWorkspace::BatchGraph &b : ws.batch_graphs)
        if (std::equal(std::begin(key), std::end(key), std::begin(b.key))) {
            *out = b.exec;
            return HYPERIM_OK;
        }
    hipGraphExec_t ex = nullptr;
    HIM_CHECK(capture_graph(ws, record, &ex));
    if (!ex) return HYPERIM_OK;
    RRWorkspace::BatchGraph b;
    std::copy(std::begin(key), std::end(key), std::begin(b.key));
    b.exec = ex;
    ws.batch_graphs.push_back(b);
    *out = ex;
    return HYPERIM_OK;
}

// One launch group: phase A over `a`'s tasks, then phase B over the sets it
// deferred, then the deferred sets' output.  Per-id outputs land at
// a.out_base + launch index.  Supersteps go in batches of steps_per_sync (the
// later ones may be shorter), and the next batch is queued before the host reads the frontier count at the end
// of the last one, so the device never waits for the host between batches
// (the batch queued after the frontier ran out finds no work).  The closing
// counter block lands in ws.host + kHostFinal; `tail` may queue more work
// behind it, and the call returns after the stream has drained.  With
// `expect_defer` false the host first checks whether phase A deferred any set.
template <class Tail>
int run_launch(RRWorkspace &ws, RRStats &st, const hyperim_tuning &tune, RRArgs &a, const LaunchShape &shape,
               uint32_t grid, uint32_t grid_b, bool expect_defer, bool trace, bool time_kernels, bool graphs,
               bool gaps, hipStream_t s, Tail &&tail) {
    unsigned long long *ctr = a.ctr;
    unsigned long long *h = ws.host;
    // the grid-wide phase reads its arguments from the device
    *reinterpret_cast<RRArgs *>(h + kHostArgs) = a;
    HIM_HIP(hipMemcpyAsync(ws.args_dev.ptr, h + kHostArgs, sizeof(RRArgs), hipMemcpyHostToDevice, s));
    const RRArgs *ap = ws.args_dev.as<RRArgs>();
    HIM_CHECK(event_pair(ws));
    auto light = shape.lds ? (gaps ? k_rr_light<true, true> : k_rr_light<true, false>)
                           : (gaps ? k_rr_light<false, true> : k_rr_light<false, false>);
    auto expand_k = gaps ? k_expand<true> : k_expand<false>;
    hipExtLaunchKernelGGL(light, dim3(grid), dim3(kWG), 0, s, ws.events[0], ws.events[1], 0u, a);
    HIM_HIP(hipGetLastError());
    st.launches += 1;

    // phase B: supersteps over the deferred sets
    bool phase_b = true;
    uint64_t ndef = 0;
    if (!expect_defer) {
        HIM_HIP(hipMemcpyAsync(h + kHostBatch, ctr, sizeof(unsigned long long) * kNumCtr, hipMemcpyDeviceToHost, s));
        HIM_HIP(hipStreamSynchronize(s));
        ndef = h[kHostBatch + kDefCount];
        phase_b = ndef != 0;
    }
    int first = trace ? 1 : (int)std::min<uint32_t>(std::max<uint32_t>(tune.steps_per_sync, 1), kMaxBatch);
    // captured batches replay the same parities every time: an even batch
    // starts every replay on counter parity 0.  Launches timed one by one
    // (events stamped by the launch itself) are not captured: an event
    // recorded inside a graph does not time against one recorded outside.
    const bool use_graphs = graphs && !trace && !time_kernels && !ws.graphs_off;
    if (use_graphs && (first & 1)) first = std::min(first + 1, kMaxBatch);
    // Most traversals are over, or nearly, after a first batch of 8 or more, and
    // each superstep queued beyond the end costs 9 us: the later batches are a
    // quarter as long (even).  777 sets of a 10000-vertex graph, first 8: 592 us
    // with later batches of 8, 549 of 4, 530 of 2; 4096 sets of a 1e5-vertex
    // graph 1.94, 1.90 and 1.90 ms.  Shorter first batches stay as asked: halving
    // 4 cost 0.7 % where there were 17 supersteps to do.
    const int later = first < 8 ? first : first / 4 & ~1;
    auto batch_size = [&](uint64_t k) { return k == 0 ? first : later; };
    auto batch_start = [&](uint64_t k) { return k == 0 ? 0ull : (uint64_t)first + (k - 1) * (uint64_t)later; };
    float ms_before = 0.f;
    auto account = [&](uint64_t k) -> int {
        const int batch = batch_size(k);
        hipEvent_t *E = batch_events(ws, k);
        float ms = 0.f;
        // first k_plan of the first batch .. last k_expand (or the batch's
        // counter copy), less the batches before: one event between batches
        HIM_HIP(hipEventElapsedTime(&ms, batch_events(ws, 0)[0], time_kernels ? E[3 + 2 * (batch - 1)] : E[1]));
        st.ms_bfs += ms - ms_before;
        st.ms_heavy += ms - ms_before;
        ms_before = ms;
        for (int i = 0; time_kernels && i < batch; ++i) {
            float me = 0.f;
            HIM_HIP(hipEventElapsedTime(&me, E[2 + 2 * i], E[3 + 2 * i]));
            st.ms_expand += me;
        }
        st.expand_launches += batch;
        st.launches += 2 * batch;
        st.supersteps += batch;
        return HYPERIM_OK;
    };
    bool queued = false;   // a batch is queued but not yet accounted
    uint64_t k = 0;
    if (phase_b) {
        // planning waves: one per deferred set; until the count is known, the
        // spare slots bound it
        uint64_t plan_sets = ndef ? ndef : std::max<uint64_t>(shape.slots - (uint64_t)grid * kWavesPerWG, 1);
        // captured batches plan with one grid wide enough for any count of
        // deferred sets (planning waves stride over the sets)
        const uint32_t plan_grid_all = (uint32_t)std::max<uint64_t>(
            1, std::min<uint64_t>(div_up(std::max<uint64_t>(shape.slots - (uint64_t)grid * kWavesPerWG, 1),
                                         kWavesPerWG),
                                  4096));
        auto issue = [&](uint64_t kb) -> int {
            const int batch = batch_size(kb);
            hipEvent_t *E = batch_events(ws, kb);
            unsigned long long *dst = h + kHostBatch + (kb & 1u) * kHostCtr;
            if (use_graphs) {
                // one replay: batch x (k_plan, k_expand) and the counter copy
                const uint64_t key[8] = {1u, (uint64_t)(kb & 1u), (uint64_t)batch, plan_grid_all,
                                         (uint64_t)grid_b, gaps ? 1u : 0u, (uint64_t)(uintptr_t)ap,
                                         (uint64_t)(uintptr_t)h ^ ((uint64_t)(uintptr_t)ctr << 1)};
                hipGraphExec_t ex = nullptr;
                HIM_CHECK(captured_batch(
                    ws, key,
                    [&](hipStream_t c) {
                        for (int i = 0; i < batch; ++i) {
                            const uint32_t parity = (uint32_t)(i & 1);
                            hipLaunchKernelGGL(k_plan, dim3(plan_grid_all), dim3(kWG), 0, c, ap, parity);
                            hipLaunchKernelGGL(expand_k, dim3(grid_b), dim3(kWG), 0, c, ap, parity);
                        }
                        hipLaunchKernelGGL(k_publish, dim3(1), dim3(kWG), 0, c, ctr, dst);
                        return hipGetLastError() == hipSuccess;
                    },
                    &ex));
                if (ex) {
                    if (kb == 0) HIM_HIP(hipEventRecord(E[0], s));
                    HIM_HIP(hipGraphLaunch(ex, s));
                    HIM_HIP(hipEventRecord(E[1], s));
                    return HYPERIM_OK;
                }
                // no capture on this device: launch directly (same parities)
            }
            const uint32_t plan_grid =
                (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(plan_sets, kWavesPerWG), 4096));
            for (int i = 0; i < batch; ++i) {
                const uint32_t parity = (uint32_t)((batch_start(kb) + (uint64_t)i) & 1u);
                hipExtLaunchKernelGGL(k_plan, dim3(plan_grid), dim3(kWG), 0, s, kb == 0 && i == 0 ? E[0] : nullptr, nullptr,
                                      0u, ap, parity);
                // timed: the launch itself stamps its start and end events (no
                // stream markers between the kernels)
                if (time_kernels)
                    hipExtLaunchKernelGGL(expand_k, dim3(grid_b), dim3(kWG), 0, s, E[2 + 2 * i], E[3 + 2 * i], 0u,
                                          ap, parity);
                else
                    hipLaunchKernelGGL(expand_k, dim3(grid_b), dim3(kWG), 0, s, ap, parity);
            }
            hipLaunchKernelGGL(k_publish, dim3(1), dim3(kWG), 0, s, ctr, dst);
            HIM_HIP(hipGetLastError());
            HIM_HIP(hipEventRecord(E[1], s));
            return HYPERIM_OK;
        };
        HIM_CHECK(issue(0));
        uint64_t planned_before = 0;
        for (;;) {
            HIM_CHECK(issue(k + 1));   // queued before batch k is read
            HIM_CHECK(wait_event(ws, batch_events(ws, k)[1], s, "a grid-wide superstep batch"));
            const unsigned long long *hb = h + kHostBatch + (k & 1u) * kHostCtr;
            ndef = hb[kDefCount];
            plan_sets = std::max<uint64_t>(ndef, 1);
            const uint32_t last = (uint32_t)((batch_start(k + 1) - 1) & 1u);
            const uint64_t items = hb[kItems + last];
            HIM_CHECK(account(k));
            if (trace)
                fprintf(stderr, "[hyperim] superstep %llu: %llu items, %llu entries planned\n",
                        (unsigned long long)batch_start(k + 1), (unsigned long long)items,
                        (unsigned long long)hb[kPlanned]);
            // the deferred sets hold at most slot_n members each
            const int chk = phase_b_check(planned_before, hb[kPlanned], items,
                                          (uint64_t)a.slot_n * std::max<uint64_t>(ndef, 1));
            if (chk == kLoopDone) break;   // the last superstep found no frontier left
            if (chk != kLoopContinue) {
                HIM_HIP(hipStreamSynchronize(s));
                set_error_detail(chk == kLoopStalled
                                     ? "grid-wide phase stalled: a batch of supersteps with work planned no entry"
                                     : "grid-wide phase planned more entries than its sets can hold");
                return HYPERIM_EHIP;
            }
            planned_before = hb[kPlanned];
            ++k;
        }
        queued = true;   // batch k + 1, which finds no work
    }
    if (ndef) {
        hipExtLaunchKernelGGL(k_finish, dim3((uint32_t)std::min<uint64_t>(ndef, 4096)), dim3(kWG), 0, s,
                              ws.events[2], ws.events[3], 0u, a, (uint32_t)ndef);
        HIM_HIP(hipGetLastError());
        st.launches += 1;
    }
    HIM_HIP(hipMemcpyAsync(h + kHostFinal, ctr, sizeof(unsigned long long) * kCtrWords, hipMemcpyDeviceToHost, s));
    const int rc = tail();
    HIM_HIP(hipStreamSynchronize(s));
    HIM_CHECK(rc);
    float ms = 0.f;
    HIM_HIP(hipEventElapsedTime(&ms, ws.events[0], ws.events[1]));
    st.ms_bfs += ms;
    st.ms_light += ms;
    if (queued) HIM_CHECK(account(k + 1));
    if (ndef) {
        HIM_HIP(hipEventElapsedTime(&ms, ws.events[2], ws.events[3]));
        st.ms_bfs += ms;
        st.ms_heavy += ms;
    }
    st.deferred += h[kHostFinal + kDefCount];
    return HYPERIM_OK;
}

// One launch group of linear-threshold sets: one walk per set (k_lt_walk).
// Ends like run_launch: closing counter block in ws.host + kHostFinal,
// `tail` queued behind it, stream drained.
template <class Tail>
int run_lt_launch(RRWorkspace &ws, RRStats &st, const RRArgs &a, const LaunchShape &shape, uint32_t grid,
                  hipStream_t s, Tail &&tail) {
    unsigned long long *h = ws.host;
    HIM_CHECK(event_pair(ws));
    if (shape.lds)
        hipExtLaunchKernelGGL(k_lt_walk<true>, dim3(grid), dim3(kWG), 0, s, ws.events[0], ws.events[1], 0u, a);
    else
        hipExtLaunchKernelGGL(k_lt_walk<false>, dim3(grid), dim3(kWG), 0, s, ws.events[0], ws.events[1], 0u, a);
    HIM_HIP(hipGetLastError());
    st.launches += 1;
    HIM_HIP(hipMemcpyAsync(h + kHostFinal, a.ctr, sizeof(unsigned long long) * kCtrWords, hipMemcpyDeviceToHost, s));
    const int rc = tail();
    HIM_HIP(hipStreamSynchronize(s));
    HIM_CHECK(rc);
    float ms = 0.f;
    HIM_HIP(hipEventElapsedTime(&ms, ws.events[0], ws.events[1]));
    st.ms_bfs += ms;
    st.ms_light += ms;
    return HYPERIM_OK;
}

// One launch group of stratified-setting sets (k_layered), with the per-lane
// pick lists in the workspace.  Ends like run_launch.
template <class Tail>
int run_layered_launch(RRWorkspace &ws, RRStats &st, const RRArgs &a, const LaunchShape &shape, uint32_t grid,
                       hipStream_t s, Tail &&tail) {
    unsigned long long *h = ws.host;
    HIM_CHECK(ws.picks.reserve(sizeof(uint32_t) * (size_t)grid * kWavesPerWG * kWave * kMaxPick, s));
    HIM_CHECK(event_pair(ws));
    if (shape.lds)
        hipExtLaunchKernelGGL(k_layered<true>, dim3(grid), dim3(kWG), 0, s, ws.events[0], ws.events[1], 0u, a,
                              ws.picks.as<uint32_t>());
    else
        hipExtLaunchKernelGGL(k_layered<false>, dim3(grid), dim3(kWG), 0, s, ws.events[0], ws.events[1], 0u, a,
                              ws.picks.as<uint32_t>());
    HIM_HIP(hipGetLastError());
    st.launches += 1;
    HIM_HIP(hipMemcpyAsync(h + kHostFinal, a.ctr, sizeof(unsigned long long) * kCtrWords, hipMemcpyDeviceToHost, s));
    const int rc = tail();
    HIM_HIP(hipStreamSynchronize(s));
    HIM_CHECK(rc);
    float ms = 0.f;
    HIM_HIP(hipEventElapsedTime(&ms, ws.events[0], ws.events[1]));
    st.ms_bfs += ms;
    st.ms_light += ms;
    return HYPERIM_OK;
}

// Bytes of the bundled-mode state per bundle for a graph of n vertices:
// seen and nxt masks, frontier and next-level lists, output counts, batch marks.
uint64_t ms_bytes_per_bundle(uint32_t n) {
    const uint64_t nvb = div_up(std::max<uint32_t>(n, 1), kMsOutVerts);
    return (uint64_t)n * (8 + 8 + 16 + 8) + nvb * kMsSets * 4 + div_up(n, kWave) * 4 + 4096;
}

// One bundled launch group: ids [0, a.count) of one task (all on graph g),
// bundles of 64 sets grown level by level, then written out in ascending
// order per set.  Ends like run_launch: closing counter block in
// ws.host + kHostFinal, `tail` queued behind it, stream drained.
template <class Tail>
int run_ms_launch(RRWorkspace &ws, RRStats &st, const hyperim_tuning &tune, RRArgs &a, const LaunchShape &shape,
                  hyperim_graph g, const TaskDesc &t, bool trace, bool time_kernels, bool graphs, hipStream_t s,
                  Tail &&tail) {
    const uint32_t n = g->n;
    const uint32_t nbundles = (uint32_t)div_up(a.count, kMsSets);
    const uint64_t stride = std::max<uint32_t>(n, 1);
    const uint64_t list_cap = (uint64_t)nbundles * stride;
    const uint32_t nvb = (uint32_t)div_up(stride, kMsOutVerts);
    if (list_cap >= (1ull << 31)) {
        set_error_detail("bundled launch group too large");
        return HYPERIM_EINVAL;
    }
    HIM_CHECK(ws.ms_seen.reserve(sizeof(unsigned long long) * nbundles * stride, s));
    HIM_CHECK(ws.ms_nxt.reserve(sizeof(unsigned long long) * nbundles * stride, s));
    HIM_CHECK(ws.ms_cur.reserve((sizeof(uint32_t) * 2 + sizeof(unsigned long long)) * list_cap, s));
    HIM_CHECK(ws.ms_next.reserve(sizeof(uint32_t) * 2 * list_cap, s));
    HIM_CHECK(ws.ms_batch.reserve(sizeof(uint32_t) * div_up(list_cap, kWave), s));
    HIM_CHECK(ws.ms_vcnt.reserve(sizeof(uint32_t) * (uint64_t)nbundles * nvb * kMsSets, s));
    HIM_CHECK(ws.ms_ctr.reserve(sizeof(unsigned long long) * kMsNumCtr, s));
    MsArgs m{};
    m.graph = graph_desc(g);
    m.bytesw = g->bytesw.as<unsigned long long>();
    m.first_id = t.first_id;
    m.pool = t.pool;
    m.key0 = t.key0;
    m.key1 = t.key1;
    m.qlog = a.qlog;
    m.nbundles = nbundles;
    m.chunk = a.chunk;
    m.seg = a.seg;
    m.filter = std::max<uint32_t>(tune.ms_filter, 1);
    m.count = a.count;
    m.stride = stride;
    m.seen = ws.ms_seen.as<unsigned long long>();
    m.nxt = ws.ms_nxt.as<unsigned long long>();
    m.cur_b = ws.ms_cur.as<uint32_t>();
    m.cur_v = m.cur_b + list_cap;
    m.cur_m = reinterpret_cast<unsigned long long *>(m.cur_v + list_cap);
    m.nx_b = ws.ms_next.as<uint32_t>();
    m.nx_v = m.nx_b + list_cap;
    m.batch_epoch = ws.ms_batch.as<uint32_t>();
    m.list_cap = list_cap;
    m.ctr = ws.ms_ctr.as<unsigned long long>();
    m.stats = a.ctr;
    m.items = a.items;
    m.vcnt = ws.ms_vcnt.as<uint32_t>();
    m.nvb = nvb;
    // clean state: no set holds anything, no vertex found, no batch planned
    HIM_HIP(hipMemsetAsync(m.seen, 0, sizeof(unsigned long long) * nbundles * stride, s));
    HIM_HIP(hipMemsetAsync(m.nxt, 0, sizeof(unsigned long long) * nbundles * stride, s));
    HIM_HIP(hipMemsetAsync(m.batch_epoch, 0, sizeof(uint32_t) * div_up(list_cap, kWave), s));
    HIM_HIP(hipMemsetAsync(m.ctr, 0, sizeof(unsigned long long) * kMsNumCtr, s));
    ws.host[kHostMsStart] = 1;
    HIM_HIP(hipMemcpyAsync(m.ctr + kMsLevelDone, ws.host + kHostMsStart, sizeof(unsigned long long),
                           hipMemcpyHostToDevice, s));
    HIM_CHECK(event_pair(ws));
    HIM_HIP(hipEventRecord(ws.events[0], s));
    const uint32_t grid_b = shape.grid_b;
    hipLaunchKernelGGL(k_ms_roots, dim3((uint32_t)div_up(a.count, kWG)), dim3(kWG), 0, s, m, a);
    hipLaunchKernelGGL(k_ms_advance, dim3(grid_b), dim3(kWG), 0, s, m);
    hipLaunchKernelGGL(k_ms_ctl_advanced, dim3(1), dim3(1), 0, s, m.ctr, list_cap);
    HIM_HIP(hipGetLastError());
    // levels: plan, expand, bookkeeping, advance, bookkeeping; a level whose
    // items overflow the buffer takes several steps
    const int per_sync = (int)std::min<uint32_t>(std::max<uint32_t>(tune.steps_per_sync, 1), kMaxBatch);
    hipEvent_t *E = batch_events(ws, 0);
    uint64_t steps = 0;
    float ms = 0.f;
    // progress: (level epoch, pending frontier batches) before this batch
    uint64_t epoch_before = 0, pending_before = ~0ull;
    const unsigned long long *hm = ws.host + kHostBatch;
    static_assert(kMsNumCtr <= kHostCtr, "bundled counter block");
    // a batch of steps and the counter copy, captured once for the group
    // (the arguments are the group's) and replayed until the sets are done
    struct ExecGuard {
        hipGraphExec_t ex = nullptr;
        ~ExecGuard() {
            if (ex) (void)hipGraphExecDestroy(ex);
        }
    } batch_exec;
    auto record_batch = [&](hipStream_t c, int batch) {
        for (int k = 0; k < batch; ++k) {
            hipLaunchKernelGGL(k_ms_plan, dim3(grid_b), dim3(kWG), 0, c, m);
            if (time_kernels) {
                hipExtLaunchKernelGGL(k_ms_expand, dim3(grid_b), dim3(kWG), 0, c, E[2 + 2 * k], E[3 + 2 * k], 0u, m);
            } else {
                hipLaunchKernelGGL(k_ms_expand, dim3(grid_b), dim3(kWG), 0, c, m);
            }
            hipLaunchKernelGGL(k_ms_ctl_expanded, dim3(1), dim3(1), 0, c, m.ctr);
            hipLaunchKernelGGL(k_ms_advance, dim3(grid_b), dim3(kWG), 0, c, m);
            hipLaunchKernelGGL(k_ms_ctl_advanced, dim3(1), dim3(1), 0, c, m.ctr, list_cap);
        }
        return hipMemcpyAsync(ws.host + kHostBatch, m.ctr, sizeof(unsigned long long) * kMsNumCtr,
                              hipMemcpyDeviceToHost, c) == hipSuccess;
    };
    // (launches timed one by one are not captured, as in run_launch)
    if (graphs && !trace && !time_kernels)
        HIM_CHECK(capture_graph(ws, [&](hipStream_t c) { return record_batch(c, per_sync); }, &batch_exec.ex));
    for (;;) {
        const int batch = trace ? 1 : per_sync;
        if (batch_exec.ex) {
            HIM_HIP(hipGraphLaunch(batch_exec.ex, s));
        } else if (!record_batch(s, batch)) {
            HIM_HIP(hipGetLastError());
            set_error_detail("bundled superstep batch: a launch or copy failed");
            return HYPERIM_EHIP;
        }
        HIM_HIP(hipGetLastError());
        steps += batch;
        HIM_HIP(hipEventRecord(E[1], s));
        HIM_CHECK(wait_event(ws, E[1], s, "a bundled superstep batch"));
        const uint64_t done = hm[kMsDone];
        // a level adds at least one new (set, member) pair, so levels are
        // bounded by the members of the group's sets
        const int chk = bundled_check(epoch_before, pending_before, hm[kMsEpoch], hm[kMsPending], done,
                                      (uint64_t)nbundles * kMsSets * stride + 2);
        if (chk == kLoopStalled || chk == kLoopOverBound) {
            set_error_detail(chk == kLoopStalled ? "bundled generation stalled: a batch of steps changed no level"
                                                 : "bundled generation ran more levels than its sets can have");
            return HYPERIM_EHIP;
        }
        epoch_before = hm[kMsEpoch];
        pending_before = hm[kMsPending];
        for (int k = 0; time_kernels && k < batch; ++k) {
            float me = 0.f;
            HIM_HIP(hipEventElapsedTime(&me, E[2 + 2 * k], E[3 + 2 * k]));
            st.ms_bundled += me;
        }
        st.bundled_launches += batch;
        st.supersteps += batch;
        st.launches += 5 * batch;
        if (trace) {
            uint64_t cur = 0;
            HIM_CHECK(read_ctr(s, m.ctr, kMsCur, &cur));
            fprintf(stderr, "[hyperim] bundled step %llu: frontier %llu\n", (unsigned long long)steps,
                    (unsigned long long)cur);
        }
        if (done) break;
    }
    uint64_t overflow = 0;
    HIM_CHECK(read_ctr(s, m.ctr, kMsOverflow, &overflow));
    if (overflow) {
        set_error_detail("bundled frontier list overflow");
        return HYPERIM_EHIP;
    }
    // output: counts per vertex block, set ranges, members in ascending order
    const uint32_t out_grid = nbundles * nvb;
    hipLaunchKernelGGL(k_ms_count, dim3(out_grid), dim3(kWG), 0, s, m);
    hipLaunchKernelGGL(k_ms_record, dim3((uint32_t)div_up(a.count, kWG)), dim3(kWG), 0, s, m, a);
    hipLaunchKernelGGL(k_ms_write, dim3(out_grid), dim3(kWG), 0, s, m, a);
    HIM_HIP(hipGetLastError());
    HIM_HIP(hipMemcpyAsync(ws.host + kHostFinal, a.ctr, sizeof(unsigned long long) * kCtrWords, hipMemcpyDeviceToHost,
                           s));
    HIM_HIP(hipEventRecord(ws.events[3], s));
    const int rc = tail();
    HIM_HIP(hipStreamSynchronize(s));
    HIM_CHECK(rc);
    HIM_HIP(hipEventElapsedTime(&ms, ws.events[0], ws.events[3]));
    st.ms_bfs += ms;
    st.ms_heavy += ms;
    st.launches += 6;
    return HYPERIM_OK;
}

}  // namespace

namespace {

// Appending the staged sets with group-local indices [first, first + count)
// to pool p takes two steps around a wait for the stream.  compact_scan
// queues the offsets (an exclusive scan of the sizes from p's total) and the
// copy of the new total into *total_host.
int compact_scan(RRWorkspace &ws, hyperim_pool p, uint64_t first, uint64_t count, unsigned long long *total_host,
                 hipStream_t s) {
    if (count == 0) return HYPERIM_OK;
    HIM_CHECK(pool_reserve(p, count, 0, s));
    uint64_t *dst_off = p->off + p->count;
    HIM_CHECK(scan_u32_to_u64(ws.sizes.as<uint32_t>() + first, dst_off, count, p->total, ws.scan_tmp, s));
    HIM_HIP(hipMemcpyAsync(total_host, dst_off + count, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    return HYPERIM_OK;
}

// compact_move, once the new total is on the host, grows p's storage and
// moves the members and roots (HYPERIM_ECAPACITY beyond max_entries or a
// caller buffer; the pool is then unchanged).
int compact_move(RRWorkspace &ws, hyperim_pool p, uint64_t first, uint64_t count, uint64_t new_total,
                 uint64_t max_entries, hipStream_t s) {
    if (count == 0) return HYPERIM_OK;
    if (max_entries && new_total > max_entries) {
        set_error_detail("pool would exceed max_entries");
        return HYPERIM_ECAPACITY;
    }
    HIM_CHECK(pool_reserve(p, count, new_total - p->total, s));
    uint64_t *dst_off = p->off + p->count;   // storage may have moved
    HIM_HIP(hipMemcpyAsync(p->roots + p->count, ws.roots.as<uint32_t>() + first, sizeof(uint32_t) * count,
                           hipMemcpyDeviceToDevice, s));
    // lanes per set by the mean size
    const uint64_t mean = (new_total - p->total) / count;
    const uint32_t lanes = mean < 16 ? 4u : mean < 128 ? 16u : 64u;
    const auto move = lanes == 4u ? k_move_small<4> : lanes == 16u ? k_move_small<16> : k_move_small<64>;
    const uint32_t grid = (uint32_t)std::min<uint64_t>(div_up(count, kWG / lanes), 65535u);
    hipLaunchKernelGGL(move, dim3(std::max<uint32_t>(grid, 1)), dim3(kWG), 0, s,
                       ws.stage_off.as<uint64_t>() + first, ws.sizes.as<uint32_t>() + first, dst_off, count,
                       ws.stage.as<uint32_t>(), p->mem);
    hipLaunchKernelGGL(k_move_big, dim3(1024), dim3(kWG), 0, s, ws.big_ids.as<uint64_t>(),
                       ws.counters.as<unsigned long long>() + kBigCount, first, count, ws.stage_off.as<uint64_t>(),
                       ws.sizes.as<uint32_t>(), dst_off, ws.stage.as<uint32_t>(), p->mem);
    HIM_HIP(hipGetLastError());
    p->count += count;
    p->total = new_total;
    return HYPERIM_OK;
}

}  // namespace

size_t rr_slot_bytes(uint32_t n_max, bool lean) {
    SlotLayout L;
    return slot_layout(n_max, lean, &L) == HYPERIM_OK ? (size_t)L.bytes : 0;
}

int rr_generate_into(RRWorkspace &ws, RRStats &st, const std::vector<RRTask> &tasks,
                     const std::vector<hyperim_pool> &pools, uint32_t qlog, int form, uint64_t max_entries,
                     uint64_t stage_budget, hipStream_t s, std::vector<int> &pool_status, bool time_kernels,
                     bool graphs, bool lean) {
    // HYPERIM_TRACE=1: synchronise after every grid-wide superstep and report
    // its item count and time on stderr (diagnostics; same results)
    static const bool trace = [] {
        const char *e = getenv("HYPERIM_TRACE");
        return e && e[0] == '1';
    }();
    pool_status.assign(tasks.size(), HYPERIM_OK);
    if (tasks.empty()) return HYPERIM_OK;
    if (!ws.settled()) {
        set_error_detail("an earlier generation call gave up waiting and its work still runs");
        return HYPERIM_EHIP;
    }
    // a launch group compacts its slices after one wait, so each task needs a
    // pool of its own
    std::vector<hyperim_pool> sorted(pools);
    std::sort(sorted.begin(), sorted.end());
    if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end()) {
        set_error_detail("two tasks of one generation call share a pool");
        return HYPERIM_EINVAL;
    }
    // execution parameters of the first task's graph
    const hyperim_tuning &tune = tasks[0].g->tune;
    // graph descriptors (one per distinct graph)
    std::map<hyperim_graph, uint32_t> gid;
    std::vector<GraphDesc> gdesc;
    uint32_t n_max = 1;
    for (const RRTask &t : tasks) {
        if (gid.count(t.g)) continue;
        gid[t.g] = (uint32_t)gdesc.size();
        hyperim_graph g = t.g;
        gdesc.push_back(graph_desc(g));
        n_max = std::max(n_max, g->n);
    }
    uint64_t count = 0;
    for (const RRTask &t : tasks) count += t.id_end - t.id_begin;
    if (count == 0) return HYPERIM_OK;
    LaunchShape shape;
    HIM_CHECK(ensure_workspace(ws, n_max, lean, s, &shape));

    // launch shapes: the occupancy limits, capped per compute unit by the tuning
    auto capped = [&](uint32_t full, uint32_t per_cu) {
        return per_cu ? std::max<uint32_t>(1, std::min<uint32_t>(full, shape.cus * per_cu)) : full;
    };
    const uint32_t grid_a = capped(shape.grid, tune.blocks_a);
    const uint32_t grid_b = capped(shape.grid_b, tune.blocks_b);
    const size_t ndef_cap = shape.slots;   // stride of the deferred-set arrays
    const size_t spare = std::max<uint64_t>(shape.slots - (uint64_t)grid_a * kWavesPerWG, 1);

    // Launch groups are contiguous ranges of launch indices (the tasks laid
    // back to back), planned one at a time with what earlier groups taught.
    // A group's sets are staged, then compacted into their pools before the
    // next group runs, so the stage holds one group.  A group takes indices
    // while its predicted members fit the stage budget -- 1.3 x the graph's
    // members per set seen so far, or n (an upper bound) for a graph not
    // seen yet, whose first group then stops after kLearnIds of its sets
    // unless that bound fits for all of them and the graph has no bundled
    // mode to decide -- and (form 0) while the sets
    // it defers fit the spare slots at the
    // deferral rate seen so far (a set that finds no spare slot stays with
    // its wave).  The plain form (1) also ends a group at every (task, ladder
    // block, stratum) boundary.
    constexpr uint64_t kLearnIds = 2048;
    constexpr uint64_t kMsBudget = 8ull << 30;   // bytes of bundled-mode state per launch group
    // bundled mode for graphs whose sets are large on average (form 0 only;
    // the plain form keeps one traversal per set)
    // (a graph not seen yet starts bundled when its tuning enables the mode:
    // the first group's sets teach the estimate either way, and a graph tuned
    // for bundled mode has large sets, which the per-set mode grows slowly)
    auto bundled = [&](const RRTask &t) {
        return form == 0 && t.g->kind() == 0 && tune.ms_min != 0xFFFFFFFFu &&
               (t.g->rr_members < 0.0 || t.g->rr_members >= (double)tune.ms_min);
    };
    const double stage_words = (double)stage_budget / 4.0;
    auto per_set = [](hyperim_graph g) { return g->rr_members >= 0.0 ? 1.3 * g->rr_members + 1.0 : (double)g->n; };
    std::vector<uint64_t> tstart(tasks.size() + 1, 0);
    for (size_t i = 0; i < tasks.size(); ++i) tstart[i + 1] = tstart[i] + (tasks[i].id_end - tasks[i].id_begin);
    // unit boundaries: task ends (form 0), (task, block, stratum) ends (form 1)
    std::vector<uint64_t> unit_end;
    for (size_t i = 0; i < tasks.size(); ++i) {
        const RRTask &t = tasks[i];
        if (form == 1) {
            std::vector<std::pair<uint64_t, uint64_t>> ranges;
            stratum_ranges(t.g, t.seed, t.instance, qlog, t.pool, t.id_begin, t.id_end, &ranges);
            for (const auto &rg : ranges) unit_end.push_back(tstart[i] + (rg.second - t.id_begin));
        } else {
            unit_end.push_back(tstart[i + 1]);
        }
    }

    unsigned long long *ctr = ws.counters.as<unsigned long long>();
    RRArgs a{};
    a.qlog = qlog;
    a.heavy = tune.heavy;
    a.budget = tune.budget;
    a.reach = std::max(tune.budget, kReach);
    a.chunk = tune.chunk;
    a.seg = std::max(tune.seg, tune.chunk);
    a.prefilter_min = tune.prefilter_min;
    a.slot_n = shape.slot_n;
    a.slot_words = shape.slot_words;
    a.ctr = ctr;
    a.lists = ws.lists.as<uint32_t>();
    a.bitmaps = ws.bitmaps.as<uint32_t>();
    a.slot_total = shape.slots;
    a.out_base = 0;
    a.def_idx = ws.def_idx.as<uint64_t>();
    a.def_root = ws.def_u32.as<uint32_t>();
    a.def_slot = a.def_root + ndef_cap;
    a.def_head = a.def_slot + ndef_cap;
    a.def_size = a.def_head + ndef_cap;
    a.def_task = a.def_size + ndef_cap;
    a.items = ws.items.as<uint4>();
    HIM_CHECK(ws.graph_desc.reserve(sizeof(GraphDesc) * gdesc.size(), s));
    HIM_CHECK(ws.task_desc.reserve(sizeof(TaskDesc) * tasks.size(), s));
    // pinned staging: fixed words, then the pools' new totals (one per
    // task), task descriptors, graph descriptors
    auto words = [](size_t bytes) { return (bytes + sizeof(unsigned long long) - 1) / sizeof(unsigned long long); };
    const size_t host_totals = kHostFixed;
    const size_t host_tasks = host_totals + tasks.size();
    const size_t host_graphs = host_tasks + words(sizeof(TaskDesc) * tasks.size());
    HIM_CHECK(ensure_host(ws, host_graphs + words(sizeof(GraphDesc) * gdesc.size())));
    GraphDesc *gstage = reinterpret_cast<GraphDesc *>(ws.host + host_graphs);
    std::copy(gdesc.begin(), gdesc.end(), gstage);
    HIM_HIP(hipMemcpyAsync(ws.graph_desc.ptr, gstage, sizeof(GraphDesc) * gdesc.size(), hipMemcpyHostToDevice, s));
    a.graphs = ws.graph_desc.as<GraphDesc>();

    struct Slice {
        size_t task;
        uint64_t lo, hi;   // launch indices
    };
    size_t unit = 0;
    for (uint64_t pos = 0; pos < count;) {
        // ---- plan the next group ---------------------------------------
        double rate = 0.0;
        for (const RRTask &t : tasks) rate = std::max(rate, t.g->rr_defer >= 0.0 ? t.g->rr_defer : 0.5);
        const uint64_t def_chunk =
            form == 0 ? std::max<uint64_t>((uint64_t)((double)spare / std::max(rate * 1.25, 1.0 / 64.0)), 4096)
                      : ~0ull;
        const uint64_t lo = pos;
        double acc = 0.0;
        size_t ti = std::upper_bound(tstart.begin(), tstart.end(), pos) - tstart.begin() - 1;
        while (unit_end[unit] <= pos) ++unit;
        const bool ms = bundled(tasks[ti]);
        if (ms) {
            // bundled mode: one task, as many sets as the stage and the
            // bundle memory allow
            const RRTask &t = tasks[ti];
            const uint64_t rest = tstart[ti + 1] - pos;
            const uint64_t max_sets =
                kMsSets * std::max<uint64_t>(1, kMsBudget / ms_bytes_per_bundle(t.g->n));
            const double m = per_set(t.g);
            uint64_t take = std::min<uint64_t>(rest, max_sets);
            take = std::min<uint64_t>(take, std::max<uint64_t>(1, (uint64_t)(stage_words / m)));
            // the ids of a group share their upper words (ms_m0)
            const uint64_t id0 = t.id_begin + (pos - tstart[ti]);
            take = std::min<uint64_t>(take, (1ull << 32) - (id0 & 0xFFFFFFFFull));
            acc = (double)take * m;
            pos += take;
        }
        for (; !ms;) {
            const RRTask &t = tasks[ti];
            const double m = per_set(t.g);
            const bool learn = t.g->rr_members < 0.0;
            const uint64_t rest = (form == 1 ? unit_end[unit] : tstart[ti + 1]) - pos;
            const double room = stage_words - acc;
            // a graph not seen yet stops its first group after kLearnIds sets,
            // unless the worst case of all its remaining sets fits already and
            // no bundled mode waits for what the group would teach
            const bool cap = learn && ((double)rest * m > room || t.g->tune.ms_min != 0xFFFFFFFFu);
            const uint64_t limit = cap ? std::min(rest, kLearnIds) : rest;
            uint64_t take = std::min<uint64_t>(limit, room > 0.0 ? (uint64_t)(room / m) : 0);
            take = std::min<uint64_t>(take, def_chunk - (pos - lo));
            if (take == 0 && pos == lo) take = 1;   // one set always fits
            acc += (double)take * m;
            pos += take;
            if (take < rest || pos == count || form == 1 || pos - lo >= def_chunk) break;
            ++ti;   // form 0: the group continues with the next task ...
            // ... unless that one runs bundled or has the other cascade model
            if (bundled(tasks[ti]) || tasks[ti].g->kind() != tasks[ti - 1].g->kind()) break;
        }
        const uint64_t hi = pos;
        // descriptors of the group's task slices
        std::vector<TaskDesc> tdesc;
        std::vector<Slice> slices;
        for (size_t i = 0; i < tasks.size(); ++i) {
            const uint64_t a0 = std::max(lo, tstart[i]), a1 = std::min(hi, tstart[i + 1]);
            if (a0 >= a1) continue;
            const RRTask &t = tasks[i];
            tdesc.push_back(TaskDesc{a1 - lo, t.id_begin + (a0 - tstart[i]), t.pool, gid[t.g], (uint32_t)t.seed,
                                     t.instance});
            slices.push_back(Slice{i, a0, a1});
        }
        const uint64_t n_ids = hi - lo;
        HIM_CHECK(ws.stage_off.reserve(sizeof(uint64_t) * n_ids, s, false));
        HIM_CHECK(ws.sizes.reserve(sizeof(uint32_t) * n_ids, s, false));
        HIM_CHECK(ws.roots.reserve(sizeof(uint32_t) * n_ids, s, false));
        HIM_CHECK(ws.big_ids.reserve(sizeof(uint64_t) * n_ids, s, false));
        // stage sized from the prediction (a miss re-runs the group)
        const uint64_t predicted = (uint64_t)acc + 4 * n_ids + (1u << 20);
        if (ws.stage.bytes < sizeof(uint32_t) * predicted)
            HIM_CHECK(ws.stage.reserve(sizeof(uint32_t) * predicted, s, false));
        // descriptors go through the pinned staging (the previous group has drained)
        TaskDesc *tstage = reinterpret_cast<TaskDesc *>(ws.host + host_tasks);
        std::copy(tdesc.begin(), tdesc.end(), tstage);
        HIM_HIP(hipMemcpyAsync(ws.task_desc.ptr, tstage, sizeof(TaskDesc) * tdesc.size(), hipMemcpyHostToDevice, s));
        a.tasks = ws.task_desc.as<TaskDesc>();
        a.ntasks = (uint32_t)tdesc.size();
        a.count = n_ids;
        a.stage_off = ws.stage_off.as<uint64_t>();
        a.sizes = ws.sizes.as<uint32_t>();
        a.roots = ws.roots.as<uint32_t>();
        a.big_ids = ws.big_ids.as<uint64_t>();
        const uint32_t grid =
            form == 0 ? grid_a : (uint32_t)std::min<uint64_t>(grid_a, div_up(a.count, kWavesPerWG));
        // Index by index where a wave has few; eight grabs a wave or more, so
        // that the last ones are short.
        a.take = (uint32_t)std::clamp<uint64_t>(a.count / ((uint64_t)grid * kWavesPerWG * 8), 1, 8);
        a.free0 = grid * kWavesPerWG;
        // a graph whose sets were never deferred before is checked after phase
        // A, a small one (marks in LDS) until one of its sets was
        bool expect_defer = false;
        for (const Slice &sl : slices)
            expect_defer |= shape.lds ? tasks[sl.task].g->rr_defer > 0.0 : tasks[sl.task].g->rr_defer != 0.0;
        // compaction offsets of every slice, queued behind the launch so that
        // one wait covers both (a launch whose stage overflowed discards them)
        std::vector<int> scan_rc(slices.size(), HYPERIM_OK);
        auto scans = [&]() -> int {
            for (size_t i = 0; i < slices.size(); ++i) {
                const Slice &sl = slices[i];
                scan_rc[i] = HYPERIM_OK;
                if (pool_status[sl.task] != HYPERIM_OK) continue;
                const int rc = compact_scan(ws, pools[sl.task], sl.lo - lo, sl.hi - sl.lo, ws.host + host_totals + i, s);
                if (rc == HYPERIM_ECAPACITY) scan_rc[i] = rc;
                else if (rc != HYPERIM_OK) return rc;
            }
            return HYPERIM_OK;
        };

        // ---- run it ----------------------------------------------------
        bool staged = false;
        for (int attempt = 0; attempt < 2 && !staged; ++attempt) {
            a.stage = ws.stage.as<uint32_t>();
            a.stage_cap = ws.stage.bytes / sizeof(uint32_t);
            // Of the stage, what the waves have left at the end is at most 1/32
            // (8192 waves), what they left between steps at most a seventh of
            // the members staged that way.  A second attempt leaves nothing:
            // it needs no more than the first one asked for.
            a.stage_step = attempt ? 0u : (uint32_t)std::min<uint64_t>(256, a.stage_cap >> 18);
            HIM_HIP(hipMemsetAsync(ctr, 0, sizeof(unsigned long long) * kCtrWords, s));
            RRStats run{};
            if (ms)
                HIM_CHECK(run_ms_launch(ws, run, tune, a, shape, tasks[slices[0].task].g, tdesc[0], trace,
                                        time_kernels, graphs, s, scans));
            else if (tasks[slices[0].task].g->lt())
                HIM_CHECK(run_lt_launch(ws, run, a, shape, grid, s, scans));
            else if (tasks[slices[0].task].g->layered())
                HIM_CHECK(run_layered_launch(ws, run, a, shape, grid, s, scans));
            else
                HIM_CHECK(run_launch(ws, run, tune, a, shape, grid, grid_b, expect_defer, trace, time_kernels,
                                     graphs, tasks[slices[0].task].g->gaps(), s, scans));
            // time counts every attempt, work only the one that produced the output
            st.ms_bfs += run.ms_bfs;
            st.ms_light += run.ms_light;
            st.ms_heavy += run.ms_heavy;
            st.launches += run.launches;
            st.supersteps += run.supersteps;
            st.ms_expand += run.ms_expand;
            st.expand_launches += run.expand_launches;
            st.ms_bundled += run.ms_bundled;
            st.bundled_launches += run.bundled_launches;
            const unsigned long long *hf = ws.host + kHostFinal;
            const uint64_t bump = hf[kBump];
            for (const Slice &sl : slices) tasks[sl.task].g->rr_defer = (double)run.deferred / (double)a.count;
            if (bump <= a.stage_cap) {
                st.deferred += run.deferred;
                const uint64_t px_light = stat_sum(hf, kPhiloxA), px_bundled = stat_sum(hf, kPhiloxMs);
                st.bytes_light += stat_sum(hf, kBytesA);
                st.bytes_heavy += stat_sum(hf, kBytesB);
                st.bytes_bundled += stat_sum(hf, kBytesMs);
                st.philox += px_light + stat_sum(hf, kPhilox) + px_bundled;
                st.philox_light += px_light;
                st.philox_bundled += px_bundled;
                staged = true;
            } else {
                HIM_CHECK(ws.stage.reserve(sizeof(uint32_t) * (size_t)(bump + bump / 4 + 1024), s, false));
            }
        }
        if (!staged) {
            set_error_detail("RR stage overflow after resize");
            return HYPERIM_ENOMEM;
        }

        // ---- compact it ------------------------------------------------
        for (size_t i = 0; i < slices.size(); ++i) {
            const Slice &sl = slices[i];
            if (pool_status[sl.task] != HYPERIM_OK) continue;
            hyperim_pool p = pools[sl.task];
            const uint64_t before = p->total;
            int rc = scan_rc[i];
            if (rc == HYPERIM_OK)
                rc = compact_move(ws, p, sl.lo - lo, sl.hi - sl.lo, ws.host[host_totals + i], max_entries, s);
            if (rc == HYPERIM_ECAPACITY) {
                pool_status[sl.task] = rc;   // this pool is full; the others go on
            } else if (rc != HYPERIM_OK) {
                return rc;
            } else {
                // members per set of this graph, learned for later predictions
                hyperim_graph g = tasks[sl.task].g;
                g->rr_seen_sets += sl.hi - sl.lo;
                g->rr_seen_members += p->total - before;
                g->rr_members = (double)g->rr_seen_members / (double)g->rr_seen_sets;
            }
        }
    }
    return HYPERIM_OK;
}

int rr_incidences(hyperim_graph g, hyperim_pool p, uint64_t theta, hipStream_t s, RRWork *out) {
    uint64_t entries = 0;
    HIM_HIP(hipMemcpyAsync(&entries, p->off + theta, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    DevBuf acc;
    HIM_CHECK(acc.reserve(4 * sizeof(unsigned long long), s));
    HIM_HIP(hipMemsetAsync(acc.ptr, 0, 4 * sizeof(unsigned long long), s));
    if (entries) {
        const uint32_t grid = (uint32_t)std::min<uint64_t>(div_up(entries, kWG), 4096);
        hipLaunchKernelGGL(k_weight_sum, dim3(grid), dim3(kWG), 0, s, p->mem, entries,
                           g->weight.as<unsigned long long>(), g->bytesw.as<unsigned long long>(),
                           g->c.as<unsigned long long>(), g->phiw.as<unsigned long long>(),
                           acc.as<unsigned long long>());
    }
    unsigned long long v[4] = {0, 0, 0, 0};
    HIM_HIP(hipMemcpyAsync(v, acc.ptr, sizeof(v), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    acc.release();
    out->incidences = v[0];
    out->alg_bytes = v[1];
    out->coins = v[2];
    out->philox = v[3];
    return HYPERIM_OK;
}

}  // namespace hyperim
