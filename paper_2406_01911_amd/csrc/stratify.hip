// Sample-set division (Section 3.1.1) on the device.  For every vertex v the
// co-membership weight w(v,u) (hyperedges shared with u) of its co-members is
// counted; the layers of A(v) are the distinct w values, layer 1 the largest.
// Per vertex this yields l_v (number of layers), deg(v) = |A(v)| and top(v) =
// n(L_1).  Strata are log2 buckets of l_v, and P lists the vertices by
// (stratum, id) for stratified roots.
//
// A vertex's c(v) co-member occurrences (its hyperedges' members, itself left
// out) are counted where they fit, so that each is read once and no pair table
// goes through memory:
//   c <= 64             in the registers of one wave, one occurrence per lane;
//   c <= kWavePairs     in one wave's LDS hash table;
//   c <= kDensePairs    in one workgroup's LDS hash table (two sizes), in
//                       several passes over parts of the ids when the distinct
//                       co-members may outnumber it;
//   above, or above n / 16 (hubs)  in a row of n counters in device memory, the hub's
//                       incidences and then its counters spread over the grid.
// Reading and counting bound every class (LDS atomics; device atomics for the
// hubs).  A million vertices with 3.4e8 occurrences (Zipf 1.1 members): 46 ms
// when all pairs went through two hash tables in device memory, 10 ms now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "block_table.h"
#include "dev_common.h"
#include "internal.h"

namespace hyperim {
namespace {

constexpr int kBlock = 256;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;        // vertex ids are below 2^31
constexpr uint32_t kWavePairs = 512;            // one wave's table: load at most one half
constexpr uint32_t kBlockPairs = 3072;          // the small workgroup table
constexpr uint32_t kBlockTable = 16384;         // slots of the large one (ids up to three quarters of it)
constexpr uint32_t kDensePairs = 131072;        // ... in up to 11 passes
constexpr uint64_t kDenseBudget = 2ull << 30;   // bytes of hub counters and weight marks per batch
constexpr int kWavesPerBlock = kBlock / kWave;

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}

// What one call needs of the host: class counts, sizes, sums (device copy).
struct PrepInfo {
    uint32_t n_wave, n_block, n_big, n_hub;   // vertices per class (the rest is in registers)
    uint32_t dmax, lmax;                      // hyperedges of the largest hub; largest l_v
    unsigned long long cmax;                  // largest c(v)
    unsigned long long sum_top, sum_deg, sum_l;
    unsigned long long B[kNStrata];
};

// Incidence spans of one wave, flattened: body(u) for every member of the
// incidences [e0, e1) of irec (at most 64), v itself left out; `u` is valid
// where the lane has one (else kNoKey), and every lane calls body together.
struct SpanLds {
    uint32_t scan[kWave], hb[kWave];
};
template <class Body>
__device__ __forceinline__ void wave_members(SpanLds &L, const uint4 *__restrict__ irec,
                                             const uint32_t *__restrict__ he_mem, uint64_t e0, uint64_t e1, uint32_t v,
                                             Body &&body) {
    const uint32_t lane = lane_id();
    uint4 rec = make_uint4(0u, 0u, 0u, 0u);
    if (e0 + lane < e1) rec = irec[e0 + lane];
    const uint32_t incl = wave_incl_scan(rec.z);
    const uint32_t total = wave_bcast(incl, kWave - 1);
    wave_sync();
    L.scan[lane] = incl;
    L.hb[lane] = rec.y;
    wave_sync();
    for (uint32_t b = 0; b < total; b += kWave) {
        const uint32_t q = b + lane;
        uint32_t u = kNoKey;
        if (q < total) {
            const uint32_t k = search64(L.scan, q);
            u = he_mem[L.hb[k] + (q - (k ? L.scan[k - 1] : 0u))];
            if (u == v) u = kNoKey;
        }
        body(u);
    }
}

// Counts one occurrence of `u` in an LDS table of kSlots slots; false when the
// table is full.
template <uint32_t kSlots>
__device__ __forceinline__ bool lds_count(uint32_t *key, uint32_t *cnt, uint32_t u) {
    uint32_t h = mix32(u) & (kSlots - 1u);
    for (uint32_t p = 0; p < kSlots; ++p) {
        uint32_t cur = __hip_atomic_load(&key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == kNoKey) {
            cur = atomicCAS(&key[h], kNoKey, u);
            if (cur == kNoKey) cur = u;
        }
        if (cur == u) {
            atomicAdd(&cnt[h], 1u);
            return true;
        }
        h = (h + 1u) & (kSlots - 1u);
    }
    return false;
}

// Vertices of each class above 64 occurrences, and the largest c(v) and hub.
// kClassPer vertices per thread: one device atomic per workgroup and class
// (one per wave took 0.59 ms on a million vertices).
constexpr uint32_t kClassPer = 16;

__global__ __launch_bounds__(kBlock) void k_classify(uint32_t n, uint32_t dense, const unsigned long long *__restrict__ c,
                                                      const uint32_t *__restrict__ v_off, uint32_t *__restrict__ lists,
                                                      PrepInfo *__restrict__ info) {
    __shared__ uint32_t cnt[4], base[4], dm_s;
    __shared__ unsigned long long cm_s;
    if (threadIdx.x < 4) cnt[threadIdx.x] = 0u;
    if (threadIdx.x == 4) {
        dm_s = 0u;
        cm_s = 0ull;
    }
    __syncthreads();
    const uint64_t v0 = (uint64_t)blockIdx.x * kBlock * kClassPer + threadIdx.x;
    int cls[kClassPer];
    uint32_t at[kClassPer], dm = 0;
    unsigned long long cm = 0;
#pragma unroll
    for (uint32_t r = 0; r < kClassPer; ++r) {
        const uint64_t v = v0 + r * kBlock;
        const unsigned long long cv = v < n ? c[v] : 0ull;
        cls[r] = cv <= kWave ? -1 : cv <= kWavePairs ? 0 : cv <= kBlockPairs ? 1 : cv <= dense ? 2 : 3;
        cm = cv > cm ? cv : cm;
        if (cls[r] == 3) dm = max(dm, v_off[v + 1] - v_off[v]);
        if (cls[r] >= 0) at[r] = atomicAdd(&cnt[cls[r]], 1u);
    }
    cm = wave_max(cm);
    dm = wave_max(dm);
    if (lane_id() == 0) {
        atomicMax(&cm_s, cm);
        atomicMax(&dm_s, dm);
    }
    __syncthreads();
    if (threadIdx.x < 4 && cnt[threadIdx.x]) base[threadIdx.x] = atomicAdd(&info->n_wave + threadIdx.x, cnt[threadIdx.x]);
    if (threadIdx.x == 4) {
        if (cm_s) atomicMax(&info->cmax, cm_s);
        if (dm_s) atomicMax(&info->dmax, dm_s);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kClassPer; ++r)
        if (cls[r] >= 0) lists[(uint64_t)cls[r] * n + base[cls[r]] + at[r]] = (uint32_t)(v0 + r * kBlock);
}

// c(v) <= 64: lane i holds occurrence i; equal lanes are counted by a loop
// over the occurrences.  A wave takes 64 consecutive vertices, one after
// another.
__global__ __launch_bounds__(kBlock) void k_layers_reg(uint32_t n, const unsigned long long *__restrict__ c,
                                                        const uint32_t *__restrict__ v_off,
                                                        const uint4 *__restrict__ irec,
                                                        const uint32_t *__restrict__ he_mem, uint32_t *__restrict__ deg,
                                                        uint32_t *__restrict__ l, uint32_t *__restrict__ top) {
    __shared__ SpanLds spans[kWavesPerBlock];
    __shared__ uint32_t occ_s[kWavesPerBlock][kWave];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    uint32_t *occ = occ_s[wv];
    const uint64_t v0 = ((uint64_t)blockIdx.x * kWavesPerBlock + wv) * kWave, mine = v0 + lane;
    unsigned long long cv = ~0ull;
    uint32_t off0 = 0, off1 = 0;
    if (mine < n) {
        cv = c[mine];
        off0 = v_off[mine];
        off1 = v_off[mine + 1];
    }
    uint32_t rdeg = 0, rl = 0, rtop = 0;   // of this lane's vertex
    for (uint64_t todo = __ballot(cv != 0ull && cv <= kWave); todo; todo &= todo - 1ull) {
        const int k = __ffsll((unsigned long long)todo) - 1;
        const uint32_t v = (uint32_t)v0 + (uint32_t)k, e0 = wave_bcast(off0, k), e1 = wave_bcast(off1, k);
        uint32_t count = 0;   // occurrences found (wave-uniform)
        for (uint64_t e = e0; e < e1; e += kWave)
            wave_members(spans[wv], irec, he_mem, e, min(e + kWave, (uint64_t)e1), v, [&](uint32_t u) {
                const uint64_t has = __ballot(u != kNoKey);
                const uint32_t at = count + lane_rank(has);
                if (u != kNoKey && at < kWave) occ[at] = u;
                count += (uint32_t)__popcll(has);
            });
        wave_sync();
        count = min(count, (uint32_t)kWave);
        const uint32_t u = lane < count ? occ[lane] : kNoKey;
        uint32_t w = 0, before = 0;
        for (uint32_t j = 0; j < count; ++j) {
            const bool eq = u == wave_bcast(u, (int)j);
            w += eq ? 1u : 0u;
            before += eq && j < lane ? 1u : 0u;
        }
        const bool first = lane < count && before == 0u;   // one lane per co-member
        const uint64_t firsts = __ballot(first);
        const uint32_t wmax = wave_max(first ? w : 0u);
        uint32_t layers = 0;
        for (uint64_t left = firsts; left; ++layers)
            left &= ~__ballot(first && w == wave_bcast(w, __ffsll((unsigned long long)left) - 1));
        const uint32_t tops = (uint32_t)__popcll(__ballot(first && w == wmax));
        if (lane == (uint32_t)k) {
            rdeg = (uint32_t)__popcll(firsts);
            rl = layers;
            rtop = tops;
        }
        wave_sync();
    }
    if (mine < n && cv <= kWave) {
        deg[mine] = rdeg;
        l[mine] = rl;
        top[mine] = rtop;
    }
}

// 64 < c(v) <= kWavePairs: one wave per listed vertex.
__global__ __launch_bounds__(kBlock) void k_layers_wave(const PrepInfo *__restrict__ info,
                                                         const uint32_t *__restrict__ list,
                                                         const uint32_t *__restrict__ v_off,
                                                         const uint4 *__restrict__ irec,
                                                         const uint32_t *__restrict__ he_mem,
                                                         uint32_t *__restrict__ deg, uint32_t *__restrict__ l,
                                                         uint32_t *__restrict__ top) {
    constexpr uint32_t kSlots = 2 * kWavePairs, kBits = kWavePairs / 32 + 1;
    __shared__ SpanLds spans[kWavesPerBlock];
    __shared__ uint32_t key_s[kWavesPerBlock][kSlots], cnt_s[kWavesPerBlock][kSlots], bits_s[kWavesPerBlock][kWave];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    uint32_t *key = key_s[wv], *cnt = cnt_s[wv], *bits = bits_s[wv];
    static_assert(kBits <= kWave, "one word of weight marks per lane");
    const uint32_t count = info->n_wave;
    for (uint32_t i = blockIdx.x * kWavesPerBlock + wv; i < count; i += gridDim.x * kWavesPerBlock) {
        const uint32_t v = uni(list[i]);
        const uint32_t e0 = uni(v_off[v]), e1 = uni(v_off[v + 1]);
        for (uint32_t s = lane; s < kSlots; s += kWave) {
            key[s] = kNoKey;
            cnt[s] = 0u;
        }
        bits[lane] = 0u;
        wave_sync();
        for (uint64_t e = e0; e < e1; e += kWave)
            wave_members(spans[wv], irec, he_mem, e, min(e + kWave, (uint64_t)e1), v, [&](uint32_t u) {
                if (u != kNoKey) (void)lds_count<kSlots>(key, cnt, u);   // at most kSlots / 2 keys
            });
        wave_sync();
        uint32_t d = 0, wm = 0, tops = 0;
        for (uint32_t s = lane; s < kSlots; s += kWave) {
            const uint32_t w = cnt[s];
            if (w == 0u) continue;
            ++d;
            tops = w > wm ? 1u : tops + (w == wm ? 1u : 0u);
            wm = max(w, wm);
            atomicOr(&bits[w >> 5], 1u << (w & 31u));
        }
        wave_sync();
        const uint32_t wmax = wave_max(wm);
        tops = wave_sum(wm == wmax ? tops : 0u);
        d = wave_sum(d);
        const uint32_t layers = wave_sum((uint32_t)__popc(bits[lane]));
        if (lane == 0) {
            deg[v] = d;
            l[v] = layers;
            top[v] = tops;
        }
        wave_sync();
    }
}

// One workgroup per listed vertex.  With P passes, pass p counts the ids whose
// mixed value lies in the p-th of P equal parts of the 32-bit range; weights
// of all passes meet in the weight marks.
// A vertex whose ids overflow the table in some pass joins the hubs.
template <int kThreads, uint32_t kSlots, uint32_t kMaxPairs>
__global__ __launch_bounds__(kThreads) void k_layers_block(const uint32_t *__restrict__ n_list,
                                                            const uint32_t *__restrict__ list, uint32_t n,
                                                            const unsigned long long *__restrict__ c,
                                                            const uint32_t *__restrict__ v_off,
                                                            const uint4 *__restrict__ irec,
                                                            const uint32_t *__restrict__ he_mem,
                                                            uint32_t *__restrict__ deg, uint32_t *__restrict__ l,
                                                            uint32_t *__restrict__ top, uint32_t *__restrict__ hubs,
                                                            PrepInfo *__restrict__ info) {
    constexpr uint32_t kWaves = kThreads / kWave, kLoad = kSlots / 4 * 3, kBits = kMaxPairs / 32 + 1;
    __shared__ SpanLds spans[kWaves];
    __shared__ uint32_t key[kSlots], cnt[kSlots], bits[kBits];
    __shared__ uint32_t part[3][kWaves];
    __shared__ uint32_t full;
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave), t = threadIdx.x;
    const uint32_t count = *n_list;
    for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
        const uint32_t v = uni(list[i]);
        const uint32_t e0 = uni(v_off[v]), e1 = uni(v_off[v + 1]);
        const uint32_t distinct = (uint32_t)min((unsigned long long)(n - 1u), c[v]);
        const uint32_t passes = (distinct + kLoad - 1u) / kLoad;
        for (uint32_t s = t; s < kBits; s += kThreads) bits[s] = 0u;
        if (t == 0) full = 0u;
        // incidences per wave and turn
        const uint32_t step = min((uint32_t)kWave, (e1 - e0 + kWaves - 1u) / kWaves);
        uint32_t d = 0, wm = 0, tops = 0;   // this thread's slots over all passes
        for (uint32_t p = 0; p < passes; ++p) {
            for (uint32_t s = t; s < kSlots; s += kThreads) {
                key[s] = kNoKey;
                cnt[s] = 0u;
            }
            __syncthreads();
            for (uint64_t e = (uint64_t)e0 + (uint64_t)wv * step; e < e1; e += (uint64_t)kWaves * step)
                wave_members(spans[wv], irec, he_mem, e, min(e + step, (uint64_t)e1), v, [&](uint32_t u) {
                    if (u != kNoKey && (passes == 1u || __umulhi(mix32(u ^ 0x9E3779B9u), passes) == p) &&
                        !lds_count<kSlots>(key, cnt, u))
                        full = 1u;
                });
            __syncthreads();
            for (uint32_t s = t; s < kSlots; s += kThreads) {
                const uint32_t w = cnt[s];
                if (w == 0u) continue;
                ++d;
                tops = w > wm ? 1u : tops + (w == wm ? 1u : 0u);
                wm = max(w, wm);
                const uint32_t bit = 1u << (w & 31u);
                if ((bits[w >> 5] & bit) == 0u) atomicOr(&bits[w >> 5], bit);
            }
            __syncthreads();
        }
        uint32_t layers = 0;
        for (uint32_t s = t; s < kBits; s += kThreads) layers += (uint32_t)__popc(bits[s]);
        const uint32_t wmw = wave_max(wm);
        d = wave_sum(d);
        layers = wave_sum(layers);
        if (lane == 0) {
            part[0][wv] = d;
            part[1][wv] = layers;
            part[2][wv] = wmw;
        }
        __syncthreads();
        uint32_t wmax = 0;
        for (uint32_t q = 0; q < kWaves; ++q) wmax = max(wmax, part[2][q]);
        __syncthreads();
        tops = wave_sum(wm == wmax ? tops : 0u);
        if (lane == 0) part[2][wv] = tops;
        __syncthreads();
        if (t == 0) {
            uint32_t sd = 0, sl = 0, st = 0;
            for (uint32_t q = 0; q < kWaves; ++q) {
                sd += part[0][q];
                sl += part[1][q];
                st += part[2][q];
            }
            if (full) {
                hubs[atomicAdd(&info->n_hub, 1u)] = v;
                atomicMax(&info->dmax, e1 - e0);
            } else {
                deg[v] = sd;
                l[v] = sl;
                top[v] = st;
            }
        }
        __syncthreads();
    }
}

// ---- hubs --------------------------------------------------------------------
// A batch of hubs, each with a row of `n` counters and `words` words of weight
// marks.  chunk_off: exclusive prefix of the hubs' chunks of kHubChunk
// incidences (one workgroup).
constexpr uint32_t kHubChunk = 256;
constexpr uint32_t kHubTable = 4096;      // per workgroup: occurrences met before their counters
constexpr uint32_t kHubScan = 4096;       // counters per workgroup and turn

__global__ __launch_bounds__(kBlock) void k_hub_chunks(const uint32_t *__restrict__ hubs, uint32_t count,
                                                        const uint32_t *__restrict__ v_off,
                                                        unsigned long long *__restrict__ chunk_off) {
    __shared__ unsigned long long part[kWavesPerBlock];
    __shared__ unsigned long long carry;
    if (threadIdx.x == 0) carry = 0ull;
    __syncthreads();
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    for (uint32_t base = 0; base < count; base += kBlock) {
        const uint32_t i = base + threadIdx.x;
        unsigned long long x = 0;
        if (i < count) {
            const uint32_t v = hubs[i];
            x = (v_off[v + 1] - v_off[v] + (uint64_t)kHubChunk - 1u) / kHubChunk;
        }
        const unsigned long long incl = wave_incl_scan(x);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        unsigned long long before = carry;
        for (uint32_t q = 0; q < wv; ++q) before += part[q];
        if (i < count) chunk_off[i] = before + incl - x;
        __syncthreads();
        if (threadIdx.x == kBlock - 1) carry = before + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) chunk_off[count] = carry;
}

// Occurrences of the hubs into their counters, a chunk per workgroup and turn.
// The chunk's occurrences meet in an LDS table first: co-members of a hub are
// mostly hubs again, and device atomics on one counter queue up.
__global__ __launch_bounds__(kBlock) void k_hub_count(const uint32_t *__restrict__ hubs, uint32_t count,
                                                       const unsigned long long *__restrict__ chunk_off,
                                                       const uint32_t *__restrict__ v_off,
                                                       const uint4 *__restrict__ irec,
                                                       const uint32_t *__restrict__ he_mem, uint64_t n,
                                                       uint32_t *__restrict__ rows) {
    __shared__ SpanLds spans[kWavesPerBlock];
    __shared__ BlockTable<kHubTable> tab;
    __shared__ uint32_t tcnt[kHubTable];
    const uint32_t wv = uni(threadIdx.x / kWave);
    tab.clear_keys();
    for (uint32_t s = threadIdx.x; s < kHubTable; s += kBlock) tcnt[s] = 0u;
    __syncthreads();
    const unsigned long long chunks = chunk_off[count];
    for (unsigned long long ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
        uint32_t lo = 0, hi = count;   // chunk_off[lo] <= ch < chunk_off[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (chunk_off[mid] <= ch) lo = mid; else hi = mid;
        }
        const uint32_t v = uni(hubs[lo]);
        uint32_t *row = rows + (uint64_t)lo * n;
        const uint64_t e_end = v_off[v + 1];
        const uint64_t b0 = v_off[v] + (ch - chunk_off[lo]) * kHubChunk;
        const uint64_t b1 = min(b0 + kHubChunk, e_end);
        for (uint64_t e = b0 + (uint64_t)wv * kWave; e < b1; e += kBlock)
            wave_members(spans[wv], irec, he_mem, e, min(e + kWave, b1), v, [&](uint32_t u) {
                if (u == kNoKey) return;
                const uint32_t sl = tab.slot(u);
                if (sl != kTableEmpty) atomicAdd(&tcnt[sl], 1u);
                else atomicAdd(&row[u], 1u);
            });
        __syncthreads();
        for (uint32_t s = threadIdx.x; s < kHubTable; s += kBlock) {
            const uint32_t u = tab.key[s];
            if (u != kTableEmpty) {
                atomicAdd(&row[u], tcnt[s]);
                tab.key[s] = kTableEmpty;
                tcnt[s] = 0u;
            }
        }
        __syncthreads();
    }
}

// Per (hub, kHubScan counters): co-members, largest weight and how many have
// it (part: 3 words each), and the weights' marks.
__global__ __launch_bounds__(kBlock) void k_hub_scan(uint32_t n, uint32_t tiles, const uint32_t *__restrict__ rows,
                                                      uint32_t words, uint32_t *__restrict__ marks,
                                                      uint32_t *__restrict__ part) {
    constexpr uint32_t kLow = 2048;   // smaller weights are marked once per workgroup
    __shared__ uint32_t low[kLow / 32];
    __shared__ uint32_t wpart[2][kWavesPerBlock];
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint32_t hub = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const uint32_t *row = rows + (uint64_t)hub * n;
    uint32_t *mk = marks + (uint64_t)hub * words;
    for (uint32_t s = threadIdx.x; s < kLow / 32; s += kBlock) low[s] = 0u;
    __syncthreads();
    uint32_t d = 0, wm = 0, tops = 0;
    for (uint32_t i = threadIdx.x; i < kHubScan; i += kBlock) {
        const uint64_t u = (uint64_t)tile * kHubScan + i;
        const uint32_t w = u < n ? row[u] : 0u;
        if (w == 0u) continue;
        ++d;
        tops = w > wm ? 1u : tops + (w == wm ? 1u : 0u);
        wm = max(w, wm);
        const uint32_t bit = 1u << (w & 31u);
        if (w < kLow) {
            if ((low[w >> 5] & bit) == 0u) atomicOr(&low[w >> 5], bit);
        } else {
            atomicOr(&mk[w >> 5], bit);
        }
    }
    const uint32_t wmw = wave_max(wm);
    d = wave_sum(d);
    if (lane == 0) {
        wpart[0][wv] = d;
        wpart[1][wv] = wmw;
    }
    __syncthreads();
    uint32_t wmax = 0, sd = 0;
    for (uint32_t q = 0; q < kWavesPerBlock; ++q) {
        sd += wpart[0][q];
        wmax = max(wmax, wpart[1][q]);
    }
    __syncthreads();
    tops = wave_sum(wm == wmax ? tops : 0u);
    if (lane == 0) wpart[0][wv] = tops;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t st = 0;
        for (uint32_t q = 0; q < kWavesPerBlock; ++q) st += wpart[0][q];
        uint32_t *o = part + 3 * ((uint64_t)hub * tiles + tile);
        o[0] = sd;
        o[1] = wmax;
        o[2] = wmax ? st : 0u;
    }
    for (uint32_t s = threadIdx.x; s < kLow / 32 && s < words; s += kBlock)
        if (low[s]) atomicOr(&mk[s], low[s]);
}

// One workgroup per hub: its tiles' results and marks together.
__global__ __launch_bounds__(kBlock) void k_hub_final(const uint32_t *__restrict__ hubs, uint32_t tiles,
                                                       const uint32_t *__restrict__ part, uint32_t words,
                                                       const uint32_t *__restrict__ marks, uint32_t *__restrict__ deg,
                                                       uint32_t *__restrict__ l, uint32_t *__restrict__ top) {
    __shared__ uint32_t acc[4];   // co-members, largest weight, its count, layers
    if (threadIdx.x < 4) acc[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t *pt = part + 3 * (uint64_t)blockIdx.x * tiles;
    const uint32_t *mk = marks + (uint64_t)blockIdx.x * words;
    uint32_t d = 0, wm = 0, layers = 0;
    for (uint32_t i = threadIdx.x; i < tiles; i += kBlock) {
        d += pt[3 * i];
        wm = max(wm, pt[3 * i + 1]);
    }
    for (uint32_t i = threadIdx.x; i < words; i += kBlock) layers += (uint32_t)__popc(mk[i]);
    atomicAdd(&acc[0], d);
    atomicMax(&acc[1], wm);
    atomicAdd(&acc[3], layers);
    __syncthreads();
    uint32_t tops = 0;
    for (uint32_t i = threadIdx.x; i < tiles; i += kBlock)
        if (pt[3 * i + 1] == acc[1]) tops += pt[3 * i + 2];
    atomicAdd(&acc[2], tops);
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t v = hubs[blockIdx.x];
        deg[v] = acc[0];
        l[v] = acc[3];
        top[v] = acc[2];
    }
}

// Stratum of each vertex, per-tile stratum counts (stratum-major layout), the
// integer sums and the largest l_v.
__global__ __launch_bounds__(kBlock) void k_strata(uint32_t n, const uint32_t *__restrict__ l,
                                                    const uint32_t *__restrict__ deg, const uint32_t *__restrict__ top,
                                                    uint8_t *__restrict__ stratum, uint32_t *__restrict__ counts,
                                                    uint32_t tiles, PrepInfo *__restrict__ info) {
    __shared__ uint32_t cnt[kNStrata], lm;
    __shared__ unsigned long long ps[3];
    if (threadIdx.x < kNStrata) cnt[threadIdx.x] = 0;
    if (threadIdx.x < 3) ps[threadIdx.x] = 0ull;
    if (threadIdx.x == 3) lm = 0u;
    __syncthreads();
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    uint64_t a = 0, b = 0, c = 0;
    uint32_t lv = 0;
    if (v < n) {
        lv = l[v];
        uint32_t s = lv ? 32u - __clz(lv) : 0u;   // 1 + floor(log2 l_v)
        s = s < kNStrata - 1 ? s : kNStrata - 1;
        stratum[v] = (uint8_t)s;
        atomicAdd(&cnt[s], 1u);
        a = top[v];
        b = deg[v];
        c = lv;
    }
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    lv = wave_max(lv);
    if (lane_id() == 0) {
        atomicAdd(&ps[0], (unsigned long long)a);
        atomicAdd(&ps[1], (unsigned long long)b);
        atomicAdd(&ps[2], (unsigned long long)c);
        atomicMax(&lm, lv);
    }
    __syncthreads();
    if (threadIdx.x < kNStrata) counts[(uint64_t)threadIdx.x * tiles + blockIdx.x] = cnt[threadIdx.x];
    if (threadIdx.x < 3 && ps[threadIdx.x]) atomicAdd(&info->sum_top + threadIdx.x, ps[threadIdx.x]);
    if (threadIdx.x == 3 && lm) atomicMax(&info->lmax, lm);
}

__global__ void k_strata_bounds(const uint64_t *__restrict__ base, uint32_t tiles, PrepInfo *__restrict__ info) {
    if (threadIdx.x < kNStrata) info->B[threadIdx.x] = base[(uint64_t)threadIdx.x * tiles];
}

// Histogram of the layer counts (Theorem 2's theta(l*) is a sum over it):
// counts below kLhistBins in LDS per workgroup, flushed once.
constexpr uint32_t kLhistBins = 1024;

__global__ __launch_bounds__(kBlock) void k_lhist(uint32_t n, const uint32_t *__restrict__ l,
                                                   unsigned long long *__restrict__ hist) {
    __shared__ uint32_t bins[kLhistBins];
    for (uint32_t b = threadIdx.x; b < kLhistBins; b += kBlock) bins[b] = 0;
    __syncthreads();
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const uint32_t x = l[v];
        if (x < kLhistBins) atomicAdd(&bins[x], 1u);
        else atomicAdd(&hist[x], 1ull);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < kLhistBins; b += kBlock)
        if (bins[b]) atomicAdd(&hist[b], (unsigned long long)bins[b]);
}

// Stable placement of each vertex at its (stratum, id) rank.
__global__ __launch_bounds__(kBlock) void k_place(uint32_t n, const uint8_t *__restrict__ stratum,
                                                   const uint64_t *__restrict__ base, uint32_t tiles,
                                                   uint32_t *__restrict__ P) {
    __shared__ uint32_t wcount[kBlock / kWave][kNStrata];
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    const uint32_t lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const uint32_t s = v < n ? stratum[v] : kNStrata;   // out-of-range lanes match nothing
    uint32_t rank = 0;
    for (uint32_t h = 0; h < kNStrata; ++h) {
        uint64_t mask = __ballot(s == h);
        if (lane == 0) wcount[wv][h] = (uint32_t)__popcll(mask);
        if (s == h) rank = lane_rank(mask);
    }
    __syncthreads();
    if (v < n) {
        uint64_t pos = base[(uint64_t)s * tiles + blockIdx.x] + rank;
        for (uint32_t w = 0; w < wv; ++w) pos += wcount[w][s];
        P[pos] = v;
    }
}

}  // namespace

int stratify_device(hyperim_graph g, PrepWorkspace &w, hipStream_t s) {
    const uint32_t n = g->n;   // at least 1
    const size_t nn = n;
    HIM_CHECK(g->l.reserve(sizeof(uint32_t) * nn, s));
    HIM_CHECK(g->deg.reserve(sizeof(uint32_t) * nn, s));
    HIM_CHECK(g->top.reserve(sizeof(uint32_t) * nn, s));
    HIM_CHECK(g->stratum.reserve(nn, s));
    HIM_CHECK(g->P.reserve(sizeof(uint32_t) * nn, s));
    DevBuf &tmp_b = w.tmp;
    HIM_CHECK(w.info.reserve(sizeof(PrepInfo), s));
    HIM_CHECK(w.lists.reserve(sizeof(uint32_t) * 4 * nn, s));
    PrepInfo *di = w.info.as<PrepInfo>(), hi{};
    HIM_HIP(hipMemsetAsync(di, 0, sizeof(PrepInfo), s));
    uint32_t *lists = w.lists.as<uint32_t>();   // one list of n per class: wave, two workgroup sizes, hubs
    uint32_t *hubs = lists + 3 * (size_t)n;
    const uint32_t *v_off = g->v_off.as<uint32_t>(), *he_mem = g->he_mem.as<uint32_t>();
    const uint4 *irec = g->irec.as<uint4>();
    const unsigned long long *cc = g->c.as<unsigned long long>();
    uint32_t *deg = g->deg.as<uint32_t>(), *ll = g->l.as<uint32_t>(), *top = g->top.as<uint32_t>();
    const uint32_t tiles = (uint32_t)std::max<uint64_t>(div_up(n, kBlock), 1);
    // From here on a vertex is a hub.  A hub's row costs 8 n bytes and spreads
    // over the grid; below n / 16 occurrences that is more than the occurrences
    // are worth, and a workgroup's passes over them (at most 11) are short.
    // With 131072 for every n the last workgroup of a 1e5-vertex graph took
    // 0.96 ms.
    const uint32_t dense = std::min(std::max<uint32_t>(n / 16u, kBlockTable / 4u * 3u), kDensePairs);
    hipLaunchKernelGGL(k_classify, dim3((uint32_t)div_up(n, kBlock * kClassPer)), dim3(kBlock), 0, s, n, dense, cc,
                       v_off, lists, di);
    hipLaunchKernelGGL((k_layers_block<1024, kBlockTable, kDensePairs>), dim3(std::min<uint32_t>(tiles, 512)), dim3(1024), 0,
                       s, &di->n_big, lists + 2 * (size_t)n, n, cc, v_off, irec, he_mem, deg, ll, top, hubs, di);
    hipLaunchKernelGGL((k_layers_block<kBlock, 4096, kBlockPairs>), dim3(std::min<uint32_t>(tiles, 4096)), dim3(kBlock),
                       0, s, &di->n_block, lists + (size_t)n, n, cc, v_off, irec, he_mem, deg, ll, top, hubs, di);
    hipLaunchKernelGGL(k_layers_wave, dim3(std::min<uint32_t>(tiles, 2048)), dim3(kBlock), 0, s, di, lists, v_off,
                       irec, he_mem, deg, ll, top);
    HIM_HIP(hipGetLastError());
    // the class counts, before the registers' class runs: the wait is short
    HIM_HIP(hipMemcpyAsync(&hi, di, sizeof(PrepInfo), hipMemcpyDeviceToHost, s));
    hipLaunchKernelGGL(k_layers_reg, dim3(std::max<uint32_t>((uint32_t)div_up(n, kBlock), 1)), dim3(kBlock), 0, s, n,
                       cc, v_off, irec, he_mem, deg, ll, top);
    HIM_HIP(hipStreamSynchronize(s));
    if (hi.n_hub) {
        const uint32_t words = hi.dmax / 32u + 1u, row_tiles = (uint32_t)div_up(n, kHubScan);
        const uint64_t per_hub = 4ull * n + 4ull * words + 12ull * row_tiles;
        const uint32_t batch = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(hi.n_hub, kDenseBudget / per_hub));
        HIM_CHECK(w.k1.reserve(4ull * n * batch, s));
        HIM_CHECK(w.k2.reserve(4ull * words * batch, s));
        HIM_CHECK(w.vals.reserve(12ull * row_tiles * batch, s));
        HIM_CHECK(w.pc.reserve(8ull * ((size_t)batch + 1), s));
        for (uint32_t h0 = 0; h0 < hi.n_hub; h0 += batch) {
            const uint32_t cnt = std::min(batch, hi.n_hub - h0);
            HIM_HIP(hipMemsetAsync(w.k1.ptr, 0, 4ull * n * cnt, s));
            HIM_HIP(hipMemsetAsync(w.k2.ptr, 0, 4ull * words * cnt, s));
            hipLaunchKernelGGL(k_hub_chunks, dim3(1), dim3(kBlock), 0, s, hubs + h0, cnt, v_off,
                               w.pc.as<unsigned long long>());
            hipLaunchKernelGGL(k_hub_count, dim3(2048), dim3(kBlock), 0, s, hubs + h0, cnt,
                               w.pc.as<unsigned long long>(), v_off, irec, he_mem, (uint64_t)n, w.k1.as<uint32_t>());
            hipLaunchKernelGGL(k_hub_scan, dim3(cnt * row_tiles), dim3(kBlock), 0, s, n, row_tiles,
                               w.k1.as<uint32_t>(), words, w.k2.as<uint32_t>(), w.vals.as<uint32_t>());
            hipLaunchKernelGGL(k_hub_final, dim3(cnt), dim3(kBlock), 0, s, hubs + h0, row_tiles,
                               w.vals.as<uint32_t>(), words, w.k2.as<uint32_t>(), deg, ll, top);
        }
        HIM_HIP(hipGetLastError());
    }

    // strata, counts, statistics.  l distinct positive weights sum to at most
    // c(v), so l(l + 1) / 2 <= c(v) bounds the histogram of the layer counts.
    const uint64_t lbound = std::min<uint64_t>(g->m, (uint64_t)std::sqrt(2.0 * (double)hi.cmax) + 1);
    DevBuf &counts_b = w.counts, &base_b = w.base, &hist_b = w.hist;
    HIM_CHECK(counts_b.reserve(sizeof(uint32_t) * kNStrata * tiles, s));
    HIM_CHECK(base_b.reserve(sizeof(uint64_t) * (kNStrata * (size_t)tiles + 1), s));
    HIM_CHECK(hist_b.reserve(sizeof(unsigned long long) * (lbound + 1), s));
    HIM_HIP(hipMemsetAsync(hist_b.ptr, 0, sizeof(unsigned long long) * (lbound + 1), s));
    hipLaunchKernelGGL(k_strata, dim3(tiles), dim3(kBlock), 0, s, n, ll, deg, top, g->stratum.as<uint8_t>(),
                       counts_b.as<uint32_t>(), tiles, di);
    hipLaunchKernelGGL(k_lhist, dim3(std::min<uint32_t>(tiles, 64)), dim3(kBlock), 0, s, n, ll,
                       hist_b.as<unsigned long long>());
    HIM_CHECK(scan_u32_to_u64(counts_b.as<uint32_t>(), base_b.as<uint64_t>(), (uint64_t)kNStrata * tiles, 0, tmp_b,
                              s));
    hipLaunchKernelGGL(k_place, dim3(tiles), dim3(kBlock), 0, s, n, g->stratum.as<uint8_t>(), base_b.as<uint64_t>(),
                       tiles, g->P.as<uint32_t>());
    hipLaunchKernelGGL(k_strata_bounds, dim3(1), dim3(kWave), 0, s, base_b.as<uint64_t>(), tiles, di);
    HIM_HIP(hipGetLastError());
    std::vector<uint64_t> hist(lbound + 1);
    HIM_HIP(hipMemcpyAsync(&hi, di, sizeof(PrepInfo), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipMemcpyAsync(hist.data(), hist_b.ptr, sizeof(uint64_t) * hist.size(), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    const uint32_t lmax = hi.lmax;
    hyperim_strata_info &info = g->info;
    for (uint32_t h = 0; h < kNStrata; ++h) info.B[h] = (uint32_t)hi.B[h];
    info.B[kNStrata] = n;
    info.sum_top = hi.sum_top;
    info.sum_deg = hi.sum_deg;
    info.sum_l = hi.sum_l;
    double tl = 0.0;   // sum over v with l_v > 0 of l_v / ln(l_v + 1), grouped by value
    for (uint32_t lv = 1; lv <= lmax; ++lv)
        if (hist[lv]) tl += (double)hist[lv] * ((double)lv / std::log((double)lv + 1.0));
    info.alpha = info.sum_deg ? (double)info.sum_top / (double)info.sum_deg : 0.0;
    info.beta = n ? (double)info.sum_l / (double)n : 0.0;
    info.theta_l = n ? tl / (double)n : 0.0;
    g->strat_lmax = lmax;
    if (g->layered()) HIM_CHECK(layers_build_device(g, w, lmax, s));
    g->stratified = true;
    // a divided graph keeps its division (the same strata give the same one)
    g->routed = false;
    if (g->route_on) {
        uint32_t n1 = 0;
        const int rc = route_build(g, w, s, &n1);
        if (rc != HYPERIM_OK) {
            g->route_on = false;   // left undivided, as after a failed hyperim_route
            return rc;
        }
    }
    return HYPERIM_OK;
}

}  // namespace hyperim
