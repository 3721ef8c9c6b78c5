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
//   above, or above n / 48 (hubs)  brought together by ranges of ids, a range's
//                       counters in one workgroup's LDS.
// Reading and counting (LDS atomics) bound every class.  A million vertices
// with 1.9e8 occurrences (Zipf 1.1 members): 46 ms when all pairs went through
// two hash tables in device memory, 9 ms with rows of counters in device memory
// for the hubs, 4.5 ms now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

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
constexpr uint64_t kHubBudget = 2ull << 30;     // bytes of occurrences, counts and marks per batch of hubs
constexpr uint32_t kHubChunk = 512;             // a hub's incidences per workgroup and turn
constexpr int kWavesPerBlock = kBlock / kWave;

// The 32-bit finaliser of MurmurHash3 (Appleby, public domain).
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
    unsigned long long hub_occ, hub_chunks;   // the hubs' occurrences and chunks of incidences
    unsigned long long sum_top, sum_deg, sum_l;
    unsigned long long B[kNStrata];
};

// Incidence spans of one wave, flattened: body(u) for every member of the
// incidences [e0, e1) of irec (at most 64), v itself left out; `u` is valid
// where the lane has one (else kNoKey), and every lane calls body together.
struct SpanLds {
    uint32_t mark[kWave], hb[kWave];
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
    L.hb[lane] = rec.y - (incl - rec.z);   // member q of the span is he_mem[hb + q]; may wrap
    for (uint32_t b = 0; b < total; b += kWave) {
        const uint32_t q = b + lane;
        const uint32_t k = window_owner(L.mark, incl - rec.z, rec.z, b);
        uint32_t u = kNoKey;
        if (q < total) {
            u = he_mem[L.hb[k] + q];   // the sum is taken in 32 bits
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

// One thread's share of a table of weights: how many are not zero, the largest,
// how many have it (meaningless while the largest is 0), and which of 1 .. 31
// occur (bit 0: set by zeros).  Free of branches for these, which almost all
// are: with one per weight, scanning 16384 counters of a hub cost 11000 cycles.
struct Tally {
    uint32_t d = 0, wm = 0, tops = 0, low = 0;
    __device__ __forceinline__ void count(uint32_t w) {
        d += w != 0u ? 1u : 0u;
        tops = w > wm ? 1u : tops + (w == wm ? 1u : 0u);
        wm = max(w, wm);
    }
    template <class Mark>   // mark(w): a weight of 32 or more
    __device__ __forceinline__ void add(const uint4 &c, Mark &&mark) {
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) count(w[q]);
        if ((c.x | c.y | c.z | c.w) < 32u) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) low |= 1u << w[q];
        } else {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                if (w[q] < 32u) low |= 1u << w[q];
                else mark(w[q]);
            }
        }
    }
    template <class Mark>
    __device__ __forceinline__ void one(uint32_t w, Mark &&mark) {
        count(w);
        if (w < 32u) low |= 1u << w;
        else mark(w);
    }
    // The marks of the wave's weights 1 .. 31.
    __device__ __forceinline__ uint32_t wave_low() const {
        return wave_last(wave_scan_op(low, [](uint32_t a, uint32_t b) { return a | b; })) & ~1u;
    }
};

// Vertices of each class above 64 occurrences, and the largest c(v) and hub.
// kClassPer vertices per thread: one device atomic per workgroup and class
// (one per wave took 0.59 ms on a million vertices).
constexpr uint32_t kClassPer = 16;

__global__ __launch_bounds__(kBlock) void k_classify(uint32_t n, uint32_t dense, const unsigned long long *__restrict__ c,
                                                      const uint32_t *__restrict__ v_off, uint32_t *__restrict__ lists,
                                                      PrepInfo *__restrict__ info) {
    __shared__ uint32_t cnt[4], base[4], dm_s;
    __shared__ unsigned long long cm_s, occ_s, ch_s;
    if (threadIdx.x < 4) cnt[threadIdx.x] = 0u;
    if (threadIdx.x == 4) {
        dm_s = 0u;
        cm_s = occ_s = ch_s = 0ull;
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
        if (cls[r] == 3) {
            const uint32_t d = v_off[v + 1] - v_off[v];
            dm = max(dm, d);
            atomicAdd(&occ_s, cv);
            atomicAdd(&ch_s, (unsigned long long)div_up(d, kHubChunk));
        }
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
        if (dm_s) {
            atomicMax(&info->dmax, dm_s);
            atomicAdd(&info->hub_occ, occ_s);
            atomicAdd(&info->hub_chunks, ch_s);
        }
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
    __shared__ alignas(16) uint32_t key[kSlots], cnt[kSlots];
    __shared__ uint32_t bits[kBits], part[4][kWaves];
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
        Tally y;   // this thread's slots over all passes
        for (uint32_t p = 0; p < passes; ++p) {
            for (uint32_t s = t; s < kSlots / 4; s += kThreads) {
                ((uint4 *)key)[s] = make_uint4(kNoKey, kNoKey, kNoKey, kNoKey);
                ((uint4 *)cnt)[s] = make_uint4(0u, 0u, 0u, 0u);
            }
            __syncthreads();
            for (uint64_t e = (uint64_t)e0 + (uint64_t)wv * step; e < e1; e += (uint64_t)kWaves * step)
                wave_members(spans[wv], irec, he_mem, e, min(e + step, (uint64_t)e1), v, [&](uint32_t u) {
                    if (u != kNoKey && (passes == 1u || __umulhi(mix32(u ^ 0x9E3779B9u), passes) == p) &&
                        !lds_count<kSlots>(key, cnt, u))
                        full = 1u;
                });
            __syncthreads();
            for (uint32_t s = t; s < kSlots / 4; s += kThreads)
                y.add(((const uint4 *)cnt)[s], [&](uint32_t w) {
                    const uint32_t bit = 1u << (w & 31u);
                    if ((bits[w >> 5] & bit) == 0u) atomicOr(&bits[w >> 5], bit);
                });
            __syncthreads();
        }
        const uint32_t lows = y.wave_low();
        if (lane == 0 && lows) atomicOr(&bits[0], lows);
        const uint32_t wmw = wave_max(y.wm), d = wave_sum(y.d);
        const uint32_t tops = wave_sum(y.wm == wmw ? y.tops : 0u);
        if (lane == 0) {
            part[0][wv] = d;
            part[1][wv] = wmw;
            part[2][wv] = tops;
        }
        __syncthreads();
        uint32_t layers = 0;
        for (uint32_t s = t; s < kBits; s += kThreads) layers += (uint32_t)__popc(bits[s]);
        layers = wave_sum(layers);
        if (lane == 0) part[3][wv] = layers;
        __syncthreads();
        if (t == 0) {
            uint32_t sd = 0, sl = 0, st = 0, wmax = 0;
            for (uint32_t q = 0; q < kWaves; ++q) {
                sd += part[0][q];
                wmax = max(wmax, part[1][q]);
                sl += part[3][q];
            }
            for (uint32_t q = 0; q < kWaves; ++q)
                if (part[1][q] == wmax) st += part[2][q];
            if (full) {
                hubs[atomicAdd(&info->n_hub, 1u)] = v;
                atomicMax(&info->dmax, e1 - e0);
                atomicAdd(&info->hub_occ, c[v]);
                atomicAdd(&info->hub_chunks, (unsigned long long)div_up(e1 - e0, kHubChunk));
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
// Occurrences are brought together by (hub, range of kHubBin ids) before they
// are counted: a pass over the hubs' incidences counts them per range, a second
// one writes their places within the range (16 bits each) there, and a
// workgroup per (hub, range) counts them in LDS.  Chunks of kHubChunk
// incidences spread the passes over the grid; the table of counts is laid out
// (hub, range, chunk), so that its prefix sums are the places and no counter is
// shared.  The passes are bound by finding and reading the members, the count
// by LDS accesses.  The 283 largest hubs of a million vertices (Zipf 1.1), with
// 9.3e7 occurrences: 4.8 ms when each had a row of n counters in device memory
// (4.7e7 device atomics even after a table in LDS), 1.7 ms now.
constexpr uint32_t kHubBinLog = 14, kHubBin = 1u << kHubBinLog;   // ids per range: 64 KB of counters
constexpr uint32_t kHubBins = 1024;                               // ranges per pass
constexpr int kHubBlock = 1024;                                   // threads that count a range

// chunk_off: exclusive prefix of the hubs' chunks (one workgroup).
__global__ __launch_bounds__(kBlock) void k_hub_chunks(const uint32_t *__restrict__ hubs, uint32_t count,
                                                        const uint32_t *__restrict__ v_off,
                                                        uint32_t *__restrict__ chunk_off) {
    __shared__ uint32_t part[kWavesPerBlock];
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0u;
    __syncthreads();
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    for (uint32_t base = 0; base < count; base += kBlock) {
        const uint32_t i = base + threadIdx.x;
        uint32_t x = 0;
        if (i < count) {
            const uint32_t v = hubs[i];
            x = (uint32_t)div_up(v_off[v + 1] - v_off[v], kHubChunk);
        }
        const uint32_t incl = wave_incl_scan(x);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (uint32_t q = 0; q < wv; ++q) before += part[q];
        if (i < count) chunk_off[i] = before + incl - x;
        __syncthreads();
        if (threadIdx.x == kBlock - 1) carry = before + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) chunk_off[count] = carry;
}

// Largest i in [0, count) with off[i] <= x (off[0] = 0, off[count] > x), 64
// entries at a time; every lane of the wave calls it with the same x.
__device__ __forceinline__ uint32_t wave_find(const uint32_t *__restrict__ off, uint32_t count, uint32_t x) {
    uint32_t lo = 0, len = count;   // in [lo, lo + len)
    while (len > 1) {
        const uint32_t step = (len + kWave - 1u) / kWave, i = lane_id() * step;
        const uint32_t k = (uint32_t)__popcll(__ballot(i < len && off[lo + i] <= x)) - 1u;
        lo += k * step;
        len = min(step, len - k * step);
    }
    return lo;
}

// The members of the hubs' chunks with ids in the ranges [bin0, bin0 + nb):
// counted per (hub, range, chunk), or (kPlace) written to the places whose
// firsts `off` holds.
template <bool kPlace>
__global__ __launch_bounds__(kBlock) void k_hub_pass(const uint32_t *__restrict__ hubs, uint32_t count,
                                                      const uint32_t *__restrict__ chunk_off,
                                                      const uint32_t *__restrict__ v_off,
                                                      const uint4 *__restrict__ irec,
                                                      const uint32_t *__restrict__ he_mem, uint32_t bin0, uint32_t nb,
                                                      const uint64_t *__restrict__ off, uint32_t *__restrict__ cnt,
                                                      uint16_t *__restrict__ entries) {
    __shared__ SpanLds spans[kWavesPerBlock];
    __shared__ uint32_t bin[kHubBins];   // counts, or next places (below 2^32: he_mem's positions are)
    const uint32_t wv = uni(threadIdx.x / kWave);
    const uint32_t chunks = uni(chunk_off[count]);
    for (uint32_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
        const uint32_t h = uni(wave_find(chunk_off, count, ch)), v = uni(hubs[h]);
        const uint32_t c0 = uni(chunk_off[h]), nch = uni(chunk_off[h + 1]) - c0;
        const uint64_t first = (uint64_t)c0 * nb + (ch - c0);   // of this chunk's counts, nch apart
        for (uint32_t b = threadIdx.x; b < nb; b += kBlock)
            bin[b] = kPlace ? (uint32_t)off[first + (uint64_t)b * nch] : 0u;
        __syncthreads();
        const uint64_t b0 = (uint64_t)v_off[v] + (uint64_t)(ch - c0) * kHubChunk;
        const uint64_t b1 = min(b0 + kHubChunk, (uint64_t)v_off[v + 1]);
        for (uint64_t e = b0 + (uint64_t)wv * kWave; e < b1; e += kBlock)
            wave_members(spans[wv], irec, he_mem, e, min(e + kWave, b1), v, [&](uint32_t u) {
                const uint32_t b = (u >> kHubBinLog) - bin0;
                if (u == kNoKey || b >= nb) return;
                const uint32_t at = atomicAdd(&bin[b], 1u);
                if constexpr (kPlace) entries[at] = (uint16_t)(u & (kHubBin - 1u));
            });
        __syncthreads();
        if constexpr (!kPlace) {
            for (uint32_t b = threadIdx.x; b < nb; b += kBlock) cnt[first + (uint64_t)b * nch] = bin[b];
            __syncthreads();
        }
    }
}

// Per (hub, range): co-members, largest weight and how many have it (part: 3
// words each), and the weights' marks.
__global__ __launch_bounds__(kHubBlock) void k_hub_count(uint32_t count, const uint32_t *__restrict__ chunk_off,
                                                          const uint64_t *__restrict__ off,
                                                          const uint16_t *__restrict__ entries, uint32_t bin0,
                                                          uint32_t nb, uint32_t tiles, uint32_t words,
                                                          uint32_t *__restrict__ marks, uint32_t *__restrict__ part) {
    constexpr uint32_t kLow = 2048, kWaves = kHubBlock / kWave;   // smaller weights are marked once per workgroup
    __shared__ alignas(16) uint32_t cnt[kHubBin];   // zero between items
    __shared__ uint32_t low[kLow / 32];             // likewise
    __shared__ uint32_t wpart[3][kWaves];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave), t = threadIdx.x;
    for (uint32_t s = t; s < kHubBin / 4; s += kHubBlock) ((uint4 *)cnt)[s] = make_uint4(0u, 0u, 0u, 0u);
    if (t < kLow / 32) low[t] = 0u;
    __syncthreads();
    // (hub, range) of an item, the workgroups' items being gridDim.x apart
    const uint32_t dh = gridDim.x / nb, db = gridDim.x % nb;
    uint32_t hub1 = blockIdx.x / nb, b1 = blockIdx.x % nb;
    uint64_t beg, end, beg1 = 0, end1 = 0;   // of this item and the next, read one item ahead
    auto span = [&]() {
        beg1 = end1 = 0;
        if (hub1 >= count) return;
        const uint32_t c0 = chunk_off[hub1], nch = chunk_off[hub1 + 1] - c0;
        const uint64_t first = (uint64_t)c0 * nb + (uint64_t)b1 * nch;
        beg1 = uni64(off[first]);
        end1 = uni64(off[first + nch]);
    };
    uint32_t u[4], u1[4];   // entries of this item; the first ones of the next
    auto load = [&](uint32_t (&u)[4], uint64_t e, uint64_t to) {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) u[q] = e + q * kHubBlock < to ? entries[e + q * kHubBlock] : kNoKey;
    };
    span();
    load(u1, beg1 + t, end1);
    while (hub1 < count) {
        const uint32_t hub = hub1, b = b1;
        beg = beg1;
        end = end1;
        hub1 += dh;
        b1 += db;
        if (b1 >= nb) {
            b1 -= nb;
            ++hub1;
        }
        span();
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) u[q] = u1[q];
        uint32_t *o = part + 3 * ((uint64_t)hub * tiles + bin0 + b);
        uint32_t *mk = marks + (uint64_t)hub * words;
        for (uint64_t e = beg + t; e < end;) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (u[q] != kNoKey) atomicAdd(&cnt[u[q]], 1u);
            e += 4u * kHubBlock;
            if (e < end) load(u, e, end);
        }
        load(u1, beg1 + t, end1);
        if (beg == end) {
            if (t < 3) o[t] = 0u;
            continue;
        }
        __syncthreads();
        Tally y;
        auto mark = [&](uint32_t w) {
            const uint32_t bit = 1u << (w & 31u);
            if (w >= kLow) atomicOr(&mk[w >> 5], bit);
            else if ((low[w >> 5] & bit) == 0u) atomicOr(&low[w >> 5], bit);
        };
        if (end - beg <= 4u * kHubBlock) {
            // every entry is still in a register: whoever takes a counter first has its weight
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (u[q] != kNoKey) y.one(atomicExch(&cnt[u[q]], 0u), mark);
        } else {
            for (uint32_t s = t; s < kHubBin / 4; s += kHubBlock) {
                const uint4 c4 = ((const uint4 *)cnt)[s];
                if ((c4.x | c4.y | c4.z | c4.w) == 0u) continue;
                ((uint4 *)cnt)[s] = make_uint4(0u, 0u, 0u, 0u);
                y.add(c4, mark);
            }
        }
        uint32_t wmw = 0, lows = 0, d = 0, tops = 0;
        if (__ballot(y.d != 0u)) {
            wmw = wave_max(y.wm);
            lows = y.wave_low();
            d = wave_sum(y.d);
            tops = wave_sum(y.wm == wmw ? y.tops : 0u);
        }
        if (lane == 0) {
            wpart[0][wv] = d;
            wpart[1][wv] = wmw;
            wpart[2][wv] = tops;
            if (lows) atomicOr(&low[0], lows);
        }
        __syncthreads();
        if (wv == 0) {
            const uint32_t w = lane < kWaves ? wpart[1][lane] : 0u, wmax = wave_max(w);
            const uint32_t sd = wave_sum(lane < kWaves ? wpart[0][lane] : 0u);
            const uint32_t st = wave_sum(lane < kWaves && w == wmax ? wpart[2][lane] : 0u);
            if (lane < 3) o[lane] = lane == 0 ? sd : lane == 1 ? wmax : st;
        } else if (wv == 1) {
            static_assert(kLow / 32 == kWave, "one word of marks per lane");
            const uint32_t m = low[lane];
            low[lane] = 0u;
            if (lane < words && m) atomicOr(&mk[lane], m);
        }
    }
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
    // Above this a vertex is a hub.  A hub costs its occurrences twice through
    // memory and n / 16384 ranges, a workgroup's passes grow with the square of
    // the occurrences (at most 11 passes).  On a million vertices the large
    // workgroups and the hubs take 3.6 ms together with n / 16, 2.9 with n / 42,
    // 3.1 with 12000 and 3.5 with 8000; with 131072 for every n the last
    // workgroup of a 1e5-vertex graph took 0.96 ms.
    const uint32_t dense = std::min(std::max<uint32_t>(n / 48u, kBlockTable / 4u * 3u), kDensePairs);
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
        const uint32_t words = hi.dmax / 32u + 1u, bins = (uint32_t)div_up(n, kHubBin), nb = std::min(bins, kHubBins);
        // Batches of hubs: 2 bytes an occurrence, 12 a chunk and range of a
        // pass, and the marks and parts of a hub.  Most graphs' hubs are one
        // batch, and their sizes stay on the device.
        const uint64_t per_chunk = 12ull * nb, per_hub = 4ull * words + 12ull * bins;
        std::vector<std::pair<uint32_t, uint64_t>> batches{{hi.n_hub, hi.hub_chunks}};   // hubs, chunks
        uint64_t occ = hi.hub_occ;   // of the largest batch
        if (2 * hi.hub_occ + per_chunk * hi.hub_chunks + per_hub * hi.n_hub > kHubBudget) {
            std::vector<uint32_t> ids(hi.n_hub), ends(n + 1ull);
            std::vector<uint64_t> cv(n);
            HIM_HIP(hipMemcpyAsync(ids.data(), hubs, 4ull * hi.n_hub, hipMemcpyDeviceToHost, s));
            HIM_HIP(hipMemcpyAsync(ends.data(), v_off, 4ull * (n + 1ull), hipMemcpyDeviceToHost, s));
            HIM_HIP(hipMemcpyAsync(cv.data(), cc, 8ull * n, hipMemcpyDeviceToHost, s));
            HIM_HIP(hipStreamSynchronize(s));
            batches.clear();
            occ = 0;
            uint64_t used = 0, occ_b = 0;
            for (uint32_t v : ids) {
                const uint64_t chunks = div_up(ends[v + 1ull] - ends[v], kHubChunk);
                const uint64_t need = 2 * cv[v] + per_chunk * chunks + per_hub;
                if (batches.empty() || used + need > kHubBudget) {
                    batches.push_back({0, 0});
                    used = occ_b = 0;
                }
                batches.back().first += 1;
                batches.back().second += chunks;
                used += need;
                occ_b += cv[v];
                occ = std::max(occ, occ_b);
            }
        }
        uint64_t hubs_max = 0, chunks_max = 0;
        for (const auto &b : batches) {
            hubs_max = std::max<uint64_t>(hubs_max, b.first);
            chunks_max = std::max(chunks_max, b.second);
        }
        HIM_CHECK(w.k1.reserve(2ull * occ, s));
        HIM_CHECK(w.k2.reserve(4ull * words * hubs_max, s));
        HIM_CHECK(w.vals.reserve(12ull * bins * hubs_max, s));
        HIM_CHECK(w.pc.reserve(4ull * (hubs_max + 1), s));
        HIM_CHECK(w.hub_cnt.reserve(4ull * nb * chunks_max, s));
        HIM_CHECK(w.hub_off.reserve(8ull * (nb * chunks_max + 1), s));
        uint32_t *chunk_off = w.pc.as<uint32_t>(), *cnt = w.hub_cnt.as<uint32_t>();
        uint64_t *off = w.hub_off.as<uint64_t>();
        uint16_t *entries = w.k1.as<uint16_t>();
        const uint32_t *hub = hubs;
        for (const auto &[count, chunks] : batches) {
            HIM_HIP(hipMemsetAsync(w.k2.ptr, 0, 4ull * words * count, s));
            hipLaunchKernelGGL(k_hub_chunks, dim3(1), dim3(kBlock), 0, s, hub, count, v_off, chunk_off);
            const dim3 grid((uint32_t)std::min<uint64_t>(chunks, 2048));
            for (uint32_t bin0 = 0; bin0 < bins; bin0 += kHubBins) {
                const uint32_t now = std::min(bins - bin0, kHubBins);
                hipLaunchKernelGGL(k_hub_pass<false>, grid, dim3(kBlock), 0, s, hub, count, chunk_off, v_off, irec,
                                   he_mem, bin0, now, off, cnt, entries);
                HIM_CHECK(scan_u32_to_u64(cnt, off, chunks * now, 0, tmp_b, s));
                hipLaunchKernelGGL(k_hub_pass<true>, grid, dim3(kBlock), 0, s, hub, count, chunk_off, v_off, irec,
                                   he_mem, bin0, now, off, cnt, entries);
                hipLaunchKernelGGL(k_hub_count, dim3((uint32_t)std::min<uint64_t>((uint64_t)count * now, 2048)),
                                   dim3(kHubBlock), 0, s, count, chunk_off, off, entries, bin0, now, bins, words,
                                   w.k2.as<uint32_t>(), w.vals.as<uint32_t>());
            }
            hipLaunchKernelGGL(k_hub_final, dim3(count), dim3(kBlock), 0, s, hub, bins, w.vals.as<uint32_t>(), words,
                               w.k2.as<uint32_t>(), deg, ll, top);
            hub += count;
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
