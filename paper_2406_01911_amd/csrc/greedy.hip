// Greedy max coverage over an RR-set pool (Algorithm 1 with the marginal
// coverage of Equation (2)) and the coverage count Lambda_R(S) of a seed set
// (Equation (1)'s estimator numerator).
//
// Coverage counts cnt[v] start as the number of sets containing v.  Each round
// takes the argmax of the key (cnt+1, -v) over unchosen vertices -- largest
// marginal coverage, ties to the smallest id -- then covers the not yet covered
// sets of the seed: each of their members loses one count.  Every set is
// covered at most once, so all rounds together touch each pool entry at most
// once.
//
// A round is two kernels (three with big sets).  k_scan reads the counts: each
// workgroup leaves its best key in a slot of its own.  k_cover reduces the
// slots in every workgroup (no atomics on one address, which queue up at 15 to
// 40 ns each across the eight XCDs) and covers the seed's sets: small sets come
// from an inverted index (counting sort by vertex), a wave or 16 lanes per set;
// whether a big set (above kBigSet members, ascending) holds the seed is looked
// up by a 17-ary search in the set itself, so big sets need no index.  k_sub
// then takes the members of the newly covered big sets off the counts.
//
// Equation (8) wants the sum of the k largest counts before each round (and
// after the last).  k_scan also lists the counts of at least `lo`, a guess
// below the k-th largest (the values next to it once each, with how many
// vertices share them), and keeps a copy of all counts; one workgroup of
// k_cover selects the exact sum from the list while the others cover, or from
// the copy when the guess was too high, and sets the next guess.
//
// Bound by launches and latency on small pools, by reading entries on pools of
// big sets.  100 rounds over 2048 sets of 85,000 members on average: 8.2 ms with
// an inverted index of all sets and one histogram of 4096 bins per workgroup and
// round, 1.45 ms now; a round over a million vertices and small sets with
// Equation (8): 48 us, 14 us now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "dev_common.h"
#include "internal.h"

namespace hyperim {
namespace {

constexpr int kWG = 256;
constexpr int kWavesPerWG = kWG / kWave;
constexpr uint32_t kBigSet = 4096;
constexpr uint32_t kGroup = 16;                   // lanes that share a set
constexpr uint32_t kGroupsPerWG = kWG / kGroup;
constexpr uint32_t kScanMax = 512;                // workgroups of k_scan (slots)
constexpr uint32_t kCoverMax = 512;               // workgroups of k_cover
constexpr uint32_t kRange = 8192;                 // vertices per LDS count range of big sets
constexpr uint32_t kMaxRanges = 512;              // ... up to this many ranges

__global__ void k_hist(const uint32_t *__restrict__ mem, uint64_t entries, uint32_t *__restrict__ cnt) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < entries;
         e += (uint64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[mem[e]], 1u);
}

// The sets above kBigSet members, how many, and (members not null) their members.
__global__ void k_big_list(const uint64_t *__restrict__ off, uint64_t theta, uint64_t *__restrict__ list,
                           unsigned long long *__restrict__ count, unsigned long long *__restrict__ members) {
    for (uint64_t j0 = (uint64_t)blockIdx.x * blockDim.x; j0 < theta; j0 += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t j = j0 + threadIdx.x;
        const uint64_t size = j < theta ? off[j + 1] - off[j] : 0u;
        const bool big = size > kBigSet;
        const uint64_t who = __ballot(big);
        if (who == 0ull) continue;
        if (members) {
            const uint64_t sum = wave_sum(big ? size : (uint64_t)0);
            if (lane_id() == 0) atomicAdd(members, (unsigned long long)sum);
        }
        unsigned long long base = 0;
        if (lane_id() == 0) base = atomicAdd(count, (unsigned long long)__popcll(who));
        base = wave_bcast64(base, 0);
        if (big) list[base + lane_rank(who)] = j;
    }
}

// body(e0, count) for the members [beg, end) of a set that kLanes lanes share:
// kTurn positions per lane and turn (e0, e0 + kLanes, ..., the first `count`
// of them inside), so that a long set's reads are in flight together.
constexpr uint32_t kUnroll = 4;
template <uint32_t kLanes, uint32_t kTurn = kUnroll, class Body>
__device__ __forceinline__ void for_members(uint64_t beg, uint64_t end, Body &&body) {
    for (uint64_t e = beg + threadIdx.x % kLanes; e < end; e += kTurn * kLanes)
        body(e, (uint32_t)min((end - e + kLanes - 1u) / kLanes, (uint64_t)kTurn));
}

// take(set, member) for every member of the sets [0, theta) of at most kBigSet
// members, kLanes lanes per set.
template <uint32_t kLanes, class Take>
__device__ __forceinline__ void for_small_sets(const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                               uint64_t theta, Take &&take) {
    constexpr uint32_t kPerWG = kWG / kLanes;
    for (uint64_t j = (uint64_t)blockIdx.x * kPerWG + threadIdx.x / kLanes; j < theta;
         j += (uint64_t)gridDim.x * kPerWG) {
        const uint64_t beg = off[j], end = off[j + 1];
        if (end - beg > kBigSet) continue;
        for_members<kLanes>(beg, end, [&](uint64_t e, uint32_t count) {
            uint32_t u[kUnroll];
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) u[t] = t < count ? mem[e + t * kLanes] : 0u;
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t)
                if (t < count) take(j, u[t]);
        });
    }
}

template <uint32_t kLanes>
__global__ __launch_bounds__(kWG) void k_hist_small(const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                                     uint64_t theta, uint32_t *__restrict__ cnt) {
    for_small_sets<kLanes>(off, mem, theta, [&](uint64_t, uint32_t u) { atomicAdd(&cnt[u], 1u); });
}

template <uint32_t kLanes>
__global__ __launch_bounds__(kWG) void k_inv_small(const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                                    uint64_t theta, const uint64_t *__restrict__ inv_off,
                                                    uint32_t *__restrict__ cursor, uint32_t *__restrict__ inv) {
    for_small_sets<kLanes>(off, mem, theta, [&](uint64_t j, uint32_t u) {
        inv[inv_off[u] + atomicAdd(&cursor[u], 1u)] = (uint32_t)j;
    });
}

// dir[b * (ranges + 1) + r]: members of big set b below vertex r * kRange.
__global__ __launch_bounds__(kWG) void k_dir(const uint64_t *__restrict__ list, uint64_t nbig, uint32_t ranges,
                                              const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                              uint32_t *__restrict__ dir) {
    const uint64_t total = nbig * (ranges + 1u);
    for (uint64_t i = (uint64_t)blockIdx.x * kWG + threadIdx.x; i < total; i += (uint64_t)gridDim.x * kWG) {
        const uint64_t b = i / (ranges + 1u);
        const uint64_t v = (i - b * (ranges + 1u)) * kRange, j = list[b];
        const uint32_t *m = mem + off[j];
        uint32_t lo = 0, hi = (uint32_t)(off[j + 1] - off[j]);
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            if (m[mid] < v) lo = mid + 1u; else hi = mid;
        }
        dir[i] = lo;
    }
}

// Adds (sign 1) or takes off (sign -1) the members of big sets pick(i), i in
// [i0, i1), that lie in vertex range r: counted in LDS, a wave per set, then
// one device atomic per vertex met.  Members arrive in order, so the slices
// are read coalesced and no two workgroups of a range meet often.
template <int kSign, class Pick>
__device__ __forceinline__ void range_counts(uint32_t *lds, uint32_t r, uint64_t i0, uint64_t i1, uint32_t n,
                                             uint32_t ranges, const uint64_t *__restrict__ list,
                                             const uint32_t *__restrict__ dir, const uint64_t *__restrict__ off,
                                             const uint32_t *__restrict__ mem, uint32_t *__restrict__ cnt,
                                             Pick &&pick) {
    // sets of few neighbouring vertices leave most ranges empty
    bool any = false;
    for (uint64_t i = i0 + threadIdx.x; i < i1; i += kWG) {
        const uint32_t *d = dir + pick(i) * (ranges + 1u) + r;
        any |= d[0] != d[1];
    }
    if (!__syncthreads_or(any ? 1 : 0)) return;
    for (uint32_t x = threadIdx.x; x < kRange; x += kWG) lds[x] = 0u;
    __syncthreads();
    const uint32_t base = r * kRange;
    for (uint64_t i = i0 + threadIdx.x / kWave; i < i1; i += kWavesPerWG) {
        const uint64_t b = pick(i);
        const uint32_t *m = mem + off[list[b]];
        const uint32_t *d = dir + b * (ranges + 1u) + r;
        for_members<kWave, 8>(d[0], d[1], [&](uint64_t e, uint32_t count) {
            uint32_t u[8];
#pragma unroll
            for (uint32_t t = 0; t < 8; ++t) u[t] = t < count ? m[e + t * kWave] : base;
#pragma unroll
            for (uint32_t t = 0; t < 8; ++t)
                if (t < count) atomicAdd(&lds[u[t] - base], 1u);
        });
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < kRange && base + x < n; x += kWG)
        if (lds[x]) {
            if constexpr (kSign > 0) atomicAdd(&cnt[base + x], lds[x]);
            else atomicSub(&cnt[base + x], lds[x]);
        }
    __syncthreads();
}

// One workgroup per (range, `per` big sets).
__global__ __launch_bounds__(kWG) void k_hist_big(const uint64_t *__restrict__ list, uint64_t nbig, uint32_t per,
                                                   uint32_t n, uint32_t ranges, const uint32_t *__restrict__ dir,
                                                   const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                                   uint32_t *__restrict__ cnt) {
    __shared__ uint32_t lds[kRange];
    const uint32_t r = blockIdx.x % ranges;
    const uint64_t i0 = (uint64_t)(blockIdx.x / ranges) * per, i1 = min(i0 + per, nbig);
    range_counts<1>(lds, r, i0, i1, n, ranges, list, dir, off, mem, cnt, [](uint64_t i) { return i; });
}

// State that rounds hand on (device memory).
struct RoundState {
    uint32_t lo;          // list counts of at least this
    float gap;            // lo is this share below the expected k-th largest count
    unsigned long long covered;   // sets covered so far
};

// Arguments of the per-round kernels.
struct GreedyParams {
    const uint64_t *off;
    const uint32_t *mem;
    const uint64_t *inv_off;
    const uint32_t *inv;
    const uint32_t *nsmall;          // per vertex: its entries in the inverted index
    uint32_t *covered;               // per set: 0, or the round that covered it, plus one
    uint32_t *cnt;
    uint8_t *chosen;
    uint32_t *seeds;
    unsigned long long *gains;
    uint32_t n, k, quads;            // quads: 4-vertex loads per thread of k_scan
    uint64_t theta;
    unsigned long long *slot_key;    // per k_scan workgroup: best key
    // big sets
    const uint64_t *big;
    uint64_t nbig, big_mean;         // how many, and their members on average
    const uint32_t *dir;             // null: no ranges (n above kRange * kMaxRanges)
    uint32_t ranges;
    uint32_t *hit;                   // per k_cover workgroup and big set of its share: newly covered big sets
    uint32_t *hit_n;                 // per k_cover workgroup: how many
    // Equation (8)
    uint32_t *snap;                  // copy of the counts
    uint2 *above;                    // per k_scan workgroup, room for its share and kWG more: counts >= lo
    uint32_t *above_n;               // per k_scan workgroup: how many
    RoundState *state;
    unsigned long long *ub;          // k + 1 top-k sums, one per greedy prefix
};

// First guess of `lo`: the counts of an even sample of the vertices, at a rank
// that leaves a few times k of them above.
constexpr uint32_t kSample = 4096;
constexpr uint32_t kBins = 2048;
constexpr uint32_t kTopList = 4096;   // list entries held in LDS

// Suffix search over an LDS histogram of kBins bins: the bin in which the
// number of values in it and above reaches `need`, and the number above it.
// false: fewer than `need` in all.  The whole workgroup calls it.
__device__ __forceinline__ bool bin_search(const uint32_t *hc, uint32_t need, uint32_t *bin, uint32_t *above) {
    constexpr uint32_t kPer = kBins / kWG;
    __shared__ uint32_t wc[kWavesPerWG], hit[2], found;
    const uint32_t t = threadIdx.x, wv = t / kWave;
    // thread t owns bins from the top: kBins - 1 - t * kPer downwards
    const uint32_t top = kBins - 1u - t * kPer;
    uint32_t h[kPer], c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
        h[i] = hc[top - i];
        c += h[i];
    }
    const uint32_t ci = wave_incl_scan(c);
    if (lane_id() == kWave - 1) wc[wv] = ci;
    if (t == 0) found = 0u;
    __syncthreads();
    uint32_t cb = ci - c;
    for (uint32_t q = 0; q < wv; ++q) cb += wc[q];
    if (cb < need && cb + c >= need) {   // exactly one thread, if any
        uint32_t i = 0;
        for (; cb + h[i] < need; ++i) cb += h[i];
        hit[0] = top - i;
        hit[1] = cb;
        found = 1u;
    }
    __syncthreads();
    *bin = hit[0];
    *above = hit[1];
    const bool ok = found != 0u;
    __syncthreads();
    return ok;
}

template <typename T>
__device__ __forceinline__ T block_sum(T x) {
    __shared__ T part[kWavesPerWG];
    x = wave_sum(x);
    if (lane_id() == 0) part[threadIdx.x / kWave] = x;
    __syncthreads();
    T m = 0;
    for (uint32_t q = 0; q < kWavesPerWG; ++q) m += part[q];
    __syncthreads();
    return m;
}

// Shift that brings a range of values into kBins bins.
__device__ __forceinline__ uint32_t bin_shift(uint32_t range) {
    uint32_t s = 0;
    while ((range >> s) >= kBins) ++s;
    return s;
}

// The sum of the `k` largest of the values lo <= x <= max that visit(f) passes
// to f(x, c), c of each (every thread visits its own), and the k-th largest of
// them; false when there are fewer than k (then *sum is the sum of them all).
// Levels of kBins bins: the first spans all values, each further one the bin
// that holds the k-th; then one pass adds what is larger.  Small counts fall
// into a few bins: the lanes that share the first one's bin add once.  The whole
// workgroup calls it.
template <class Visit>
__device__ __forceinline__ bool top_sum(uint32_t *hc, uint32_t lo, uint32_t max, uint32_t k, Visit &&visit,
                                        unsigned long long *sum, uint32_t *kth) {
    uint32_t need = k, base = lo, width = max >= lo ? max - lo : 0u;   // values base .. base + width
    bool ok;
    for (;;) {
        const uint32_t sh = bin_shift(width);
        for (uint32_t i = threadIdx.x; i < kBins; i += kWG) hc[i] = 0u;
        __syncthreads();
        visit([&](uint32_t x, uint32_t c) {
            if (x < base || x - base > width) return;
            const uint32_t b = (x - base) >> sh, b0 = uni(b);
            const bool one = b == b0 && c == 1u;
            const uint64_t same = __ballot(one);
            if (!one) atomicAdd(&hc[b], c);
            else if (lane_rank(same) == 0u) atomicAdd(&hc[b0], (uint32_t)__popcll(same));
        });
        __syncthreads();
        uint32_t bin, above;
        ok = bin_search(hc, need, &bin, &above);
        if (!ok) break;
        need -= above;
        base += bin << sh;
        if (sh == 0u) break;
        width = (1u << sh) - 1u;
    }
    const uint32_t floor = ok ? base : 0u;   // not ok only at the first level: all values count
    unsigned long long acc = 0;
    visit([&](uint32_t x, uint32_t c) { acc += x > floor ? (unsigned long long)x * c : 0ull; });
    acc = block_sum(acc);
    *kth = base;
    *sum = ok ? acc + (unsigned long long)need * base : acc;
    return ok;
}

__global__ __launch_bounds__(kWG) void k_first_lo(const GreedyParams *__restrict__ P) {
    constexpr uint32_t kPer = kSample / kWG;
    __shared__ uint32_t hc[kBins];
    __shared__ uint32_t part[kWavesPerWG];
    const uint32_t n = P->n, m = min(n, kSample);
    uint32_t x[kPer], most = 0;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint32_t i = threadIdx.x + r * kWG;
        x[r] = i < m ? P->cnt[(uint64_t)i * n / m] : 0u;
        most = max(most, x[r]);
    }
    most = wave_max(most);
    if (lane_id() == 0) part[threadIdx.x / kWave] = most;
    __syncthreads();
    for (uint32_t q = 0; q < kWavesPerWG; ++q) most = max(most, part[q]);
    const uint64_t rank = (3ull * P->k * m + n - 1u) / n + 8u;
    uint32_t kth = 1;
    unsigned long long sum;
    const bool ok = top_sum(hc, 1u, uni(most), (uint32_t)min(rank, (uint64_t)m),
                            [&](auto &&f) {
#pragma unroll
                                for (uint32_t r = 0; r < kPer; ++r) f(x[r], 1u);
                            },
                            &sum, &kth);
    if (threadIdx.x == 0) {
        P->state->lo = ok ? kth : 1u;
        P->state->gap = 0.3f;
        P->state->covered = 0ull;
    }
}

// key = 0 for chosen vertices, else (cnt + 1) << 32 | (~v): the max is the
// largest count, then the smallest id.
__device__ __forceinline__ unsigned long long argmax_key(uint32_t c, uint8_t chosen, uint32_t v) {
    return chosen ? 0ull : (((unsigned long long)c + 1ull) << 32) | (unsigned long long)(0xFFFFFFFFu - v);
}

// Reads the counts, 4 consecutive vertices per thread and load (cnt, chosen and
// snap are 256-byte aligned; the last quad may be partial): the workgroup's
// best key into its slot, and with kTopk the copy of the counts and the list
// of those of at least lo, as (count, how many): lo .. lo + kWG - 1 once each,
// larger ones as they come, and on small graphs all of them.  (Small counts are shared by many vertices: a
// million of them in hyperedges of ten, 100,000 sets, had 20,000 and more
// counts listed one by one, 1.9 ms a round.)
template <bool kTopk>
__global__ __launch_bounds__(kWG) void k_scan(const GreedyParams *__restrict__ P) {
    __shared__ unsigned long long part[kWavesPerWG];
    __shared__ uint32_t listed, many[kWG];
    if (threadIdx.x == 0) listed = 0u;
    many[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t n = P->n, n4 = n / 4, quads = P->quads, lo = kTopk ? P->state->lo : 0u;
    const uint4 *__restrict__ cnt4 = reinterpret_cast<const uint4 *>(P->cnt);
    const uchar4 *__restrict__ chosen4 = reinterpret_cast<const uchar4 *>(P->chosen);
    uint4 *__restrict__ snap4 = reinterpret_cast<uint4 *>(P->snap);
    uint2 *above = P->above + (uint64_t)blockIdx.x * (quads * 4u + 1u) * kWG;
    const bool merge = n > kTopList;   // else all counts fit where the list is read from
    unsigned long long m = 0;
    auto list = [&](bool in, uint32_t x, uint32_t c) {   // (every lane of the wave)
        const uint64_t who = __ballot(in);
        if (who == 0ull) return;
        uint32_t at = 0;
        if (lane_id() == 0) at = atomicAdd(&listed, (uint32_t)__popcll(who));
        at = wave_bcast(at, 0);
        if (in) above[at + lane_rank(who)] = make_uint2(x, c);
    };
    for (uint32_t i = 0; i < quads; ++i) {
        const uint64_t q = ((uint64_t)blockIdx.x * quads + i) * kWG + threadIdx.x;
        const uint64_t v = 4 * q;
        uint32_t c[4] = {0u, 0u, 0u, 0u};
        uint8_t ch[4] = {1, 1, 1, 1};
        if (q < n4) {
            const uint4 cq = cnt4[q];
            const uchar4 hq = chosen4[q];
            if (kTopk) snap4[q] = cq;
            c[0] = cq.x; c[1] = cq.y; c[2] = cq.z; c[3] = cq.w;
            ch[0] = hq.x; ch[1] = hq.y; ch[2] = hq.z; ch[3] = hq.w;
        } else if (v < n) {
            for (uint32_t t = 0; v + t < n; ++t) {
                c[t] = P->cnt[v + t];
                ch[t] = P->chosen[v + t];
                if (kTopk) P->snap[v + t] = c[t];
            }
        }
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            const unsigned long long key = argmax_key(c[t], ch[t], (uint32_t)v + t);   // absent ones count as chosen
            m = key > m ? key : m;
            if (kTopk) {
                const uint32_t b = c[t] - lo;   // lo is at least 1, absent counts are 0
                const bool in = c[t] >= lo, near = in && merge && b < (uint32_t)kWG;
                if (near) {
                    const uint32_t b0 = uni(b);
                    const uint64_t same = __ballot(b == b0);
                    if (b != b0) atomicAdd(&many[b], 1u);
                    else if (lane_rank(same) == 0u) atomicAdd(&many[b0], (uint32_t)__popcll(same));
                }
                list(in && !near, c[t], 1u);
            }
        }
    }
    if (kTopk && merge) {
        __syncthreads();
        const uint32_t c = many[threadIdx.x];
        list(c != 0u, lo + threadIdx.x, c);
    }
    m = wave_max(m);
    if (lane_id() == 0) part[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWavesPerWG; ++w) m = part[w] > m ? part[w] : m;
        P->slot_key[blockIdx.x] = m;
        if (kTopk) P->above_n[blockIdx.x] = listed;
    }
}

// The best key over k_scan's slots (the whole workgroup).
__device__ __forceinline__ unsigned long long best_key(const GreedyParams *__restrict__ P, uint32_t slots) {
    __shared__ unsigned long long part[kWavesPerWG];
    unsigned long long m = 0;
    for (uint32_t i = threadIdx.x; i < slots; i += kWG) {
        const unsigned long long x = P->slot_key[i];
        m = x > m ? x : m;
    }
    m = wave_max(m);
    if (lane_id() == 0) part[threadIdx.x / kWave] = m;
    __syncthreads();
    m = part[0];
    for (int w = 1; w < kWavesPerWG; ++w) m = part[w] > m ? part[w] : m;
    __syncthreads();
    return uni64(m);
}

// Equation (8)'s term of this round, and the next guess (one workgroup).
__device__ void round_top_k(const GreedyParams *__restrict__ P, uint32_t slots, uint32_t round,
                            unsigned long long key) {
    __shared__ uint32_t hc[kBins];
    __shared__ uint32_t scan[kScanMax];   // inclusive scan of the list lengths
    __shared__ uint32_t part[kWavesPerWG];
    __shared__ uint2 val[kTopList];
    const uint32_t k = P->k, n = P->n, lo = P->state->lo;
    const uint32_t share = (P->quads * 4u + 1u) * kWG;
    uint32_t total = 0;
    for (uint32_t base = 0; base < slots; base += kWG) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t incl = wave_incl_scan(i < slots ? P->above_n[i] : 0u);
        if (lane_id() == kWave - 1) part[threadIdx.x / kWave] = incl;
        __syncthreads();
        uint32_t before = total;
        for (uint32_t q = 0; q < kWavesPerWG; ++q) {
            if (q < threadIdx.x / kWave) before += part[q];
            total += part[q];
        }
        if (i < slots) scan[i] = before + incl;
        __syncthreads();
    }
    auto listed = [&](uint32_t i) -> uint2 {   // i-th list entry
        uint32_t a = 0, b = slots - 1u;
        while (a < b) {
            const uint32_t mid = (a + b) / 2u;
            if (scan[mid] > i) b = mid; else a = mid + 1u;
        }
        return P->above[(uint64_t)a * share + (i - (a ? scan[a - 1u] : 0u))];
    };
    const bool held = total <= kTopList;   // in LDS, so that each level reads them there
    if (held)
        for (uint32_t i = threadIdx.x; i < total; i += kWG) val[i] = listed(i);
    __syncthreads();
    unsigned long long sum = 0;
    uint32_t kth = 0;
    // no count is above the argmax's (chosen vertices have none)
    const uint32_t most = (uint32_t)(key >> 32) ? (uint32_t)(key >> 32) - 1u : 0u;
    bool ok = top_sum(hc, lo, most, k,
                      [&](auto &&f) {
                          for (uint32_t i = threadIdx.x; i < total; i += kWG) {
                              const uint2 x = held ? val[i] : listed(i);
                              f(x.x, x.y);
                          }
                      },
                      &sum, &kth);
    bool missed = false;
    if (!ok && lo > 1u) {
        // fewer than k listed: the guess was too high
        missed = true;
        ok = top_sum(hc, 1u, most, k,
                     [&](auto &&f) {
                         const uint4 *s4 = reinterpret_cast<const uint4 *>(P->snap);
                         const uint32_t n4 = n / 4u;
                         for (uint32_t q = threadIdx.x; q < n4; q += kWG) {
                             const uint4 x = s4[q];
                             f(x.x, 1u);
                             f(x.y, 1u);
                             f(x.z, 1u);
                             f(x.w, 1u);
                         }
                         if (threadIdx.x < n % 4u) f(P->snap[4u * n4 + threadIdx.x], 1u);
                     },
                     &sum, &kth);
    }
    // (still fewer: the remaining largest counts are zeros)
    if (threadIdx.x == 0) {
        P->ub[round] = sum;
        RoundState st = *P->state;
        const unsigned long long gain = (key >> 32) ? (key >> 32) - 1ull : 0ull;
        const unsigned long long left = P->theta - st.covered;
        // sets covered now take about the same share of every large count
        const float keep = left ? 1.0f - (float)gain / (float)left : 1.0f;
        // lists of a few times k up to what LDS holds: the gap below the
        // expected value widens before it misses, and narrows again
        if (missed) st.gap = fminf(0.95f, 2.0f * st.gap);
        else if (total > kTopList) st.gap *= 0.7f;
        else if (total < 4u * k + 256u) st.gap = fminf(0.95f, 1.3f * st.gap);
        const float guess = (float)kth * keep * (1.0f - st.gap);
        st.lo = ok && guess > 1.0f ? (uint32_t)guess : 1u;
        st.covered += gain;
        *P->state = st;
    }
}

// Position search in the ascending members of a big set, kGroup lanes at once
// (all of them call it with the same arguments): whether v is a member.
__device__ __forceinline__ bool group_find(const uint32_t *__restrict__ m, uint32_t size, uint32_t v) {
    const uint32_t gl = threadIdx.x % kGroup, shift = (lane_id() / kGroup) * kGroup;
    uint32_t lo = 0, hi = size;   // v, if a member, lies in [lo, hi)
    while (hi - lo > kGroup) {
        const uint32_t step = (hi - lo) / (kGroup + 1u) + 1u;
        const uint32_t at = lo + (gl + 1u) * step;
        const bool le = at < hi && m[at] <= v;
        const uint32_t c = (uint32_t)__popcll((__ballot(le) >> shift) & ((1ull << kGroup) - 1ull));
        lo += c * step;
        hi = min(hi, lo + step);
    }
    const bool eq = lo + gl < hi && m[lo + gl] == v;
    return ((__ballot(eq) >> shift) & ((1ull << kGroup) - 1ull)) != 0ull;
}

// Covers the small sets inv[x0, x1) not covered before, kLanes lanes per set.
template <uint32_t kLanes>
__device__ __forceinline__ void cover_small(const GreedyParams *__restrict__ P, uint64_t x0, uint64_t x1,
                                            uint32_t workers, uint32_t stamp) {
    constexpr uint32_t kPerWG = kWG / kLanes;
    const uint64_t *__restrict__ off = P->off;
    const uint32_t *__restrict__ mem = P->mem;
    const uint32_t *__restrict__ inv = P->inv;
    uint32_t *__restrict__ covered = P->covered;
    uint32_t *__restrict__ cnt = P->cnt;
    for (uint64_t x = x0 + (uint64_t)blockIdx.x * kPerWG + threadIdx.x / kLanes; x < x1;
         x += (uint64_t)workers * kPerWG) {
        const uint32_t j = inv[x];
        if (covered[j] != 0u) continue;
        const uint64_t beg = off[j], end = off[j + 1];
        if (threadIdx.x % kLanes == 0) covered[j] = stamp;   // the set's lanes are one wave's: all have read it
        for_members<kLanes>(beg, end, [&](uint64_t e, uint32_t count) {
            uint32_t u[kUnroll];
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) u[t] = t < count ? mem[e + t * kLanes] : 0u;
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t)
                if (t < count) atomicSub(&cnt[u[t]], 1u);
        });
    }
}

// Round `round`: the argmax seed s is recorded (by workgroup 0) and its sets
// not covered before are covered.  Small sets, one per group of kGroup lanes:
// each appears once in s's list, so its group owns it.  Big sets: looked up
// and listed for k_sub.  With kTopk the last workgroup takes Equation (8)'s
// term instead (round = k: only that).
template <bool kTopk>
__global__ __launch_bounds__(kWG) void k_cover(const GreedyParams *__restrict__ P, uint32_t slots, uint32_t round) {
    const unsigned long long key = best_key(P, slots);
    if (kTopk && blockIdx.x == gridDim.x - 1u) {
        round_top_k(P, slots, round, key);
        return;
    }
    if (round >= P->k) return;
    const uint32_t s = 0xFFFFFFFFu - (uint32_t)key;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        P->seeds[round] = s;
        P->gains[round] = (key >> 32) - 1ull;
        P->chosen[s] = 1;
    }
    const uint32_t workers = kTopk ? gridDim.x - 1u : gridDim.x;
    const uint64_t *__restrict__ off = P->off;
    const uint32_t *__restrict__ mem = P->mem;
    uint32_t *__restrict__ covered = P->covered;
    const uint32_t stamp = round + 1u, gl = threadIdx.x % kGroup;
    const uint64_t x0 = P->inv_off[s], x1 = x0 + P->nsmall[s];
    // few sets: a wave each (a set of 4096 members took 90 us with 16 lanes)
    if (x1 - x0 <= (uint64_t)workers * kWavesPerWG)
        cover_small<kWave>(P, x0, x1, workers, stamp);
    else
        cover_small<kGroup>(P, x0, x1, workers, stamp);
    const uint64_t nbig = P->nbig;
    if (nbig == 0ull) return;
    __shared__ uint32_t found;
    if (threadIdx.x == 0) found = 0u;
    __syncthreads();
    const uint64_t per = div_up(nbig, workers), b0 = blockIdx.x * per, b1 = min(b0 + per, nbig);
    for (uint64_t b = b0; b < b1; b += kGroupsPerWG) {   // whole waves stay together for the ballots
        const uint64_t i = b + threadIdx.x / kGroup;
        uint64_t j = 0, beg = 0;
        uint32_t size = 0;
        if (i < b1) {
            j = P->big[i];
            if (covered[j] == 0u) {
                beg = off[j];
                size = (uint32_t)(off[j + 1] - beg);
            }
        }
        if (group_find(mem + beg, size, s) && gl == 0) {
            covered[j] = stamp;
            P->hit[b0 + atomicAdd(&found, 1u)] = (uint32_t)i;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) P->hit_n[blockIdx.x] = found;
}

// From about this many members of newly covered sets on, k_sub counts them range
// by range in LDS; below, device atomics on the counts themselves (about 35 a
// nanosecond) cost less than a workgroup per range.  80 sets of 20,000
// neighbouring vertices of a million in each of 50 rounds: 9.5 ms by ranges with
// the members read one by one, 1.4 ms by atomics; 20 rounds over 3000 sets of
// 9,500 of 10,000 vertices: 0.98 ms with 8 workgroups per range, 0.35 with as
// many as there is work for.
constexpr uint64_t kRangeMembers = 1u << 22;
constexpr uint32_t kSubSplit = 8;      // workgroups per range at least ...
constexpr uint32_t kSubSets = 16;      // ... more while each has about this many sets and workgroups are left

// Takes the members of the newly covered big sets off the counts.  `workers`
// workgroups of k_cover listed them, `per` big sets each.
__global__ __launch_bounds__(kWG) void k_sub(const GreedyParams *__restrict__ P, uint32_t workers) {
    __shared__ uint32_t lds[kRange];
    __shared__ uint32_t scan[kCoverMax];
    __shared__ uint32_t part[kWavesPerWG];
    const uint32_t wv = threadIdx.x / kWave, lane = lane_id();
    // inclusive scan of the lists' lengths
    uint32_t carry = 0;
    for (uint32_t base = 0; base < workers; base += kWG) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t incl = wave_incl_scan(i < workers ? P->hit_n[i] : 0u);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (uint32_t q = 0; q < kWavesPerWG; ++q) {
            if (q < wv) before += part[q];
            all += part[q];
        }
        if (i < workers) scan[i] = before + incl;
        carry += all;
        __syncthreads();
    }
    const uint64_t total = carry;
    if (total == 0u) return;
    const uint64_t per = div_up(P->nbig, workers);
    auto pick = [&](uint64_t i) -> uint64_t {   // i-th newly covered big set
        uint32_t lo = 0, hi = workers - 1u;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2u;
            if (scan[mid] > i) hi = mid; else lo = mid + 1u;
        }
        return P->hit[lo * per + (i - (lo ? scan[lo - 1u] : 0u))];
    };
    if (P->dir && total * P->big_mean >= kRangeMembers) {
        const uint32_t ranges = P->ranges;
        const uint32_t split = max(kSubSplit, min(total / kSubSets, gridDim.x / ranges)), jobs = ranges * split;
        for (uint32_t job = blockIdx.x; job < jobs; job += gridDim.x) {
            const uint64_t c = job / ranges;
            range_counts<-1>(lds, job % ranges, total * c / split, total * (c + 1u) / split, P->n, ranges, P->big,
                             P->dir, P->off, P->mem, P->cnt, pick);
        }
        return;
    }
    // every set in `parts` equal shares, a workgroup each, about two per workgroup
    const uint64_t parts = min(max((uint64_t)2u * gridDim.x / total, (uint64_t)1), (uint64_t)gridDim.x);
    for (uint64_t job = blockIdx.x; job < total * parts; job += gridDim.x) {
        const uint64_t i = job / parts, p = job - i * parts, j = P->big[pick(i)];
        const uint64_t beg = P->off[j], size = P->off[j + 1] - beg;
        for_members<kWG>(beg + size * p / parts, beg + size * (p + 1u) / parts, [&](uint64_t e, uint32_t count) {
            uint32_t u[kUnroll];
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) u[t] = t < count ? P->mem[e + t * kWG] : 0u;
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t)
                if (t < count) atomicSub(&P->cnt[u[t]], 1u);
        });
    }
}

// Seed flags; ids >= n are ignored.
__global__ void k_mark(const uint32_t *__restrict__ seeds, uint32_t k, uint32_t n, uint8_t *__restrict__ flags) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < k && seeds[i] < n) flags[seeds[i]] = 1;
}

// Small sets that hold a flagged vertex: kLanes lanes per set.
template <uint32_t kLanes>
__global__ __launch_bounds__(kWG) void k_hits_small(const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                                     uint64_t theta, const uint8_t *__restrict__ flags,
                                                     unsigned long long *__restrict__ hits) {
    constexpr uint32_t kPerWG = kWG / kLanes;
    constexpr uint64_t kMask = kLanes == 64 ? ~0ull : (1ull << kLanes) - 1ull;
    __shared__ uint32_t sum;
    if (threadIdx.x == 0) sum = 0u;
    __syncthreads();
    const uint32_t gl = threadIdx.x % kLanes, shift = (lane_id() / kLanes) * kLanes;
    uint32_t mine = 0;
    for (uint64_t j = (uint64_t)blockIdx.x * kPerWG + threadIdx.x / kLanes; j < theta;
         j += (uint64_t)gridDim.x * kPerWG) {
        const uint64_t beg = off[j], end = off[j + 1];
        if (end - beg > kBigSet) continue;
        for (uint64_t e0 = beg; e0 < end; e0 += kUnroll * kLanes) {
            uint32_t u[kUnroll], hit = 0;
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) {
                const uint64_t e = e0 + t * kLanes + gl;
                u[t] = e < end ? mem[e] : mem[beg];   // the first member stands in
            }
#pragma unroll
            for (uint32_t t = 0; t < kUnroll; ++t) hit |= flags[u[t]];
            if ((__ballot(hit != 0u) >> shift) & kMask) {
                mine += gl == 0 ? 1u : 0u;
                break;
            }
        }
    }
    if (mine) atomicAdd(&sum, mine);
    __syncthreads();
    if (threadIdx.x == 0 && sum) atomicAdd(hits, (unsigned long long)sum);
}

// Big sets that hold a seed, one wave per set: the lanes search for a seed
// each in the ascending members, 64 at a time; when the searches would read
// more than the members (k above size / kSearchCost), the members' flags are
// read instead.  2048 sets of 85,000 members, k = 100: 0.65 ms with flags.
constexpr uint64_t kSearchCost = 64;

__global__ __launch_bounds__(kWG) void k_hits_big(const uint64_t *__restrict__ list,
                                                   const unsigned long long *__restrict__ count,
                                                   const uint64_t *__restrict__ off, const uint32_t *__restrict__ mem,
                                                   const uint32_t *__restrict__ seeds, uint32_t k,
                                                   const uint8_t *__restrict__ flags,
                                                   unsigned long long *__restrict__ hits) {
    const uint64_t nb = *count, waves = (uint64_t)gridDim.x * kWavesPerWG;
    const uint32_t lane = lane_id();
    uint32_t mine = 0;   // sets of this wave (wave-uniform)
    for (uint64_t b = (uint64_t)blockIdx.x * kWavesPerWG + threadIdx.x / kWave; b < nb; b += waves) {
        const uint64_t j = list[b], beg = off[j], size = off[j + 1] - beg;
        const uint32_t *m = mem + beg;
        bool any = false;
        if (k <= size / kSearchCost) {
            for (uint32_t i0 = 0; i0 < k && !any; i0 += kWave) {
                bool hit = false;
                if (i0 + lane < k) {
                    const uint32_t v = seeds[i0 + lane];
                    uint64_t lo = 0, hi = size;
                    while (lo < hi) {
                        const uint64_t mid = (lo + hi) / 2u;
                        if (m[mid] < v) lo = mid + 1u; else hi = mid;
                    }
                    hit = lo < size && m[lo] == v;
                }
                any = __ballot(hit) != 0ull;
            }
        } else {
            for (uint64_t e = 0; e < size && !any; e += kWave)
                any = __ballot(e + lane < size && flags[m[e + lane]] != 0) != 0ull;
        }
        mine += any ? 1u : 0u;
    }
    if (lane == 0 && mine) atomicAdd(hits, (unsigned long long)mine);
}

uint32_t grid_for(uint64_t items, uint64_t per_block, uint32_t cap) {
    uint64_t g = div_up(items, per_block);
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(g, cap));
}

// The sets of the pool prefix above kBigSet members: list, and their number at
// ctr (zeroed by the caller), their members at `members` (likewise; may be null).
void big_list(hyperim_pool p, uint64_t theta, uint64_t *list, unsigned long long *ctr, unsigned long long *members,
              hipStream_t s) {
    if (theta)
        hipLaunchKernelGGL(k_big_list, dim3(grid_for(theta, kWG, 4096)), dim3(kWG), 0, s, p->off, theta, list, ctr,
                           members);
}

// k_hits_small with a wave per set, or a quarter of one where the pool's sets
// average fewer than 24 members.
void launch_hits_small(hyperim_pool p, uint64_t theta, const uint8_t *flags, unsigned long long *hits, hipStream_t s) {
    const bool wide = p->total >= 24u * p->count;
    const uint32_t grid = grid_for(theta, wide ? kWavesPerWG : kGroupsPerWG, 8192);
    hipLaunchKernelGGL(wide ? k_hits_small<kWave> : k_hits_small<kGroup>, dim3(grid), dim3(kWG), 0, s, p->off, p->mem,
                       theta, flags, hits);
}

// Byte offsets of arrays laid out one after another, 256-byte aligned.
struct Layout {
    size_t bytes = 0;
    size_t add(size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) & ~(size_t)255;
        return at;
    }
};

}  // namespace

int greedy_device(GreedyWorkspace &w, hyperim_graph g, hyperim_pool p, uint64_t theta, uint32_t k, hipStream_t s,
                  uint32_t *seeds_host, uint64_t *gains_host, uint64_t *ub_host) {
    const uint32_t n = g->n;
    const bool topk = ub_host != nullptr;
    // big sets and entries of the prefix
    HIM_CHECK(w.big.reserve(sizeof(uint64_t) * std::max<uint64_t>(theta, 1), s));
    HIM_CHECK(w.counters.reserve(4 * sizeof(unsigned long long), s));
    unsigned long long *ctr = w.counters.as<unsigned long long>();
    HIM_HIP(hipMemsetAsync(ctr, 0, 2 * sizeof(unsigned long long), s));
    big_list(p, theta, w.big.as<uint64_t>(), ctr, ctr + 1, s);
    uint64_t entries = 0, big[2] = {0, 0};
    HIM_HIP(hipMemcpyAsync(&entries, p->off + theta, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipMemcpyAsync(big, ctr, 2 * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    const uint64_t nbig = big[0];

    const uint32_t ranges = (uint32_t)div_up(n, kRange);
    const bool by_range = nbig && ranges <= kMaxRanges;
    // k_scan: at most kScanMax workgroups of `quads` 4-vertex loads per thread
    const uint32_t quads = (uint32_t)div_up(n, (uint64_t)4 * kWG * kScanMax);
    const uint32_t scan_grid = (uint32_t)div_up(n, (uint64_t)4 * kWG * quads);
    // k_cover: a group per set that a seed can have, and one more workgroup
    const uint32_t cover_grid = grid_for(std::max<uint64_t>(theta, kGroupsPerWG * div_up(nbig, kGroupsPerWG)),
                                         kGroupsPerWG, kCoverMax - 1u) + (topk ? 1u : 0u);
    const uint32_t workers = cover_grid - (topk ? 1u : 0u);
    // zeroed in one go, then arrays that are written before they are read
    Layout z, o;
    const size_t z_cnt = z.add(4ull * n), z_cursor = z.add(4ull * n), z_covered = z.add(4ull * std::max<uint64_t>(theta, 1)),
                 z_chosen = z.add(n);
    const size_t o_key = o.add(8ull * kScanMax), o_state = o.add(sizeof(RoundState)), o_ub = o.add(8ull * ((size_t)k + 1)),
                 o_hit_n = o.add(4ull * kCoverMax), o_above_n = o.add(4ull * kScanMax),
                 o_hit = o.add(4ull * div_up(nbig, workers) * workers), o_snap = o.add(topk ? 4ull * n : 0u),
                 o_above = o.add(topk ? 8ull * kWG * (4ull * quads + 1u) * scan_grid : 0u),
                 o_dir = o.add(by_range ? 4ull * nbig * (ranges + 1u) : 0u);
    HIM_CHECK(w.zeroed.reserve(z.bytes, s));
    HIM_CHECK(w.round.reserve(o.bytes, s));
    HIM_CHECK(w.inv_off.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(w.out.reserve(sizeof(uint64_t) * k + sizeof(uint32_t) * k, s));
    // the index holds the small sets; without ranges its offsets leave room
    // for the big ones' counts too
    const uint64_t inv_entries = by_range ? std::min<uint64_t>(entries, (theta - nbig) * kBigSet) : entries;
    HIM_CHECK(w.inv.reserve(sizeof(uint32_t) * std::max<uint64_t>(inv_entries, 1), s));
    HIM_CHECK(w.params.reserve(sizeof(GreedyParams), s));
    char *zb = w.zeroed.as<char>(), *ob = w.round.as<char>();
    HIM_HIP(hipMemsetAsync(zb, 0, z.bytes, s));
    GreedyParams hp{};
    hp.off = p->off;
    hp.mem = p->mem;
    hp.inv_off = w.inv_off.as<uint64_t>();
    hp.inv = w.inv.as<uint32_t>();
    hp.cnt = reinterpret_cast<uint32_t *>(zb + z_cnt);
    uint32_t *cursor = reinterpret_cast<uint32_t *>(zb + z_cursor);
    hp.nsmall = cursor;
    hp.covered = reinterpret_cast<uint32_t *>(zb + z_covered);
    hp.chosen = reinterpret_cast<uint8_t *>(zb + z_chosen);
    hp.gains = w.out.as<unsigned long long>();
    hp.seeds = reinterpret_cast<uint32_t *>(hp.gains + k);
    hp.n = n;
    hp.k = k;
    hp.quads = quads;
    hp.theta = theta;
    hp.slot_key = reinterpret_cast<unsigned long long *>(ob + o_key);
    hp.big = w.big.as<uint64_t>();
    hp.nbig = nbig;
    hp.big_mean = nbig ? big[1] / nbig : 0u;
    hp.dir = by_range ? reinterpret_cast<uint32_t *>(ob + o_dir) : nullptr;
    hp.ranges = ranges;
    hp.hit = reinterpret_cast<uint32_t *>(ob + o_hit);
    hp.hit_n = reinterpret_cast<uint32_t *>(ob + o_hit_n);
    hp.snap = reinterpret_cast<uint32_t *>(ob + o_snap);
    hp.above = reinterpret_cast<uint2 *>(ob + o_above);
    hp.above_n = reinterpret_cast<uint32_t *>(ob + o_above_n);
    hp.state = reinterpret_cast<RoundState *>(ob + o_state);
    hp.ub = reinterpret_cast<unsigned long long *>(ob + o_ub);
    static_assert(sizeof(GreedyParams) <= sizeof(w.params_host), "parameter block");
    memcpy(w.params_host, &hp, sizeof(hp));
    HIM_HIP(hipMemcpyAsync(w.params.ptr, w.params_host, sizeof(GreedyParams), hipMemcpyHostToDevice, s));
    const GreedyParams *P = w.params.as<GreedyParams>();

    // counts, the inverted index of the small sets: a wave per set, or a
    // quarter of one where sets average fewer than 24 members
    const bool wide = entries >= 24u * theta;
    const uint32_t set_grid = grid_for(theta, wide ? kWavesPerWG : kGroupsPerWG, 8192);
    if (by_range) {
        if (theta > nbig)
            hipLaunchKernelGGL(wide ? k_hist_small<kWave> : k_hist_small<kGroup>, dim3(set_grid), dim3(kWG), 0, s,
                               p->off, p->mem, theta, hp.cnt);
    } else if (entries) {
        hipLaunchKernelGGL(k_hist, dim3(grid_for(entries, kWG, 8192)), dim3(kWG), 0, s, p->mem, entries, hp.cnt);
    }
    if (theta > nbig) {
        HIM_CHECK(scan_u32_to_u64(hp.cnt, w.inv_off.as<uint64_t>(), n, 0, w.scan_tmp, s));
        hipLaunchKernelGGL(wide ? k_inv_small<kWave> : k_inv_small<kGroup>, dim3(set_grid), dim3(kWG), 0, s, p->off,
                           p->mem, theta, hp.inv_off, cursor, w.inv.as<uint32_t>());
    } else {
        HIM_HIP(hipMemsetAsync(w.inv_off.ptr, 0, sizeof(uint64_t) * ((size_t)n + 1), s));
    }
    if (by_range) {
        uint32_t *dir = const_cast<uint32_t *>(hp.dir);
        hipLaunchKernelGGL(k_dir, dim3(grid_for(nbig * (ranges + 1u), kWG, 8192)), dim3(kWG), 0, s, hp.big, nbig, ranges,
                           p->off, p->mem, dir);
        // about 2048 workgroups, at least 16 sets each
        const uint32_t per = (uint32_t)std::max<uint64_t>(16, div_up(nbig * ranges, 2048));
        hipLaunchKernelGGL(k_hist_big, dim3((uint32_t)div_up(nbig, per) * ranges), dim3(kWG), 0, s, hp.big, nbig, per, n,
                           ranges, dir, p->off, p->mem, hp.cnt);
    }
    // the k rounds; with Equation (8) one more for the term after the last
    if (topk) hipLaunchKernelGGL(k_first_lo, dim3(1), dim3(kWG), 0, s, P);
    for (uint32_t i = 0; i < k + (topk ? 1u : 0u); ++i) {
        if (topk) {
            hipLaunchKernelGGL(k_scan<true>, dim3(scan_grid), dim3(kWG), 0, s, P);
            hipLaunchKernelGGL(k_cover<true>, dim3(i < k ? cover_grid : 1u), dim3(kWG), 0, s, P, scan_grid, i);
        } else {
            hipLaunchKernelGGL(k_scan<false>, dim3(scan_grid), dim3(kWG), 0, s, P);
            hipLaunchKernelGGL(k_cover<false>, dim3(cover_grid), dim3(kWG), 0, s, P, scan_grid, i);
        }
        if (nbig && i + 1 < k + (topk ? 1u : 0u))
            hipLaunchKernelGGL(k_sub, dim3(1024), dim3(kWG), 0, s, P, workers);
    }
    HIM_HIP(hipGetLastError());
    if (seeds_host) HIM_HIP(hipMemcpyAsync(seeds_host, hp.seeds, sizeof(uint32_t) * k, hipMemcpyDeviceToHost, s));
    if (gains_host) HIM_HIP(hipMemcpyAsync(gains_host, hp.gains, sizeof(uint64_t) * k, hipMemcpyDeviceToHost, s));
    if (ub_host)
        HIM_HIP(hipMemcpyAsync(ub_host, hp.ub, sizeof(uint64_t) * ((size_t)k + 1), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    w.seeds_dev = hp.seeds;
    return HYPERIM_OK;
}

int coverage_device(GreedyWorkspace &w, hyperim_graph g, hyperim_pool p, uint64_t theta, const uint32_t *seeds_dev,
                    uint32_t k, hipStream_t s, uint64_t *covered_host) {
    const uint32_t n = g->n;
    // hit and big-set counters, then the seed flags, zeroed together
    HIM_CHECK(w.flags.reserve(256 + (size_t)n, s));
    HIM_CHECK(w.big.reserve(sizeof(uint64_t) * std::max<uint64_t>(theta, 1), s));
    unsigned long long *ctr = w.flags.as<unsigned long long>();
    uint8_t *flags = w.flags.as<uint8_t>() + 256;
    HIM_HIP(hipMemsetAsync(ctr, 0, 256 + (size_t)n, s));
    hipLaunchKernelGGL(k_mark, dim3(grid_for(k, kWG, 65535)), dim3(kWG), 0, s, seeds_dev, k, n, flags);
    big_list(p, theta, w.big.as<uint64_t>(), ctr + 1, nullptr, s);
    if (theta) {
        launch_hits_small(p, theta, flags, ctr, s);
        hipLaunchKernelGGL(k_hits_big, dim3(grid_for(theta, kWavesPerWG, 1024)), dim3(kWG), 0, s, w.big.as<uint64_t>(),
                           ctr + 1, p->off, p->mem, seeds_dev, k, flags, ctr);
    }
    HIM_HIP(hipGetLastError());
    unsigned long long h = 0;
    HIM_HIP(hipMemcpyAsync(&h, ctr, sizeof(h), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    *covered_host = h;
    return HYPERIM_OK;
}

// ---- coverage without allocation ---------------------------------------------
// Scratch of hyperim_coverage_noalloc: the hit counters, the seed flags (n
// bytes) and the list of big sets (8 bytes per set), in one static device
// array.  Each device holds its own copy; host code uses the address that
// hipGetSymbolAddress returns on that device, never the array's name.
constexpr size_t kScratchBytes = 32ull << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char *g_scratch[kMaxDevices] = {};

// The device address of `scratch` on `device` (the current device), looked
// up once per device.
int scratch_address(int device, unsigned char **out) {
    if (device < 0 || device >= kMaxDevices) {
        set_error_detail("device index beyond the scratch table");
        return HYPERIM_EINVAL;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mutex);
    if (!g_scratch[device]) {
        void *p = nullptr;
        HIM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch[device] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch[device];
    return HYPERIM_OK;
}

__global__ void k_zero_words(unsigned long long *__restrict__ p, uint64_t words) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

__global__ void k_store_count(const unsigned long long *__restrict__ src, uint64_t *__restrict__ dst) { *dst = *src; }

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

}  // namespace hyperim

using namespace hyperim;

extern "C" int hyperim_coverage_noalloc(hyperim_graph g, hyperim_pool pool, uint64_t theta, const uint32_t *seeds_dev,
                                        uint32_t k, void *stream, uint64_t *covered_dev) {
    if (!g || !pool || pool->g != g || !covered_dev || (k && !seeds_dev)) return HYPERIM_EINVAL;
    HIM_CHECK(check_device(g));
    if (theta > pool->count || k > g->n) {
        set_error_detail("need theta <= pool size and k <= n");
        return HYPERIM_EINVAL;
    }
    // layout: counters (256 B), flags (n bytes, 256-aligned), big-set list
    const size_t flags_at = 256, list_at = flags_at + round256(g->n);
    if (list_at + 8 * theta > kScratchBytes) {
        set_error_detail("coverage without allocation needs n + 8 theta bytes within its 32 MiB scratch");
        return HYPERIM_ECAPACITY;
    }
    unsigned char *base = nullptr;
    HIM_CHECK(scratch_address(g->device, &base));
    hipStream_t s = as_stream(stream);
    unsigned long long *ctr = reinterpret_cast<unsigned long long *>(base);
    uint8_t *flags = base + flags_at;
    uint64_t *list = reinterpret_cast<uint64_t *>(base + list_at);
    const uint64_t words = list_at / 8;   // counters and flags start at zero
    hipLaunchKernelGGL(k_zero_words, dim3(grid_for(words, kWG, 4096)), dim3(kWG), 0, s, ctr, words);
    if (k) hipLaunchKernelGGL(k_mark, dim3(grid_for(k, kWG, 65535)), dim3(kWG), 0, s, seeds_dev, k, g->n, flags);
    if (theta) {
        big_list(pool, theta, list, ctr + 1, nullptr, s);
        launch_hits_small(pool, theta, flags, ctr, s);
        hipLaunchKernelGGL(k_hits_big, dim3(grid_for(theta, kWavesPerWG, 1024)), dim3(kWG), 0, s, list, ctr + 1,
                           pool->off, pool->mem, seeds_dev, k, flags, ctr);
    }
    hipLaunchKernelGGL(k_store_count, dim3(1), dim3(1), 0, s, ctr, covered_dev);
    HIM_HIP(hipGetLastError());
    return HYPERIM_OK;
}
