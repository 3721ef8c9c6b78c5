// Device-resident hypergraph (Section 2.1: G = (V, HE) with member lists
// V(he)).  Validates the caller's CSR, transposes it into vertex -> hyperedge
// incidence lists with ascending hyperedge ids, and derives the per-target
// coin thresholds of the IC channel model.  G_w is never materialised.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "block_table.h"
#include "dev_common.h"
#include "internal.h"

namespace hyperim {
namespace {

constexpr int kBlock = 256;
constexpr uint32_t kSmallSeg = 16;     // insertion sort by one thread
constexpr uint32_t kMidSeg = 4096;     // bitonic sort in LDS by one workgroup

enum Flag : uint32_t { kBadOffsets = 1, kBadId = 2, kDuplicate = 4 };

__global__ void k_check_offsets(const uint32_t *__restrict__ he_off, uint32_t m, uint32_t *flag) {
    uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e == 0 && he_off[0] != 0u) atomicOr(flag, (uint32_t)kBadOffsets);
    if (e < m && he_off[e + 1] < he_off[e]) atomicOr(flag, (uint32_t)kBadOffsets);
}

// Incidences per vertex.  Each workgroup takes chunks of kChunk consecutive
// incidences and adds per-vertex totals to global memory once per chunk.
constexpr uint32_t kChunkPer = 8;                 // incidences per thread per chunk
constexpr uint32_t kChunk = kBlock * kChunkPer;
constexpr uint32_t kTableSlots = 4096;

__global__ __launch_bounds__(kBlock) void k_count(const uint32_t *__restrict__ he_mem, uint64_t nnz, uint32_t n,
                                                   uint32_t *__restrict__ cnt, uint32_t *flag) {
    __shared__ BlockTable<kTableSlots> tab;
    __shared__ uint32_t tval[kTableSlots];
    tab.clear_keys();
    for (uint32_t s = threadIdx.x; s < kTableSlots; s += kBlock) tval[s] = 0;
    __syncthreads();
    for (uint64_t base = (uint64_t)blockIdx.x * kChunk; base < nnz; base += (uint64_t)gridDim.x * kChunk) {
        for (uint32_t r = 0; r < kChunkPer; ++r) {
            const uint64_t i = base + r * kBlock + threadIdx.x;
            if (i >= nnz) break;
            const uint32_t v = he_mem[i];
            if (v >= n) {
                atomicOr(flag, (uint32_t)kBadId);
                continue;
            }
            const uint32_t sl = tab.slot(v);
            if (sl != kTableEmpty) atomicAdd(&tval[sl], 1u);
            else atomicAdd(&cnt[v], 1u);
        }
        __syncthreads();
        for (uint32_t sl = threadIdx.x; sl < kTableSlots; sl += kBlock) {
            const uint32_t v = tab.key[sl];
            if (v != kTableEmpty) {
                atomicAdd(&cnt[v], tval[sl]);
                tab.key[sl] = kTableEmpty;
                tval[sl] = 0;
            }
        }
        __syncthreads();
    }
}

// Number of vertices whose segments are sorted through bitmaps.
__global__ __launch_bounds__(kBlock) void k_count_big(const uint32_t *__restrict__ cnt, uint32_t n,
                                                       uint32_t *__restrict__ out) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    const uint64_t who = __ballot(v < n && cnt[v] > kMidSeg);
    if (lane_id() == 0 && who) atomicAdd(out, (uint32_t)__popcll(who));
}

__global__ void k_u64_to_u32(const uint64_t *__restrict__ in, uint32_t *__restrict__ out, uint64_t count) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x)
        out[i] = (uint32_t)in[i];
}

// Scatter every incidence (he, position) into its vertex's segment (order
// inside a segment fixed afterwards by sorting).  Per chunk of consecutive
// incidences, each workgroup ranks its incidences of one vertex in LDS and
// reserves the vertex's places with one global atomic.  The owner hyperedge of
// an incidence is searched between those of the chunk's ends, a handful of
// offsets in L1 instead of all m (11.7M incidences: 0.89 -> 0.45 ms).
constexpr uint32_t kFillPer = 4;
constexpr uint32_t kFillChunk = kBlock * kFillPer;
constexpr uint32_t kFillSlots = 2048;

// Owner hyperedge of incidence i: the last e in [lo, hi) with he_off[e] <= i
// (skipping empty ones), given he_off[lo] <= i < he_off[hi].
__device__ __forceinline__ uint32_t owner_edge(const uint32_t *__restrict__ he_off, uint32_t lo, uint32_t hi,
                                               uint32_t i) {
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (he_off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kBlock) void k_fill(const uint32_t *__restrict__ he_off,
                                                  const uint32_t *__restrict__ he_mem, uint32_t m, uint64_t nnz,
                                                  const uint32_t *__restrict__ v_off, uint32_t *__restrict__ cursor,
                                                  uint32_t *__restrict__ v_he) {
    __shared__ BlockTable<kFillSlots> tab;
    __shared__ uint32_t tcnt[kFillSlots], tbase[kFillSlots];
    __shared__ uint32_t ends[2];
    tab.clear_keys();
    for (uint32_t s = threadIdx.x; s < kFillSlots; s += kBlock) tcnt[s] = 0;
    for (uint64_t base = (uint64_t)blockIdx.x * kFillChunk; base < nnz; base += (uint64_t)gridDim.x * kFillChunk) {
        if (threadIdx.x < 2) {   // owners of the chunk's first and last incidence
            const uint64_t i = threadIdx.x ? min(base + kFillChunk, nnz) - 1u : base;
            ends[threadIdx.x] = owner_edge(he_off, 0u, m, (uint32_t)i);
        }
        __syncthreads();
        const uint32_t elo = ends[0], ehi = ends[1] + 1u;
        uint32_t ev[kFillPer], vv[kFillPer], sl[kFillPer], rk[kFillPer];
#pragma unroll
        for (uint32_t r = 0; r < kFillPer; ++r) {
            sl[r] = kTableEmpty;
            const uint64_t i = base + r * kBlock + threadIdx.x;
            if (i >= nnz) continue;
            const uint32_t e = owner_edge(he_off, elo, ehi, (uint32_t)i), v = he_mem[i];
            ev[r] = e;
            vv[r] = v;
            sl[r] = tab.slot(v);
            if (sl[r] != kTableEmpty) rk[r] = atomicAdd(&tcnt[sl[r]], 1u);
            else v_he[v_off[v] + atomicAdd(&cursor[v], 1u)] = e;
        }
        __syncthreads();
        for (uint32_t s = threadIdx.x; s < kFillSlots; s += kBlock) {
            const uint32_t v = tab.key[s];
            if (v != kTableEmpty) tbase[s] = v_off[v] + atomicAdd(&cursor[v], tcnt[s]);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < kFillPer; ++r)
            if (sl[r] != kTableEmpty) v_he[tbase[sl[r]] + rk[r]] = ev[r];
        __syncthreads();
        for (uint32_t s = threadIdx.x; s < kFillSlots; s += kBlock) {
            tab.key[s] = kTableEmpty;
            tcnt[s] = 0;
        }
        __syncthreads();
    }
}

// Short segments: one thread, insertion sort; flags duplicates.
__global__ void k_sort_small(const uint32_t *__restrict__ v_off, uint32_t n, uint32_t *__restrict__ v_he,
                             uint32_t *__restrict__ mid_list, uint32_t *__restrict__ big_list,
                             uint32_t *__restrict__ counts, uint32_t *flag) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    uint32_t b = v_off[v], len = v_off[v + 1] - b;
    if (len > kMidSeg) {
        big_list[atomicAdd(&counts[1], 1u)] = v;
        return;
    }
    if (len > kSmallSeg) {
        mid_list[atomicAdd(&counts[0], 1u)] = v;
        return;
    }
    uint32_t a[kSmallSeg];
    for (uint32_t i = 0; i < len; ++i) a[i] = v_he[b + i];
    for (uint32_t i = 1; i < len; ++i) {
        uint32_t x = a[i];
        uint32_t k = i;
        while (k > 0 && a[k - 1] > x) {
            a[k] = a[k - 1];
            --k;
        }
        a[k] = x;
    }
    for (uint32_t i = 0; i < len; ++i) {
        if (i && a[i] == a[i - 1]) atomicOr(flag, (uint32_t)kDuplicate);
        v_he[b + i] = a[i];
    }
}

// Medium segments: one workgroup per vertex, bitonic sort in LDS.
__global__ __launch_bounds__(kBlock) void k_sort_mid(const uint32_t *__restrict__ v_off,
                                                     const uint32_t *__restrict__ list, const uint32_t *counts,
                                                     uint32_t *__restrict__ v_he, uint32_t *flag) {
    __shared__ uint32_t buf[kMidSeg];
    const uint32_t nlist = counts[0];
    for (uint32_t w = blockIdx.x; w < nlist; w += gridDim.x) {
        const uint32_t v = list[w];
        const uint32_t b = v_off[v], len = v_off[v + 1] - b;
        uint32_t P = 1;
        while (P < len) P <<= 1;
        for (uint32_t i = threadIdx.x; i < P; i += blockDim.x) buf[i] = i < len ? v_he[b + i] : 0xFFFFFFFFu;
        __syncthreads();
        for (uint32_t k = 2; k <= P; k <<= 1) {
            for (uint32_t jj = k >> 1; jj > 0; jj >>= 1) {
                for (uint32_t i = threadIdx.x; i < P; i += blockDim.x) {
                    uint32_t x = i ^ jj;
                    if (x > i) {
                        uint32_t p = buf[i], q = buf[x];
                        bool up = (i & k) == 0;
                        if ((p > q) == up) {
                            buf[i] = q;
                            buf[x] = p;
                        }
                    }
                }
                __syncthreads();
            }
        }
        for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) {
            uint32_t x = buf[i];
            if (i && buf[i - 1] == x) atomicOr(flag, (uint32_t)kDuplicate);
            v_he[b + i] = x;
        }
        __syncthreads();
    }
}

// Long segments (hub vertices): the hyperedge ids are marked in a bitmap over
// all m hyperedges and read back in ascending order.  A repeated id shows up
// as fewer set bits than the segment length.  A batch of hubs at a time, each
// step spread over the whole grid -- kBigParts workgroups mark a segment, one
// workgroup per kBigTile words counts and later writes -- where one workgroup
// per hub took 4.2 ms against 0.4 (a million vertices, 2e6 hyperedges, Zipf
// 1.1).
constexpr uint32_t kBigParts = 32;
constexpr uint32_t kBigTile = 2048;              // bitmap words per workgroup
constexpr uint64_t kBigBudget = 1ull << 30;      // bytes of bitmaps per batch

__global__ __launch_bounds__(kBlock) void k_big_mark(const uint32_t *__restrict__ v_off,
                                                     const uint32_t *__restrict__ list,
                                                     const uint32_t *__restrict__ v_he, uint32_t *__restrict__ bitmaps,
                                                     uint32_t words) {
    const uint32_t h = blockIdx.x / kBigParts, part = blockIdx.x % kBigParts;
    const uint32_t v = list[h], b = v_off[v];
    const uint64_t len = v_off[v + 1] - b;
    uint32_t *bm = bitmaps + (uint64_t)h * words;
    const uint64_t i1 = len * (part + 1u) / kBigParts;
    for (uint64_t i = len * part / kBigParts + threadIdx.x; i < i1; i += kBlock) {
        const uint32_t e = v_he[b + i];
        atomicOr(&bm[e >> 5], 1u << (e & 31u));
    }
}

__global__ __launch_bounds__(kBlock) void k_big_tiles(const uint32_t *__restrict__ bitmaps, uint32_t words,
                                                      uint32_t tiles, uint32_t *__restrict__ tile_cnt) {
    __shared__ uint32_t tot;
    if (threadIdx.x == 0) tot = 0u;
    __syncthreads();
    const uint32_t h = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const uint32_t *bm = bitmaps + (uint64_t)h * words;
    uint32_t c = 0;
    for (uint32_t i = threadIdx.x; i < kBigTile; i += kBlock) {
        const uint64_t w = (uint64_t)tile * kBigTile + i;
        if (w < words) c += (uint32_t)__popc(bm[w]);
    }
    c = wave_sum(c);
    if (lane_id() == 0) atomicAdd(&tot, c);
    __syncthreads();
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = tot;
}

// One workgroup per hub: its tile counts become offsets; the duplicate check.
__global__ __launch_bounds__(kBlock) void k_big_scan(const uint32_t *__restrict__ v_off,
                                                     const uint32_t *__restrict__ list, uint32_t tiles,
                                                     uint32_t *__restrict__ tile_cnt, uint32_t *flag) {
    __shared__ uint32_t part[kBlock / kWave];
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    uint32_t *tc = tile_cnt + (uint64_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < tiles; base += kBlock) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < tiles ? tc[i] : 0u;
        const uint32_t incl = wave_incl_scan(x);
        if (lane == kWave - 1) part[wv] = incl;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (uint32_t q = 0; q < kBlock / kWave; ++q) {
            if (q < wv) before += part[q];
            all += part[q];
        }
        if (i < tiles) tc[i] = before + incl - x;
        carry += all;
        __syncthreads();
    }
    const uint32_t v = list[blockIdx.x];
    if (threadIdx.x == 0 && carry != v_off[v + 1] - v_off[v]) atomicOr(flag, (uint32_t)kDuplicate);
}

// Writes a tile's ids; with a duplicate in the segment fewer ids come out than
// were in it (never more).
__global__ __launch_bounds__(kBlock) void k_big_write(const uint32_t *__restrict__ v_off,
                                                      const uint32_t *__restrict__ list,
                                                      const uint32_t *__restrict__ bitmaps, uint32_t words,
                                                      uint32_t tiles, const uint32_t *__restrict__ tile_off,
                                                      uint32_t *__restrict__ v_he) {
    constexpr uint32_t kPer = kBigTile / kBlock;   // consecutive words per thread
    __shared__ uint32_t part[kBlock / kWave];
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint32_t h = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const uint32_t *bm = bitmaps + (uint64_t)h * words;
    const uint64_t w0 = (uint64_t)tile * kBigTile + threadIdx.x * kPer;
    uint32_t word[kPer], c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
        word[i] = w0 + i < words ? bm[w0 + i] : 0u;
        c += (uint32_t)__popc(word[i]);
    }
    const uint32_t incl = wave_incl_scan(c);
    if (lane == kWave - 1) part[wv] = incl;
    __syncthreads();
    uint32_t at = v_off[list[h]] + tile_off[blockIdx.x] + incl - c;
    for (uint32_t q = 0; q < wv; ++q) at += part[q];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i)
        while (word[i]) {
            const uint32_t bit = (uint32_t)__ffs(word[i]) - 1u;
            word[i] &= word[i] - 1u;
            v_he[at++] = (uint32_t)(w0 + i) * 32u + bit;
        }
}

// c(v) from the channel prefix over v's incidences, coin thresholds and
// per-vertex incidence weights.
__global__ void k_thresholds(uint32_t n, uint32_t model, float p, const uint32_t *__restrict__ v_off,
                             const unsigned long long *__restrict__ chan, unsigned long long *__restrict__ c,
                             uint32_t *__restrict__ thr, unsigned long long *__restrict__ weight,
                             unsigned long long *__restrict__ bytesw) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const uint32_t e0 = v_off[v], e1 = v_off[v + 1];
    const unsigned long long cv = chan[e1] - chan[e0];
    c[v] = cv;
    float pv;
    if (model == HYPERIM_MODEL_CONST || model == HYPERIM_MODEL_LT_CONST || model == HYPERIM_MODEL_GAPS_CONST) {
        pv = p;
    } else {
        pv = cv ? (float)(1.0 / (double)cv) : 0.0f;
    }
    uint32_t t;
    if (pv >= 1.0f) t = kAlways;
    else if (!(pv > 0.0f)) t = 0u;
    else t = (uint32_t)floor(ldexp((double)pv, 32));
    thr[v] = t;
    // d hyperedges of total size S = c + d: a member reads its offset pair (8 B),
    // d hyperedge ids and offset pairs (12 B each), S member ids (4 B each), and
    // costs 12 B of visited/queue/output traffic
    const unsigned long long d = e1 - e0;
    weight[v] = 2ull * d + cv;
    bytesw[v] = 20ull + 16ull * d + 4ull * cv;
}

// Philox blocks of a vertex's expansion: sum over its hyperedges of
// ceil(|he| / 4), from the prefix of those over the incidences.
// With it the vertex records are complete.
__global__ void k_philox_weight(uint32_t n, const uint32_t *__restrict__ v_off,
                                const unsigned long long *__restrict__ pre, const uint32_t *__restrict__ thr,
                                unsigned long long *__restrict__ phiw, uint4 *__restrict__ vrec) {
    const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const uint32_t e0 = v_off[v], e1 = v_off[v + 1];
    const unsigned long long q = pre[e1] - pre[e0];
    phiw[v] = q;
    vrec[v] = make_uint4(e0, e1 - e0, thr[v], (uint32_t)min(q, 0xFFFFFFFFull));
}

// Per incidence: its record, its channels |he| - 1 (the members other than the
// vertex itself) and its Philox blocks ceil(|he| / 4).
__global__ void k_incidence_spans(uint64_t nnz, const uint32_t *__restrict__ v_he, const uint32_t *__restrict__ he_off,
                                  uint4 *__restrict__ irec, uint32_t *__restrict__ channels,
                                  uint32_t *__restrict__ quads) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t he = v_he[e];
        const uint32_t b = he_off[he], sz = he_off[he + 1] - b;
        irec[e] = make_uint4(he, b, sz, 0u);
        channels[e] = sz - 1u;
        quads[e] = (sz + 3u) / 4u;
    }
}

// Channels of each incidence (v, he): |he| - 1.
__global__ void k_channel_counts(uint64_t nnz, const uint4 *__restrict__ irec, uint32_t *__restrict__ cnt) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (uint64_t)gridDim.x * blockDim.x)
        cnt[e] = irec[e].z - 1u;
}

uint32_t grid_for(uint64_t items, uint32_t block = kBlock, uint32_t cap = 65535u * 8u) {
    uint64_t g = div_up(items, block);
    if (g == 0) g = 1;
    return (uint32_t)std::min<uint64_t>(g, cap);
}

}  // namespace

// Exclusive prefix over all incidences of their channel counts |he| - 1: the
// channels into v are chan[v_off[v]] .. chan[v_off[v + 1]] (needs irec).
// cnt and tmp are scratch the caller keeps alive until the stream has run.
int channel_prefix(hyperim_graph g, DevBuf &cnt, DevBuf &tmp, hipStream_t s) {
    const uint64_t nnz = g->nnz;
    HIM_CHECK(g->chan.reserve(sizeof(uint64_t) * (nnz + 1), s));
    HIM_CHECK(cnt.reserve(sizeof(uint32_t) * std::max<uint64_t>(nnz, 1), s));
    if (nnz)
        hipLaunchKernelGGL(k_channel_counts, dim3(grid_for(nnz, kBlock, 8192)), dim3(kBlock), 0, s, nnz,
                           g->irec.as<uint4>(), cnt.as<uint32_t>());
    HIM_HIP(hipGetLastError());
    return scan_u32_to_u64(cnt.as<uint32_t>(), g->chan.as<uint64_t>(), nnz, 0, tmp, s);
}

int graph_build_device(hyperim_graph g, PrepWorkspace &w, hipStream_t s) {
    const uint32_t n = g->n, m = g->m;   // n at least 1
    const uint64_t nnz = g->nnz;
    DevBuf &flag_b = w.flag, &cnt_b = w.cnt, &off64_b = w.off64, &tmp_b = w.tmp;
    HIM_CHECK(flag_b.reserve(4 * sizeof(uint32_t), s));
    uint32_t *flag = flag_b.as<uint32_t>();   // flags, middle and long segments listed, long segments counted
    HIM_HIP(hipMemsetAsync(flag, 0, 4 * sizeof(uint32_t), s));

    hipLaunchKernelGGL(k_check_offsets, dim3(grid_for((uint64_t)m + 1)), dim3(kBlock), 0, s,
                       g->he_off.as<uint32_t>(), m, flag);
    HIM_CHECK(cnt_b.reserve(sizeof(uint32_t) * ((size_t)n + 1), s));
    HIM_HIP(hipMemsetAsync(cnt_b.ptr, 0, sizeof(uint32_t) * ((size_t)n + 1), s));
    hipLaunchKernelGGL(k_count, dim3(grid_for(nnz, kChunk, 4096)), dim3(kBlock), 0, s, g->he_mem.as<uint32_t>(), nnz, n,
                       cnt_b.as<uint32_t>(), flag);
    hipLaunchKernelGGL(k_count_big, dim3(grid_for(n)), dim3(kBlock), 0, s, cnt_b.as<uint32_t>(), n, flag + 3);
    uint32_t hflag[4] = {0, 0, 0, 0};
    HIM_HIP(hipMemcpyAsync(hflag, flag, sizeof(hflag), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    if (hflag[0]) {
        set_error_detail(hflag[0] & kBadOffsets ? "hyperedge offsets decrease or do not start at 0"
                                                : "member id >= n");
        return HYPERIM_EINVAL;
    }

    HIM_CHECK(off64_b.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(scan_u32_to_u64(cnt_b.as<uint32_t>(), off64_b.as<uint64_t>(), n, 0, tmp_b, s));
    HIM_CHECK(g->v_off.reserve(sizeof(uint32_t) * ((size_t)n + 1), s));
    hipLaunchKernelGGL(k_u64_to_u32, dim3(grid_for((uint64_t)n + 1)), dim3(kBlock), 0, s,
                       off64_b.as<uint64_t>(), g->v_off.as<uint32_t>(), (uint64_t)n + 1);

    HIM_CHECK(g->v_he.reserve(sizeof(uint32_t) * std::max<uint64_t>(nnz, 1), s));
    HIM_HIP(hipMemsetAsync(cnt_b.ptr, 0, sizeof(uint32_t) * ((size_t)n + 1), s));
    if (nnz)
        hipLaunchKernelGGL(k_fill, dim3(grid_for(nnz, kFillChunk, 4096)), dim3(kBlock), 0, s, g->he_off.as<uint32_t>(),
                           g->he_mem.as<uint32_t>(), m, nnz, g->v_off.as<uint32_t>(), cnt_b.as<uint32_t>(),
                           g->v_he.as<uint32_t>());

    // order every segment by hyperedge id
    DevBuf &lists_b = w.lists, &bm_b = w.bm;
    HIM_CHECK(lists_b.reserve(sizeof(uint32_t) * 2 * ((size_t)n + 1), s));
    uint32_t *mid_list = lists_b.as<uint32_t>();
    uint32_t *big_list = mid_list + n + 1;
    uint32_t *counts = flag + 1;  // [0] mid, [1] big
    const uint32_t *v_off = g->v_off.as<uint32_t>();
    uint32_t *v_he = g->v_he.as<uint32_t>();
    hipLaunchKernelGGL(k_sort_small, dim3(grid_for(n)), dim3(kBlock), 0, s, v_off, n, v_he, mid_list, big_list, counts,
                       flag);
    hipLaunchKernelGGL(k_sort_mid, dim3(std::min<uint32_t>(n, 4096)), dim3(kBlock), 0, s, v_off, mid_list, counts,
                       v_he, flag);
    if (const uint32_t nbig = hflag[3]) {
        const uint32_t words = (m + 31u) / 32u, tiles = (uint32_t)div_up(words, kBigTile);
        const uint32_t batch = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(nbig, kBigBudget / (4ull * words)));
        HIM_CHECK(bm_b.reserve(sizeof(uint32_t) * ((size_t)words + tiles) * batch, s));
        uint32_t *bitmaps = bm_b.as<uint32_t>(), *tile_cnt = bitmaps + (size_t)words * batch;
        for (uint32_t b0 = 0; b0 < nbig; b0 += batch) {
            const uint32_t cnt = std::min(batch, nbig - b0);
            HIM_HIP(hipMemsetAsync(bitmaps, 0, sizeof(uint32_t) * (size_t)words * cnt, s));
            hipLaunchKernelGGL(k_big_mark, dim3(cnt * kBigParts), dim3(kBlock), 0, s, v_off, big_list + b0, v_he,
                               bitmaps, words);
            hipLaunchKernelGGL(k_big_tiles, dim3(cnt * tiles), dim3(kBlock), 0, s, bitmaps, words, tiles, tile_cnt);
            hipLaunchKernelGGL(k_big_scan, dim3(cnt), dim3(kBlock), 0, s, v_off, big_list + b0, tiles, tile_cnt, flag);
            hipLaunchKernelGGL(k_big_write, dim3(cnt * tiles), dim3(kBlock), 0, s, v_off, big_list + b0, bitmaps,
                               words, tiles, tile_cnt, v_he);
        }
    }
    HIM_HIP(hipGetLastError());
    HIM_HIP(hipMemcpyAsync(hflag, flag, sizeof(uint32_t), hipMemcpyDeviceToHost, s));

    // spans, c(v) and the Philox weights: prefixes over the incidences, so a
    // hub costs what its incidences cost (with one wave per vertex the largest
    // hub of a million-vertex graph, 8e5 incidences, took 6-8 ms alone)
    HIM_CHECK(g->thr.reserve(sizeof(uint32_t) * n, s));
    HIM_CHECK(g->c.reserve(sizeof(uint64_t) * n, s));
    HIM_CHECK(g->weight.reserve(sizeof(uint64_t) * n, s));
    HIM_CHECK(g->bytesw.reserve(sizeof(uint64_t) * n, s));
    HIM_CHECK(g->phiw.reserve(sizeof(uint64_t) * n, s));
    HIM_CHECK(g->vrec.reserve(sizeof(uint4) * n, s));
    HIM_CHECK(g->irec.reserve(sizeof(uint4) * std::max<uint64_t>(nnz, 1), s));
    const size_t cnt_words = std::max<uint64_t>(nnz, 1);
    HIM_CHECK(w.k1.reserve(2 * sizeof(uint32_t) * cnt_words, s));
    HIM_CHECK(w.k2.reserve(sizeof(uint64_t) * (nnz + 1), s));
    uint32_t *channels = w.k1.as<uint32_t>(), *quads = channels + cnt_words;
    // linear-threshold and stratified-setting graphs keep the channel prefix
    const bool keep = g->lt() || g->layered();
    if (keep) HIM_CHECK(g->chan.reserve(sizeof(uint64_t) * (nnz + 1), s));
    uint64_t *chan = keep ? g->chan.as<uint64_t>() : w.k2.as<uint64_t>();
    if (nnz)
        hipLaunchKernelGGL(k_incidence_spans, dim3(grid_for(nnz, kBlock, 8192)), dim3(kBlock), 0, s, nnz, v_he,
                           g->he_off.as<uint32_t>(), g->irec.as<uint4>(), channels, quads);
    HIM_CHECK(scan_u32_to_u64(channels, chan, nnz, 0, tmp_b, s));
    hipLaunchKernelGGL(k_thresholds, dim3(grid_for(n)), dim3(kBlock), 0, s, n, g->prob.model, g->prob.p, v_off,
                       reinterpret_cast<const unsigned long long *>(chan), g->c.as<unsigned long long>(),
                       g->thr.as<uint32_t>(), g->weight.as<unsigned long long>(), g->bytesw.as<unsigned long long>());
    HIM_CHECK(scan_u32_to_u64(quads, w.k2.as<uint64_t>(), nnz, 0, tmp_b, s));
    hipLaunchKernelGGL(k_philox_weight, dim3(grid_for(n)), dim3(kBlock), 0, s, n, v_off,
                       w.k2.as<unsigned long long>(), g->thr.as<uint32_t>(), g->phiw.as<unsigned long long>(),
                       g->vrec.as<uint4>());
    HIM_HIP(hipGetLastError());
    HIM_HIP(hipStreamSynchronize(s));
    if (hflag[0] & kDuplicate) {
        set_error_detail("a vertex appears twice in one hyperedge");
        return HYPERIM_EINVAL;
    }
    return HYPERIM_OK;
}

}  // namespace hyperim
