// Sample-set division (Section 3.1.1) as tables, for the stratified-setting
// model: per vertex v the members of A(v) layer by layer (layer 1 = largest
// w(v,u)), ascending ids within a layer, plus the layer ends, and the host
// tables of ln(l + 1) and e^-P(L_i) that the RR kernel's count draws use.
//
// Built once per graph at stratify time, on the device:
//   1. every co-member occurrence (v, u) is written as the key u << b | v (b =
//      bits of a vertex id) at the incidences' channel prefixes, v's
//      incidences after those of smaller ids: ascending in the low half;
//   2. a stable device-wide radix sort by the high half alone (rocPRIM) leaves
//      the occurrences in order of both (they are symmetric: which half is
//      whose is not told apart any more, and the high one is called v);
//   3. a run of equal keys is a distinct pair (v, u), its length w(v, u).  Runs
//      of one key, most of them, are v's last layer and are in order already:
//      they go to their places, told by prefix sums;
//   4. the longer runs are sorted, stable, by v and descending w;
//   5. positions where that key changes are the other layers' ends.
// The passes over all occurrences bound it: sorting by both halves was five
// passes instead of three, and sorting all distinct pairs by 32 + b bits seven
// passes of 12 bytes: the sorts of a million vertices with 1.9e8 occurrences
// took 18.4 ms, 7.8 now, all of the tables 30 ms, 13 now.
// The buffers of 1-5 serve twice where one step's input is spent, and stay in
// the workspace up to kKeepBytes: allocating and freeing 15 GB per call took up
// to half a second (a million vertices, 1.9e8 occurrences).
// ln and e^-P are evaluated on the host with the C library's log and exp, so
// the device uses the same doubles as any host code that calls them.
#include <hip/hip_runtime.h>

#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>
#include <cmath>
#include <vector>

#include "dev_common.h"
#include "internal.h"

namespace hyperim {
namespace {

constexpr uint32_t kBlock = 256;

uint32_t grid_for(uint64_t items, uint32_t cap = 8192) {
    const uint64_t g = std::max<uint64_t>(div_up(items, kBlock), 1);
    return (uint32_t)std::min<uint64_t>(g, cap);
}

// Owner vertex of incidence e: the last v in [lo, hi) with v_off[v] <= e, given
// v_off[lo] <= e < v_off[hi].
__device__ __forceinline__ uint32_t owner(const uint32_t *__restrict__ v_off, uint32_t lo, uint32_t hi, uint64_t e) {
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (v_off[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

// 1. Occurrences: incidence e = (v, he) writes u << b | v for the members u of
// he other than v, at chan[e] ...  A wave takes 64 incidences, flattened over
// their members; bound by the writes.  (One thread per incidence, its members
// one after another and its owner searched among all vertices: 4.4 ms for 1.9e8
// occurrences, 1.2 now.)
__global__ __launch_bounds__(kBlock) void k_occ_emit(uint32_t n, uint64_t nnz, uint32_t b,
                                                      const uint32_t *__restrict__ v_off,
                                                      const uint4 *__restrict__ irec,
                                                      const uint32_t *__restrict__ he_mem,
                                                      const unsigned long long *__restrict__ chan,
                                                      unsigned long long *__restrict__ occ) {
    __shared__ uint32_t mark_s[kBlock / kWave][kWave], hb_s[kBlock / kWave][kWave], own_s[kBlock / kWave][kWave];
    const uint32_t lane = lane_id(), wv = uni(threadIdx.x / kWave);
    uint32_t *hb = hb_s[wv], *own = own_s[wv];
    const uint64_t waves = (uint64_t)gridDim.x * (kBlock / kWave);
    for (uint64_t e0 = ((uint64_t)blockIdx.x * (kBlock / kWave) + wv) * kWave; e0 < nnz; e0 += waves * kWave) {
        const uint64_t e = min(e0 + lane, nnz - 1u);
        // the owners of the ends first, the others between them
        const uint32_t end = lane < 2 ? owner(v_off, 0u, n, lane ? min(e0 + kWave, nnz) - 1u : e0) : 0u;
        const uint32_t v = owner(v_off, wave_bcast(end, 0), wave_bcast(end, 1) + 1u, e);
        uint4 rec = irec[e];
        if (e0 + lane >= nnz) rec.z = 0u;
        const uint32_t incl = wave_incl_scan(rec.z), total = wave_bcast(incl, kWave - 1);
        uint64_t at = chan[e0];
        wave_sync();
        hb[lane] = rec.y - (incl - rec.z);   // member q of the span is he_mem[hb + q]; may wrap
        own[lane] = v;
        for (uint32_t q0 = 0; q0 < total; q0 += kWave) {
            const uint32_t q = q0 + lane, k = window_owner(mark_s[wv], incl - rec.z, rec.z, q0);
            uint32_t u = 0, o = 0;
            if (q < total) {
                u = he_mem[hb[k] + q];   // the sum is taken in 32 bits
                o = own[k];
            }
            const uint64_t who = __ballot(u != o);   // never for lanes without a member
            if (u != o) occ[at + lane_rank(who)] = ((unsigned long long)u << b) | o;
            at += (uint64_t)__popcll(who);
        }
    }
}

// Tiles of kTile entries: kPer consecutive ones per thread.
constexpr uint32_t kPer = 8;
constexpr uint32_t kTile = kBlock * kPer;

// Exclusive prefix of this thread's count over the workgroup; *total: all of it.
__device__ __forceinline__ uint32_t block_prefix(uint32_t c, uint32_t *total) {
    __shared__ uint32_t part[kBlock / kWave];
    const uint32_t wv = threadIdx.x / kWave;
    const uint32_t incl = wave_incl_scan(c);
    if (lane_id() == kWave - 1) part[wv] = incl;
    __syncthreads();
    uint32_t before = incl - c, all = 0;
    for (uint32_t q = 0; q < kBlock / kWave; ++q) {
        if (q < wv) before += part[q];
        all += part[q];
    }
    *total = all;
    return before;
}

// The runs that begin at the sorted keys k[1 .. kPer] (k[0] and k[kPer + 1]:
// their neighbours), positions i0 ..: of one key (single) and longer.
__device__ __forceinline__ void run_heads(const unsigned long long (&k)[kPer + 2], uint64_t i0, uint64_t total,
                                          uint32_t *single, uint32_t *longer) {
    *single = *longer = 0u;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint64_t i = i0 + r;
        if (i >= total || (i != 0 && k[r + 1] == k[r])) continue;
        if (i + 1 < total && k[r + 2] == k[r + 1]) *longer |= 1u << r;
        else *single |= 1u << r;
    }
}
__device__ __forceinline__ void load_keys(const unsigned long long *__restrict__ key, uint64_t i0, uint64_t total,
                                          unsigned long long (&k)[kPer + 2]) {
    k[0] = i0 > 0 && i0 <= total ? key[i0 - 1] : 0ull;
#pragma unroll
    for (uint32_t r = 0; r <= kPer; ++r) k[r + 1] = i0 + r < total ? key[i0 + r] : 0ull;
}

// 3. Runs per tile: of one key, and longer ones (two halves of tile_cnt).
__global__ __launch_bounds__(kBlock) void k_head_count(uint64_t total, uint32_t tiles,
                                                        const unsigned long long *__restrict__ key,
                                                        uint32_t *__restrict__ tile_cnt) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 2];
    uint32_t single, longer, all;
    load_keys(key, i0, total, k);
    run_heads(k, i0, total, &single, &longer);
    (void)block_prefix((uint32_t)__popc(single) | ((uint32_t)__popc(longer) << 16), &all);   // at most kTile each
    if (threadIdx.x == 0) {
        tile_cnt[blockIdx.x] = all & 0xFFFFu;
        tile_cnt[tiles + blockIdx.x] = all >> 16;
    }
}

// Per vertex: runs of one key up to its end, longer runs before it and up to its end.
struct VertexRuns {
    uint32_t *s_end, *l_beg, *l_end;
};

// The longer runs' starts, in order, and each vertex's counts (written where
// the vertex of the keys changes).
__global__ __launch_bounds__(kBlock) void k_head_write(uint64_t total, uint32_t tiles, uint32_t b,
                                                        const unsigned long long *__restrict__ key,
                                                        const uint64_t *__restrict__ tile_off, VertexRuns vr,
                                                        uint32_t *__restrict__ run_start) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 2];
    uint32_t single, longer, all;
    load_keys(key, i0, total, k);
    run_heads(k, i0, total, &single, &longer);
    const uint32_t pre = block_prefix((uint32_t)__popc(single) | ((uint32_t)__popc(longer) << 16), &all);
    // offsets are prefixes over both halves: the second half's begin at all singles
    uint32_t s = (uint32_t)tile_off[blockIdx.x] + (pre & 0xFFFFu);
    uint32_t l = (uint32_t)(tile_off[tiles + blockIdx.x] - tile_off[tiles]) + (pre >> 16);
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint64_t i = i0 + r;
        if (i >= total) break;
        const uint32_t v = (uint32_t)(k[r + 1] >> b);
        if (i == 0 || (uint32_t)(k[r] >> b) != v) vr.l_beg[v] = l;
        s += (single >> r) & 1u;
        if ((longer >> r) & 1u) run_start[l++] = (uint32_t)i;
        if (i + 1 == total || (uint32_t)(k[r + 2] >> b) != v) {
            vr.s_end[v] = s;
            vr.l_end[v] = l;
        }
    }
}

// The runs of one key: the last of their vertex's co-members, in order.
__global__ __launch_bounds__(kBlock) void k_last_write(uint64_t total, uint32_t b,
                                                        const unsigned long long *__restrict__ key,
                                                        const uint64_t *__restrict__ tile_off, VertexRuns vr,
                                                        const unsigned long long *__restrict__ nb_off,
                                                        uint32_t *__restrict__ nb) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 2];
    uint32_t single, longer, all;
    load_keys(key, i0, total, k);
    run_heads(k, i0, total, &single, &longer);
    uint32_t s = (uint32_t)tile_off[blockIdx.x] + block_prefix((uint32_t)__popc(single), &all);
    const unsigned long long umask = (1ull << b) - 1ull;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if ((single >> r) & 1u) {
            const uint32_t v = (uint32_t)(k[r + 1] >> b);
            nb[nb_off[v + 1] - (vr.s_end[v] - s)] = (uint32_t)(k[r + 1] & umask);
            ++s;
        }
}

// 4. Sort keys of the longer runs: v << wb | (2^wb - 1 - w), ascending v and
// descending w (w < 2^wb); the value is u.  A run's end is found by doubling
// steps from its start, then halving them: most are two or three keys long.
__global__ __launch_bounds__(kBlock) void k_wkeys(uint64_t runs, uint64_t total, uint32_t b, uint32_t wb,
                                                   const unsigned long long *__restrict__ key,
                                                   const uint32_t *__restrict__ run_start,
                                                   unsigned long long *__restrict__ key2, uint32_t *__restrict__ val) {
    const unsigned long long umask = (1ull << b) - 1ull, wmask = (1ull << wb) - 1ull;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < runs; k += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = run_start[k];
        const unsigned long long me = key[i];
        uint64_t w = 2, step = 1;   // key[i .. i + w) is in the run
        while (i + w + step - 1 < total && key[i + w + step - 1] == me) {
            w += step;
            step *= 2;
        }
        for (; step; step /= 2)
            if (i + w + step - 1 < total && key[i + w + step - 1] == me) w += step;
        key2[k] = ((me >> b) << wb) | (wmask - w);
        val[k] = (uint32_t)(me & umask);
    }
}

// The sorted longer runs' co-members: the first of their vertex.
__global__ __launch_bounds__(kBlock) void k_first_write(uint64_t runs, uint32_t wb,
                                                         const unsigned long long *__restrict__ key2,
                                                         const uint32_t *__restrict__ val, VertexRuns vr,
                                                         const unsigned long long *__restrict__ nb_off,
                                                         uint32_t *__restrict__ nb) {
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < runs; k += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t v = (uint32_t)(key2[k] >> wb);
        nb[nb_off[v] + (k - vr.l_beg[v])] = val[k];
    }
}

// Vertices with a layer of runs of one key (w = 1): 1 each, and its end.
__global__ __launch_bounds__(kBlock) void k_last_layer(uint32_t n, const uint32_t *__restrict__ deg,
                                                        const uint32_t *__restrict__ l, VertexRuns vr,
                                                        const unsigned long long *__restrict__ ly_off,
                                                        uint32_t *__restrict__ has, uint32_t *__restrict__ ly_end) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    const uint32_t d = deg[v];
    const bool last = d != 0u && vr.l_end[v] - vr.l_beg[v] != d;
    has[v] = last ? 1u : 0u;
    if (last) ly_end[ly_off[v] + l[v] - 1u] = d;
}

// 5. The other layers' ends: sorted run k ends a layer when the next key
// differs (another weight or another vertex) or k is the last one.  Counted per
// tile, then written, after the layers of w = 1 of the vertices before (last_off).
__global__ __launch_bounds__(kBlock) void k_end_count(uint64_t runs, const unsigned long long *__restrict__ key2,
                                                       uint32_t *__restrict__ tile_cnt) {
    const uint64_t k0 = (uint64_t)blockIdx.x * kTile;
    uint32_t c = 0, all;
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint64_t k = k0 + r * kBlock + threadIdx.x;
        c += k < runs && (k + 1 == runs || key2[k + 1] != key2[k]) ? 1u : 0u;
    }
    (void)block_prefix(c, &all);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = all;
}

__global__ __launch_bounds__(kBlock) void k_end_write(uint64_t runs, uint32_t wb,
                                                       const unsigned long long *__restrict__ key2,
                                                       const uint64_t *__restrict__ tile_off, VertexRuns vr,
                                                       const uint64_t *__restrict__ last_off,
                                                       uint32_t *__restrict__ ly_end) {
    const uint64_t k0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 1];
    uint32_t ends = 0, all;
#pragma unroll
    for (uint32_t r = 0; r <= kPer; ++r) k[r] = k0 + r < runs ? key2[k0 + r] : ~0ull;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if (k0 + r < runs && (k0 + r + 1 == runs || k[r + 1] != k[r])) ends |= 1u << r;
    uint64_t at = block_prefix((uint32_t)__popc(ends), &all);
    at += tile_off[blockIdx.x];
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if ((ends >> r) & 1u) {
            const uint32_t v = (uint32_t)(k[r] >> wb);
            ly_end[last_off[v] + at++] = (uint32_t)(k0 + r + 1) - vr.l_beg[v];
        }
}

constexpr size_t kKeepBytes = 8ull << 30;   // scratch kept between calls

}  // namespace

int layers_build_device(hyperim_graph g, PrepWorkspace &w, uint32_t lmax, hipStream_t s) {
    const uint32_t n = g->n;
    const uint64_t nnz = g->nnz;
    // occurrences: sum over v of c(v)
    uint64_t total = 0;
    HIM_HIP(hipMemcpyAsync(&total, g->chan.as<unsigned long long>() + nnz, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    HIM_HIP(hipStreamSynchronize(s));
    const uint64_t uniq = g->info.sum_deg, nlay = g->info.sum_l;
    if (total >= (1ull << 32) || lmax > 16384u) {
        set_error_detail("stratified-setting tables: more than 2^32 co-member occurrences or 16384 layers");
        return HYPERIM_EINVAL;
    }
    // scratch beyond kKeepBytes goes back when the call ends
    struct Scratch {
        PrepWorkspace &w;
        hipStream_t s;
        DevBuf *all[5] = {&w.occ, &w.occ2, &w.sort_tmp, &w.run_start, &w.pair_val};
        ~Scratch() {
            size_t b = 0;
            for (const DevBuf *x : all) b += x->bytes;
            if (b <= kKeepBytes) return;
            (void)hipStreamSynchronize(s);
            for (DevBuf *x : all) x->release();
        }
    } scratch{w, s};
    const uint32_t b = n > 1 ? 32u - (uint32_t)__builtin_clz(n - 1u) : 1u;   // bits of a vertex id
    const uint32_t wb = 32u - (uint32_t)__builtin_clz(std::max(g->m, 1u));         // bits of a weight (at most m)
    const uint64_t total1 = std::max<uint64_t>(total, 1), uniq1 = std::max<uint64_t>(uniq, 1);
    const uint64_t runs1 = std::max<uint64_t>(std::min(uniq, total / 2), 1);       // longer runs, at most
    HIM_CHECK(w.occ.reserve(sizeof(uint64_t) * total1, s));
    HIM_CHECK(w.occ2.reserve(sizeof(uint64_t) * total1, s));
    HIM_CHECK(w.run_start.reserve(sizeof(uint32_t) * runs1, s));
    HIM_CHECK(w.pair_val.reserve(2 * sizeof(uint32_t) * runs1, s));
    HIM_CHECK(w.vals.reserve(4 * sizeof(uint32_t) * (size_t)n, s));
    HIM_CHECK(w.base.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    const uint32_t tiles = (uint32_t)std::max<uint64_t>(div_up(total, kTile), 1);
    HIM_CHECK(w.k1.reserve(2 * sizeof(uint32_t) * (size_t)tiles, s));
    HIM_CHECK(w.k2.reserve(sizeof(uint64_t) * (2 * (size_t)tiles + 1), s));
    uint32_t *tile_cnt = w.k1.as<uint32_t>();
    uint64_t *tile_off = w.k2.as<uint64_t>();
    uint32_t *per_v = w.vals.as<uint32_t>(), *has_last = per_v + 3 * (size_t)n;
    const VertexRuns vr{per_v, per_v + n, per_v + 2 * (size_t)n};
    using Key = unsigned long long;
    // 1., 2. all occurrences by (v, u)
    rocprim::double_buffer<Key> keys(w.occ.as<Key>(), w.occ2.as<Key>());
    uint64_t found[2] = {0, 0};   // runs of one key; all runs
    if (total) {
        hipLaunchKernelGGL(k_occ_emit, dim3(grid_for(nnz, 2048)), dim3(kBlock), 0, s, n, nnz, b,
                           g->v_off.as<uint32_t>(), g->irec.as<uint4>(), g->he_mem.as<uint32_t>(), g->chan.as<Key>(),
                           keys.current());
        HIM_HIP(hipGetLastError());
        size_t tbytes = 0;
        HIM_HIP(rocprim::radix_sort_keys(nullptr, tbytes, keys, (size_t)total, b, 2u * b, s));
        HIM_CHECK(w.sort_tmp.reserve(std::max<size_t>(tbytes, 1), s));
        HIM_HIP(rocprim::radix_sort_keys(w.sort_tmp.ptr, tbytes, keys, (size_t)total, b, 2u * b, s));
        // 3. runs
        hipLaunchKernelGGL(k_head_count, dim3(tiles), dim3(kBlock), 0, s, total, tiles, keys.current(), tile_cnt);
        HIM_CHECK(scan_u32_to_u64(tile_cnt, tile_off, 2 * (uint64_t)tiles, 0, w.tmp, s));
        HIM_HIP(hipMemcpyAsync(found, tile_off + tiles, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        HIM_HIP(hipMemcpyAsync(found + 1, tile_off + 2 * (size_t)tiles, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        HIM_HIP(hipStreamSynchronize(s));
    }
    if (found[1] != uniq) {
        set_error_detail("stratified-setting tables: distinct co-members disagree with deg");
        return HYPERIM_EHIP;
    }
    const uint64_t runs = found[1] - found[0];
    // per-vertex ranges of the distinct co-members (deg prefix) and of the
    // layers (l prefix)
    HIM_CHECK(g->lay_nb.reserve(sizeof(uint32_t) * uniq1, s));
    HIM_CHECK(g->lay_nb_off.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(g->lay_ly_off.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(scan_u32_to_u64(g->deg.as<uint32_t>(), g->lay_nb_off.as<uint64_t>(), n, 0, w.tmp, s));
    HIM_CHECK(scan_u32_to_u64(g->l.as<uint32_t>(), g->lay_ly_off.as<uint64_t>(), n, 0, w.tmp, s));
    HIM_CHECK(g->lay_ly_end.reserve(sizeof(uint32_t) * std::max<uint64_t>(nlay, 1), s));
    if (total) {
        const Key *nb_off = g->lay_nb_off.as<Key>();
        uint32_t *nb = g->lay_nb.as<uint32_t>();
        hipLaunchKernelGGL(k_head_write, dim3(tiles), dim3(kBlock), 0, s, total, tiles, b, keys.current(), tile_off,
                           vr, w.run_start.as<uint32_t>());
        hipLaunchKernelGGL(k_last_write, dim3(tiles), dim3(kBlock), 0, s, total, b, keys.current(), tile_off, vr,
                           nb_off, nb);
        hipLaunchKernelGGL(k_last_layer, dim3((uint32_t)div_up(n, kBlock)), dim3(kBlock), 0, s, n,
                           g->deg.as<uint32_t>(), g->l.as<uint32_t>(), vr, g->lay_ly_off.as<Key>(), has_last,
                           g->lay_ly_end.as<uint32_t>());
        HIM_CHECK(scan_u32_to_u64(has_last, w.base.as<uint64_t>(), n, 0, w.tmp, s));
        if (runs) {
            // 4. the longer runs by v and descending w, in the spent key buffer's
            // halves (at most total / 2 runs); values u
            uint32_t *val = w.pair_val.as<uint32_t>();
            hipLaunchKernelGGL(k_wkeys, dim3(grid_for(runs)), dim3(kBlock), 0, s, runs, total, b, wb, keys.current(),
                               w.run_start.as<uint32_t>(), keys.alternate(), val);
            rocprim::double_buffer<Key> wkeys(keys.alternate(), keys.alternate() + total / 2);
            rocprim::double_buffer<uint32_t> vals(val, val + runs1);
            size_t tbytes = 0;
            HIM_HIP(rocprim::radix_sort_pairs(nullptr, tbytes, wkeys, vals, (size_t)runs, 0u, wb + b, s));
            HIM_CHECK(w.sort_tmp.reserve(std::max<size_t>(tbytes, 1), s));
            HIM_HIP(rocprim::radix_sort_pairs(w.sort_tmp.ptr, tbytes, wkeys, vals, (size_t)runs, 0u, wb + b, s));
            hipLaunchKernelGGL(k_first_write, dim3(grid_for(runs)), dim3(kBlock), 0, s, runs, wb, wkeys.current(),
                               vals.current(), vr, nb_off, nb);
            // 5. their layers' ends
            const uint32_t rtiles = (uint32_t)div_up(runs, kTile);
            hipLaunchKernelGGL(k_end_count, dim3(rtiles), dim3(kBlock), 0, s, runs, wkeys.current(), tile_cnt);
            HIM_CHECK(scan_u32_to_u64(tile_cnt, tile_off, rtiles, 0, w.tmp, s));
            hipLaunchKernelGGL(k_end_write, dim3(rtiles), dim3(kBlock), 0, s, runs, wb, wkeys.current(), tile_off, vr,
                               w.base.as<uint64_t>(), g->lay_ly_end.as<uint32_t>());
        }
    }
    HIM_HIP(hipGetLastError());
    // host tables: ln(l + 1) for l <= lmax, and e^-P(L_i) with
    // P(L_i) = 1 / (i ln(l + 1)) at index l (l - 1) / 2 + i - 1
    std::vector<double> ln((size_t)lmax + 1), expm(std::max<size_t>((size_t)lmax * (lmax + 1) / 2, 1));
    for (uint32_t l = 0; l <= lmax; ++l) ln[l] = std::log((double)l + 1.0);
    for (uint32_t l = 1; l <= lmax; ++l)
        for (uint32_t i = 1; i <= l; ++i) {
            const double P = 1.0 / ((double)i * std::log((double)l + 1.0));
            expm[(size_t)l * (l - 1) / 2 + i - 1] = std::exp(-P);
        }
    HIM_CHECK(g->lay_ln.reserve(sizeof(double) * ln.size(), s));
    HIM_CHECK(g->lay_expm.reserve(sizeof(double) * expm.size(), s));
    HIM_HIP(hipMemcpyAsync(g->lay_ln.ptr, ln.data(), sizeof(double) * ln.size(), hipMemcpyHostToDevice, s));
    HIM_HIP(hipMemcpyAsync(g->lay_expm.ptr, expm.data(), sizeof(double) * expm.size(), hipMemcpyHostToDevice, s));
    HIM_HIP(hipStreamSynchronize(s));   // ln and expm are the copies' sources
    g->lay_lmax = lmax;
    g->lay_ready = true;
    return HYPERIM_OK;
}

}  // namespace hyperim
