// Sample-set division (Section 3.1.1) as tables, for the stratified-setting
// model: per vertex v the members of A(v) layer by layer (layer 1 = largest
// w(v,u)), ascending ids within a layer, plus the layer ends, and the host
// tables of ln(l + 1) and e^-P(L_i) that the RR kernel's count draws use.
//
// Built once per graph at stratify time, on the device:
//   1. every co-member occurrence (v, u) of incidence e is written, as the
//      key v << b | u (b = bits of a vertex id), at the incidence's channel
//      prefix chan[e] (the graph's exclusive prefix of |he| - 1 over v_he);
//   2. a device-wide radix sort orders the keys (rocPRIM), so each vertex's
//      occurrences are contiguous and ascending in u;
//   3. run heads give the distinct pairs (v, u) and their run lengths w(v,u)
//      (heads are counted per tile, then written at the tiles' offsets: two
//      reads of the keys and no per-key flag or offset);
//   4. a second, stable radix sort by the key v << 32 | ~w puts each vertex's
//      co-members in layers (descending w; equal w keep ascending u);
//   5. positions where the key changes are the layer ends.
// The buffers of 1-5 serve twice where one step's input is spent, and stay in
// the workspace up to kKeepBytes: allocating and freeing 15 GB per call took up
// to half a second (a million vertices, 3.4e8 occurrences).
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

// Owner vertex of incidence e: the last v with v_off[v] <= e.
__device__ __forceinline__ uint32_t owner(const uint32_t *__restrict__ v_off, uint32_t n, uint64_t e) {
    uint32_t lo = 0, hi = n;   // v_off[lo] <= e < v_off[hi]
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (v_off[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

// 1. Occurrences: incidence e = (v, he) writes v << b | u for the members u
// of he other than v at chan[e] ...
__global__ void k_occ_emit(uint32_t n, uint64_t nnz, uint32_t b, const uint32_t *__restrict__ v_off,
                           const uint32_t *__restrict__ v_he, const uint32_t *__restrict__ he_off,
                           const uint32_t *__restrict__ he_mem, const unsigned long long *__restrict__ chan,
                           unsigned long long *__restrict__ occ) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t v = owner(v_off, n, e), he = v_he[e];
        uint64_t at = chan[e];
        for (uint32_t i = he_off[he]; i < he_off[he + 1]; ++i) {
            const uint32_t u = he_mem[i];
            if (u != v) occ[at++] = ((unsigned long long)v << b) | u;
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

// 3. Run heads of the sorted keys: their count per tile.
__global__ __launch_bounds__(kBlock) void k_head_count(uint64_t total, const unsigned long long *__restrict__ key,
                                                        uint32_t *__restrict__ tile_cnt) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kTile;
    uint32_t c = 0, all;
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint64_t i = i0 + r * kBlock + threadIdx.x;
        c += i < total && (i == 0 || key[i] != key[i - 1]) ? 1u : 0u;
    }
    (void)block_prefix(c, &all);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = all;
}

// Distinct pair k (at run head i): its key and its run's start.
__global__ __launch_bounds__(kBlock) void k_head_write(uint64_t total, const unsigned long long *__restrict__ key,
                                                        const uint64_t *__restrict__ tile_off,
                                                        unsigned long long *__restrict__ ukey,
                                                        uint32_t *__restrict__ run_start) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 1];
    k[0] = i0 > 0 && i0 <= total ? key[i0 - 1] : 0ull;
    uint32_t heads = 0, all;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        k[r + 1] = i0 + r < total ? key[i0 + r] : k[r];
        if (i0 + r < total && (i0 + r == 0 || k[r + 1] != k[r])) heads |= 1u << r;
    }
    uint64_t at = block_prefix((uint32_t)__popc(heads), &all);
    at += tile_off[blockIdx.x];
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if ((heads >> r) & 1u) {
            ukey[at] = k[r + 1];
            run_start[at] = (uint32_t)(i0 + r);
            ++at;
        }
}

// Layer sort key of distinct pair k: v << 32 | ~w (ascending keys: v, then
// descending w); the value is u.
__global__ void k_wkeys(uint64_t uniq, uint64_t total, uint32_t b, const unsigned long long *__restrict__ ukey,
                        const uint32_t *__restrict__ run_start, unsigned long long *__restrict__ key2,
                        uint32_t *__restrict__ val) {
    const unsigned long long umask = (1ull << b) - 1ull;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < uniq; k += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t end = k + 1 < uniq ? run_start[k + 1] : (uint32_t)total;
        const uint32_t w = end - run_start[k];
        const unsigned long long v = ukey[k] >> b;
        key2[k] = (v << 32) | (unsigned long long)(~w);
        val[k] = (uint32_t)(ukey[k] & umask);
    }
}

// 5. Layer ends: entry k ends a layer when the next key differs (another
// weight or another vertex) or k is the last entry.  Counted per tile, then
// written.
__global__ __launch_bounds__(kBlock) void k_end_count(uint64_t uniq, const unsigned long long *__restrict__ key2,
                                                       uint32_t *__restrict__ tile_cnt) {
    const uint64_t k0 = (uint64_t)blockIdx.x * kTile;
    uint32_t c = 0, all;
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint64_t k = k0 + r * kBlock + threadIdx.x;
        c += k < uniq && (k + 1 == uniq || key2[k + 1] != key2[k]) ? 1u : 0u;
    }
    (void)block_prefix(c, &all);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = all;
}

__global__ __launch_bounds__(kBlock) void k_end_write(uint64_t uniq, const unsigned long long *__restrict__ key2,
                                                       const uint64_t *__restrict__ tile_off,
                                                       const unsigned long long *__restrict__ nb_off,
                                                       uint32_t *__restrict__ ly_end) {
    const uint64_t k0 = (uint64_t)blockIdx.x * kTile + threadIdx.x * kPer;
    unsigned long long k[kPer + 1];
    uint32_t ends = 0, all;
#pragma unroll
    for (uint32_t r = 0; r <= kPer; ++r) k[r] = k0 + r < uniq ? key2[k0 + r] : ~0ull;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if (k0 + r < uniq && (k0 + r + 1 == uniq || k[r + 1] != k[r])) ends |= 1u << r;
    uint64_t at = block_prefix((uint32_t)__popc(ends), &all);
    at += tile_off[blockIdx.x];
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r)
        if ((ends >> r) & 1u) ly_end[at++] = (uint32_t)(k0 + r + 1 - nb_off[(uint32_t)(k[r] >> 32)]);
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
    const uint64_t total1 = std::max<uint64_t>(total, 1), uniq1 = std::max<uint64_t>(uniq, 1);
    HIM_CHECK(w.occ.reserve(sizeof(uint64_t) * total1, s));
    HIM_CHECK(w.occ2.reserve(sizeof(uint64_t) * total1, s));
    HIM_CHECK(w.run_start.reserve(sizeof(uint32_t) * uniq1, s));
    HIM_CHECK(w.pair_val.reserve(2 * sizeof(uint32_t) * uniq1, s));
    const uint32_t tiles = (uint32_t)std::max<uint64_t>(div_up(total, kTile), 1);
    HIM_CHECK(w.k1.reserve(sizeof(uint32_t) * tiles, s));
    HIM_CHECK(w.k2.reserve(sizeof(uint64_t) * ((size_t)tiles + 1), s));
    uint32_t *tile_cnt = w.k1.as<uint32_t>();
    uint64_t *tile_off = w.k2.as<uint64_t>();
    using Key = unsigned long long;
    // 1., 2. all occurrences by (v, u)
    rocprim::double_buffer<Key> keys(w.occ.as<Key>(), w.occ2.as<Key>());
    if (total) {
        hipLaunchKernelGGL(k_occ_emit, dim3(grid_for(nnz)), dim3(kBlock), 0, s, n, nnz, b, g->v_off.as<uint32_t>(),
                           g->v_he.as<uint32_t>(), g->he_off.as<uint32_t>(), g->he_mem.as<uint32_t>(),
                           g->chan.as<Key>(), keys.current());
        HIM_HIP(hipGetLastError());
        size_t tbytes = 0;
        HIM_HIP(rocprim::radix_sort_keys(nullptr, tbytes, keys, (size_t)total, 0u, 2u * b, s));
        HIM_CHECK(w.sort_tmp.reserve(std::max<size_t>(tbytes, 1), s));
        HIM_HIP(rocprim::radix_sort_keys(w.sort_tmp.ptr, tbytes, keys, (size_t)total, 0u, 2u * b, s));
    }
    // 3. distinct pairs and their weights, into the other key buffer
    uint64_t uniq_dev = 0;
    if (total) {
        hipLaunchKernelGGL(k_head_count, dim3(tiles), dim3(kBlock), 0, s, total, keys.current(), tile_cnt);
        HIM_CHECK(scan_u32_to_u64(tile_cnt, tile_off, tiles, 0, w.tmp, s));
        HIM_HIP(hipMemcpyAsync(&uniq_dev, tile_off + tiles, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        HIM_HIP(hipStreamSynchronize(s));
    }
    if (uniq_dev != uniq) {
        set_error_detail("stratified-setting tables: distinct co-members disagree with deg");
        return HYPERIM_EHIP;
    }
    Key *ukey = keys.alternate(), *key2 = keys.current();   // the sorted occurrences are spent after k_head_write
    uint32_t *val = w.pair_val.as<uint32_t>(), *val2 = val + uniq1;
    if (total) {
        hipLaunchKernelGGL(k_head_write, dim3(tiles), dim3(kBlock), 0, s, total, keys.current(), tile_off, ukey,
                           w.run_start.as<uint32_t>());
        hipLaunchKernelGGL(k_wkeys, dim3(grid_for(uniq)), dim3(kBlock), 0, s, uniq, total, b, ukey,
                           w.run_start.as<uint32_t>(), key2, val);
    }
    // per-vertex ranges of the distinct co-members (deg prefix) and of the
    // layers (l prefix)
    HIM_CHECK(g->lay_nb.reserve(sizeof(uint32_t) * uniq1, s));
    HIM_CHECK(g->lay_nb_off.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(g->lay_ly_off.reserve(sizeof(uint64_t) * ((size_t)n + 1), s));
    HIM_CHECK(scan_u32_to_u64(g->deg.as<uint32_t>(), g->lay_nb_off.as<uint64_t>(), n, 0, w.tmp, s));
    HIM_CHECK(scan_u32_to_u64(g->l.as<uint32_t>(), g->lay_ly_off.as<uint64_t>(), n, 0, w.tmp, s));
    HIM_CHECK(g->lay_ly_end.reserve(sizeof(uint32_t) * std::max<uint64_t>(nlay, 1), s));
    if (uniq) {
        // 4. layers: stable sort of the distinct pairs by v << 32 | ~w, values u
        rocprim::double_buffer<Key> wkeys(key2, ukey);
        rocprim::double_buffer<uint32_t> vals(val, val2);
        size_t tbytes = 0;
        HIM_HIP(rocprim::radix_sort_pairs(nullptr, tbytes, wkeys, vals, (size_t)uniq, 0u, 32u + b, s));
        HIM_CHECK(w.sort_tmp.reserve(std::max<size_t>(tbytes, 1), s));
        HIM_HIP(rocprim::radix_sort_pairs(w.sort_tmp.ptr, tbytes, wkeys, vals, (size_t)uniq, 0u, 32u + b, s));
        HIM_HIP(hipMemcpyAsync(g->lay_nb.ptr, vals.current(), sizeof(uint32_t) * uniq, hipMemcpyDeviceToDevice, s));
        // 5. layer ends
        const uint32_t utiles = (uint32_t)div_up(uniq, kTile);
        hipLaunchKernelGGL(k_end_count, dim3(utiles), dim3(kBlock), 0, s, uniq, wkeys.current(), tile_cnt);
        HIM_CHECK(scan_u32_to_u64(tile_cnt, tile_off, utiles, 0, w.tmp, s));
        hipLaunchKernelGGL(k_end_write, dim3(utiles), dim3(kBlock), 0, s, uniq, wkeys.current(), tile_off,
                           g->lay_nb_off.as<Key>(), g->lay_ly_end.as<uint32_t>());
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
    return HYPERIM_OK;
}

}  // namespace hyperim
