// Device-side building blocks shared by the gfx950 kernels of libhyperim:
// the counter-based Philox4x32-10 generator (Salmon et al., SC'11) used for
// every coin and root offset, the channel-coin keying, and 64-lane wavefront
// primitives (scan, ballot ranks, broadcasts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hyperim {

constexpr int kWave = 64;                 // CDNA wavefront width
constexpr uint32_t kAlways = 0xFFFFFFFFu; // threshold meaning "channel always live"
constexpr uint32_t kNStrata = 8;

// a ^ b ^ c: one v_bitop3_b32 (truth table 0x96) on the device, where the
// compiler would issue two v_xor_b32.
__host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
    return a ^ b ^ c;
#endif
}

// Philox4x32-10 block function: ten S-P rounds over a 128-bit counter, the
// 64-bit key advanced by the Weyl increments between rounds.  Each round
// multiplies counter words 0 and 2 by the Philox constants, keeps both halves
// of the 64-bit products and mixes the high halves with the other words and
// the key.  VALU-bound: 20 v_mad_u64_u32 and 20 three-input xors per block
// with the key schedule in scalar registers, 845 Gblocks/s on MI355X at full
// occupancy (two-input xors: 40 of them, 661-695 Gblocks/s).
constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;   // multipliers of words 0 and 2
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;   // key increments

// Rounds kFirst .. 9 on the state before round kFirst; key: that of round 0.
template <int kFirst>
__host__ __device__ __forceinline__ uint4 philox_rounds(uint4 ctr, uint2 key) {
    key.x += (uint32_t)kFirst * kPhiloxW0;
    key.y += (uint32_t)kFirst * kPhiloxW1;
#pragma unroll
    for (int round = kFirst; round < 10; ++round) {
        const uint64_t m0 = (uint64_t)kPhiloxM0 * (uint64_t)ctr.x;
        const uint64_t m2 = (uint64_t)kPhiloxM1 * (uint64_t)ctr.z;
        uint4 next;
        next.x = xor3((uint32_t)(m2 >> 32), ctr.y, key.x);
        next.y = (uint32_t)m2;
        next.z = xor3((uint32_t)(m0 >> 32), ctr.w, key.y);
        next.w = (uint32_t)m0;
        ctr = next;
        key.x += kPhiloxW0;
        key.y += kPhiloxW1;
    }
    return ctr;
}

__host__ __device__ __forceinline__ uint4 philox4x32_10(uint4 ctr, uint2 key) { return philox_rounds<0>(ctr, key); }

// Counter of the four coins of channels (he, u -> v) in RR set j whose
// source positions pos in he satisfy pos >> 2 == quad.  Word (pos & 3) of the
// block is the coin; pool tag in bit 31, bits 32..38 of j in bits 24..30.
__host__ __device__ __forceinline__ uint4 coin_counter(uint64_t j, uint32_t he, uint32_t v,
                                                       uint32_t pool, uint32_t quad) {
    return make_uint4((uint32_t)j, he, v, (pool << 31) | ((uint32_t)(j >> 32) << 24) | quad);
}

// Counter of the random offset of ladder block b of a pool (he and v words
// hold ids no hyperedge or vertex can take).
__host__ __device__ __forceinline__ uint4 root_counter(uint32_t b, uint32_t pool) {
    return make_uint4(b, 0xFFFFFFFFu, 0xFFFFFFFFu, pool);
}

__device__ __forceinline__ bool channel_live(uint32_t coin, uint32_t thr) {
    return thr == kAlways || coin < thr;
}

// ---- wavefront primitives --------------------------------------------------
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ uint32_t lane_rank(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Scans and reductions move values between lanes with DPP, inside the vector
// ALU: four shifts within rows of 16 lanes, then lane 15 of each row to the
// next row and lane 31 to the upper half.  (A shuffle is an LDS access of
// about 60 cycles, and a scan is a chain of six: with shuffles a range of 777
// small RR sets took 1.32 ms, with DPP 1.15 ms.)  Every lane of the wave must
// be active.  `idle` stands in for a lane without a source.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_move(uint32_t idle, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)idle, (int)x, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows, typename T>
__device__ __forceinline__ T dpp_from(T x) {   // idle = 0
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit values");
    if constexpr (sizeof(T) == 4) {
        return (T)dpp_move<kCtrl, kRows>(0u, (uint32_t)x);
    } else {
        const uint32_t lo = dpp_move<kCtrl, kRows>(0u, (uint32_t)(uint64_t)x);
        const uint32_t hi = dpp_move<kCtrl, kRows>(0u, (uint32_t)((uint64_t)x >> 32));
        return (T)(((uint64_t)hi << 32) | lo);
    }
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;   // rows 1 and 3 / rows 2 and 3 receive

// The inclusive scan of x under `op` (identity 0: unsigned sums, maxima, ors).
template <typename T, typename Op>
__device__ __forceinline__ T wave_scan_op(T x, Op op) {
    x = op(x, dpp_from<kRowShr1, 0xf>(x));
    x = op(x, dpp_from<kRowShr2, 0xf>(x));
    x = op(x, dpp_from<kRowShr4, 0xf>(x));
    x = op(x, dpp_from<kRowShr8, 0xf>(x));
    x = op(x, dpp_from<kRowBcast15, 0xa>(x));
    x = op(x, dpp_from<kRowBcast31, 0xc>(x));
    return x;
}

// The value of lane `src` (the same on every lane) as a scalar.
__device__ __forceinline__ uint32_t wave_bcast(uint32_t x, int src) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, src);
}
__device__ __forceinline__ uint64_t wave_bcast64(uint64_t x, int src) {
    return ((uint64_t)wave_bcast((uint32_t)(x >> 32), src) << 32) | (uint64_t)wave_bcast((uint32_t)x, src);
}

template <typename T>
__device__ __forceinline__ T wave_last(T x) {
    if constexpr (sizeof(T) == 4) return (T)wave_bcast((uint32_t)x, kWave - 1);
    else return (T)wave_bcast64((uint64_t)x, kWave - 1);
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T x) {
    return wave_scan_op(x, [](T a, T b) { return (T)(a + b); });
}

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
    return wave_last(wave_incl_scan(x));
}

template <typename T>
__device__ __forceinline__ T wave_max(T x) {
    return wave_last(wave_scan_op(x, [](T a, T b) { return a > b ? a : b; }));
}

// Wave-uniform values kept in scalar registers: the value of the first active
// lane (callers pass values that are equal on every active lane).
__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
    return ((uint64_t)uni((uint32_t)(x >> 32)) << 32) | (uint64_t)uni((uint32_t)x);
}
template <typename P>
__device__ __forceinline__ P uni_ptr(P p) {
    return (P)uni64((uint64_t)p);
}

// Make this wave's earlier LDS and global writes visible to its own later
// reads by other lanes, and keep the compiler from moving memory accesses
// across the point.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Smallest k in [0, 64) with scan[k] > g, for a 64-entry nondecreasing array
// whose last entry exceeds g.
__device__ __forceinline__ uint32_t search64(const uint32_t *scan, uint32_t g) {
    uint32_t k = 0;
#pragma unroll
    for (uint32_t s = 32; s > 0; s >>= 1)
        if (scan[k + s - 1] <= g) k += s;
    return k;
}

// Lanes own consecutive runs of slots (lane k: [start, start + count), starts
// ascending).  For the window of slots base .. base + 63 this gives each lane
// the owner of slot base + lane (a slot that somebody owns; else any lane): the
// owners that begin inside the window leave their lane number at their first
// slot, a running maximum over the lanes carries it on.  Three LDS accesses in a
// row and six DPP moves, where a binary search over the starts was a chain of
// six LDS reads.  Every lane of the wave calls it.
__device__ __forceinline__ uint32_t window_owner(uint32_t *mark, uint32_t start, uint32_t count, uint32_t base) {
    const uint32_t lane = lane_id();
    const uint64_t first = __ballot(start <= base && base - start < count);   // owner of slot base
    const uint32_t rel = start - base;                                        // wraps for earlier starts
    mark[lane] = 0u;
    wave_sync();
    if (count != 0u && start >= base && rel < kWave) mark[rel] = lane + 1u;
    wave_sync();
    uint32_t x = mark[lane];
    x = wave_scan_op(x, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
    return x ? x - 1u : (uint32_t)__ffsll((unsigned long long)first) - 1u;
}

__host__ __device__ __forceinline__ uint64_t div_up(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

}  // namespace hyperim
