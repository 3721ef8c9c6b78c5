// Host models of a planning wave of the grid-wide RR-generation phase and of
// the progress rules of the host loops, for the CPU tests.  They run the layout
// arithmetic and the rules of plan_layout.h, as the device planners k_plan and
// k_ms_plan do, over plain arrays instead of wave registers: chunk lengths by
// incidences and members, per-lane heavy splits, light segments, one reservation
// for several batches, what happens when the items do not fit, and the owner
// search that spreads a batch's heavy chunks over the wave.  Nothing here runs
// on the device or in the generation path.
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "internal.h"
#include "plan_layout.h"

using namespace hyperim;

// One batch.  mode 0: per-set planner (entries may be marked expanded; a batch
// whose items exceed item_cap plans its first entry alone), of entries whose
// hyperedges hold few members; mode 1: bundled planner (entry weights are
// incidences times sets).
// Lanes [0, nb) carry deg[l], e0[l], sets[l] (mode 1) and expanded[l]
// (mode 0).  Items go to items[4 * i ..] as (lane, count, 0, 0) for a light
// segment starting at `lane` and (lane | 1 << 31, lo, hi, 0) for a heavy
// chunk of lane's incidences [lo, hi); *n_items receives the batch's
// reservation, *taken the entries the batch consumes.  Returns 0, or -1 when
// an argument is out of range or `items` holds fewer than cap_out items.
extern "C" int hyperim_model_plan_batch(uint32_t mode, uint32_t nb, const uint32_t *deg, const uint32_t *e0,
                                        const uint32_t *sets, const uint8_t *expanded, uint32_t chunk, uint32_t seg,
                                        uint32_t item_cap, uint32_t *items, uint32_t cap_out, uint32_t *n_items,
                                        uint32_t *taken) {
    constexpr uint32_t W = 64;
    if (mode > 1 || nb == 0 || nb > W || !deg || !e0 || !items || !n_items || !taken || chunk == 0 || seg == 0 ||
        (mode == 1 && !sets))
        return -1;
    seg = seg > chunk ? seg : chunk;   // as the library sets it
    uint32_t hv[W] = {0}, len[W] = {0}, light[W] = {0};
    bool live[W] = {false};
    bool any = false;
    for (uint32_t l = 0; l < nb; ++l) {
        live[l] = mode == 1 || !expanded || !expanded[l];
        if (!live[l]) continue;
        any = true;
        const HeavySplit h = mode == 0 ? heavy_split(deg[l], weighted_chunk(deg[l], 0u, chunk))
                                       : ms_heavy_split(deg[l], sets[l], chunk);
        hv[l] = h.count;
        len[l] = h.len;
        light[l] = hv[l] ? 0u : (mode == 0 ? light_weight(deg[l], 0u) : deg[l] * sets[l]);
    }
    *n_items = 0;
    *taken = nb;
    if (!any) return 0;   // every entry already expanded
    // segments of light entries: a lane starts one when its segment index
    // differs from the previous lane's
    uint32_t segidx[W] = {0};
    bool first[W] = {false};
    uint32_t acc = 0, nseg = 0;
    for (uint32_t l = 0; l < nb; ++l) {
        acc += light[l];
        segidx[l] = segment_of(acc, light[l], seg);
        first[l] = l == 0 || segidx[l] != segidx[l - 1];
        nseg += first[l] ? 1u : 0u;
    }
    uint32_t hscan[W] = {0};
    auto rescan = [&]() {
        uint32_t s = 0;
        for (uint32_t l = 0; l < W; ++l) {
            s += hv[l];
            hscan[l] = s;
        }
    };
    rescan();
    uint64_t need = (uint64_t)nseg + hscan[W - 1];
    if (mode == 0 && plan_fit((uint32_t)std::min<uint64_t>(need, ~0u), 1u, item_cap) == kPlanOneEntry) {
        nb = 1;
        for (uint32_t l = 1; l < W; ++l) hv[l] = 0;
        for (uint32_t l = 1; l < W; ++l) first[l] = false;
        nseg = 1;
        rescan();
        need = 1u + (uint64_t)hscan[W - 1];
        *taken = 1;
    }
    if (need > cap_out) return -1;
    uint32_t out = 0;
    for (uint32_t l = 0; l < nb; ++l) {
        if (!first[l]) continue;
        uint32_t next = l + 1;
        while (next < nb && !first[next]) ++next;
        uint32_t *it = items + 4 * (size_t)out++;
        it[0] = l;
        it[1] = next - l;
        it[2] = it[3] = 0;
    }
    const uint32_t H = hscan[W - 1];
    for (uint32_t q = 0; q < H; ++q) {
        const uint32_t k = scan_owner([&](uint32_t i) { return hscan[i]; }, q);
        const uint32_t excl = hscan[k] - hv[k];
        const ChunkRange c = chunk_range(e0[k], deg[k], len[k], q - excl);
        uint32_t *it = items + 4 * (size_t)(nseg + q);
        it[0] = k | 0x80000000u;
        it[1] = c.lo;
        it[2] = c.hi;
        it[3] = 0;
    }
    *n_items = (uint32_t)need;
    return 0;
}

namespace {

// The layout of one batch of up to 64 entries.
struct Batch {
    uint32_t nb = 0, nseg = 0, need = 0;
    uint32_t hv[64] = {}, len[64] = {}, hscan[64] = {};
    bool first[64] = {};
    void count() {
        uint32_t h = 0;
        nseg = 0;
        for (uint32_t l = 0; l < 64; ++l) {
            nseg += first[l] ? 1u : 0u;
            hscan[l] = h += hv[l];
        }
        need = nseg + h;
    }
    // Items from items[4 * at] on; entries are numbered from f0.
    void write(uint32_t f0, const uint32_t *deg, const uint32_t *e0, uint32_t *items, uint64_t at) const {
        for (uint32_t l = 0; l < nb; ++l) {
            if (!first[l]) continue;
            uint32_t next = l + 1;
            while (next < nb && !first[next]) ++next;
            const uint32_t it[4] = {f0 + l, next - l, 0u, 0u};
            std::copy(it, it + 4, items + 4 * at++);
        }
        for (uint32_t q = 0; q < hscan[63]; ++q) {
            const uint32_t k = scan_owner([&](uint32_t i) { return hscan[i]; }, q);
            const ChunkRange c = chunk_range(e0[f0 + k], deg[f0 + k], len[k], q - (hscan[k] - hv[k]));
            const uint32_t it[4] = {(f0 + k) | 0x80000000u, c.lo, c.hi, 0u};
            std::copy(it, it + 4, items + 4 * at++);
        }
    }
};

Batch lay_out(uint32_t mode, uint32_t f0, uint32_t n, const uint32_t *deg, const uint32_t *quads,
              const uint32_t *sets, const uint8_t *expanded, uint32_t chunk, uint32_t seg) {
    Batch b;
    b.nb = std::min(64u, n - f0);
    uint32_t acc = 0, before = 0;
    bool any = false;
    for (uint32_t l = 0; l < b.nb; ++l) {
        const uint32_t i = f0 + l;
        uint32_t light = 0;
        if (mode == 1 || !expanded[i]) {
            any = true;
            const HeavySplit h = mode == 0 ? heavy_split(deg[i], weighted_chunk(deg[i], quads[i], chunk))
                                           : ms_heavy_split(deg[i], sets[i], chunk);
            b.hv[l] = h.count;
            b.len[l] = h.len;
            light = h.count ? 0u : mode == 0 ? light_weight(deg[i], quads[i]) : deg[i] * sets[i];
        }
        acc += light;
        const uint32_t s = segment_of(acc, light, seg);
        b.first[l] = l == 0 || s != before;
        before = s;
    }
    if (!any) return Batch();   // nothing to plan in it
    b.count();
    return b;
}

}  // namespace

// A planning wave's share of a superstep: entries [0, n) of one set (mode 0) or
// of the level's frontier (mode 1).  deg[i] incidences from e0[i] on, quads[i]
// runs of four member positions (mode 0), sets[i] sets (mode 1).  *counter is the
// item buffer's, of item_cap items, as other waves left it, and is moved on.
// mode 0: expanded[i] marks entries that are done; *taken receives the entries
// planned, a prefix.  mode 1: expanded[i / 64] marks batches planned before and
// receives 1 for those planned now, *taken their number.  Items as above, with
// entries in place of lanes, and (0xFFFFFFFF, ..) where a reservation did not
// fit.  Returns 0, or -1 when an argument is out of range.
extern "C" int hyperim_model_plan_wave(uint32_t mode, uint32_t n, const uint32_t *deg, const uint32_t *quads,
                                       const uint32_t *e0, const uint32_t *sets, uint8_t *expanded, uint32_t chunk,
                                       uint32_t seg, uint32_t item_cap, uint32_t *items, uint64_t *counter,
                                       uint32_t *taken) {
    if (mode > 1 || n >= 0x80000000u || !deg || !e0 || !expanded || !items || !counter || !taken || chunk == 0 ||
        seg == 0 || (mode == 0 && !quads) || (mode == 1 && !sets))
        return -1;
    seg = std::max(seg, chunk);
    *taken = 0;
    auto reserve = [&](uint64_t need, uint64_t *base) {
        *base = *counter;
        *counter += need;
        if (*base + need <= item_cap) return true;
        for (uint64_t x = *base; x < item_cap; ++x) items[4 * x] = 0xFFFFFFFFu;
        return false;
    };
    uint64_t base = 0;
    if (mode == 0) {
        uint32_t head = 0, most = kPlanBatches;
        while (head < n) {
            const uint32_t batches = std::min(most, (n - head + 63u) / 64u);
            std::vector<Batch> bs;
            uint32_t need = 0;
            for (uint32_t b = 0; b < batches; ++b) {
                bs.push_back(lay_out(0, head + 64 * b, n, deg, quads, sets, expanded, chunk, seg));
                need += bs.back().need;
            }
            uint32_t entries = std::min(64 * batches, n - head);
            if (const PlanFit fit = plan_fit(need, batches, item_cap)) {
                if (fit == kPlanOneBatch) {
                    most = 1;
                    continue;
                }
                entries = 1;
                Batch &b = bs[0];
                b.nb = 1;
                for (uint32_t l = 1; l < 64; ++l) {
                    b.hv[l] = 0;
                    b.first[l] = false;
                }
                b.count();
                need = b.need;
            }
            if (need) {
                if (!reserve(need, &base)) break;
                for (uint32_t b = 0; b < batches; ++b) {
                    bs[b].write(head + 64 * b, deg, e0, items, base);
                    base += bs[b].need;
                }
                most = kPlanBatches;
            }
            head += entries;
        }
        *taken = head;
        return 0;
    }
    const uint32_t nbatch = (n + 63u) / 64u;
    for (uint32_t b0 = 0; b0 < nbatch; b0 += kPlanBatches) {
        const uint32_t b1 = std::min(b0 + kPlanBatches, nbatch);
        std::vector<Batch> bs(b1 - b0);
        uint64_t need = 0;
        for (uint32_t b = b0; b < b1; ++b) {
            if (expanded[b]) continue;
            bs[b - b0] = lay_out(1, 64 * b, n, deg, quads, sets, nullptr, chunk, seg);
            need += bs[b - b0].need;
        }
        if (need == 0) continue;
        const bool together = plan_together(need, item_cap);
        if (together && !reserve(need, &base)) continue;
        for (uint32_t b = b0; b < b1; ++b) {
            const Batch &x = bs[b - b0];
            if (x.need == 0 || (!together && !reserve(x.need, &base))) continue;
            x.write(64 * b, deg, e0, items, base);
            base += x.need;
            expanded[b] = 1;
            *taken += 1;
        }
    }
    return 0;
}

// which 0: phase_b_check(a, b, c, d); which 1: bundled_check(a, b, c, d, e, f).
extern "C" int hyperim_model_loop_check(uint32_t which, uint64_t a, uint64_t b, uint64_t c, uint64_t d, uint64_t e,
                                        uint64_t f) {
    if (which == 0) return phase_b_check(a, b, c, d);
    if (which == 1) return bundled_check(a, b, c, d, e, f);
    return -1;
}
