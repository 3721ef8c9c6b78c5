// Host-code checks of libhyperim.so over the stand-in runtime: one scenario per
// run (argv[1]); prints "ok ..." or says what is wrong and exits with 1.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <chrono>
#include <future>
#include <new>
#include <thread>
#include <vector>

#include "fake_hip.h"
#include "hyperim.h"

namespace {
bool no_memory = false;   // of the host
}

void *operator new(size_t n) {
    void *p = no_memory ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return no_memory ? nullptr : malloc(n ? n : 1); }
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

namespace {

#define NEED(cond, ...)                               \
    do {                                              \
        if (!(cond)) {                                \
            printf("line %d: %s: ", __LINE__, #cond); \
            printf(__VA_ARGS__);                      \
            printf("\n");                             \
            return 1;                                 \
        }                                             \
    } while (0)

hipStream_t stream(int i) { return reinterpret_cast<hipStream_t>((uintptr_t)(16 * (i + 1))); }

// n vertices in hyperedges of two.
hyperim_graph pairs(uint32_t n, hipStream_t s, uint32_t model = HYPERIM_MODEL_CONST, bool stratify = true) {
    std::vector<uint32_t> off(n / 2 + 1), mem(n / 2 * 2);
    for (uint32_t e = 0; e <= n / 2; ++e) off[e] = 2 * e;
    for (uint32_t v = 0; v < mem.size(); ++v) mem[v] = v;
    hyperim_prob p{model, 0.5f};
    hyperim_graph g = nullptr;
    if (hyperim_build_graph(n, n / 2, off.data(), mem.data(), 0, p, s, &g) != HYPERIM_OK) return nullptr;
    if (stratify && hyperim_stratify(g, s, nullptr) != HYPERIM_OK) return nullptr;
    return g;
}

// The shared workspace is one stream's at a time: no call queues work on its
// stream while an earlier call's work waits on another.
int streams() {
    constexpr int kThreads = 3, kCalls = 20;
    hyperim_graph g[kThreads];
    hyperim_pool p[kThreads], q[kThreads];
    for (int t = 0; t < kThreads; ++t) {
        g[t] = pairs(50000 + 1000 * t, stream(t));
        NEED(g[t], "graph");
        NEED(hyperim_pool_create(g[t], nullptr, 0, 0, &p[t]) == HYPERIM_OK, "pool");
        NEED(hyperim_pool_create(g[t], nullptr, 0, 0, &q[t]) == HYPERIM_OK, "pool");
    }
    (void)hipDeviceSynchronize();
    fake::sync_us = 300;
    fake::watch = true;
    int bad[kThreads] = {};
    std::vector<std::thread> ts;
    for (int t = 0; t < kThreads; ++t)
        ts.emplace_back([&, t] {
            for (uint64_t i = 0; i < kCalls; ++i) {
                bad[t] |= hyperim_generate_rr(g[t], 7, 0, 0, 100 * i, 100 * i + 100, p[t], stream(t));
                hyperim_rr_task task{g[t], q[t], 7, 0, 1, 100 * i, 100 * i + 100};
                bad[t] |= hyperim_generate_rr_batch(&task, 1, (uint32_t)(i & 1), stream(t));
                uint32_t seeds[2];
                uint64_t gains[2], cov;
                bad[t] |= hyperim_greedy(g[t], p[t], 100, 2, stream(t), seeds, gains);
                bad[t] |= hyperim_stratify(g[t], stream(t), nullptr);
            }
        });
    for (auto &x : ts) x.join();
    fake::watch = false;
    for (int t = 0; t < kThreads; ++t) NEED(bad[t] == 0, "thread %d: a call failed", t);
    NEED(fake::overlaps == 0, "%ld times", fake::overlaps.load());
    printf("ok %ld launches\n", fake::launches.load());
    return 0;
}

// Memory that runs out at the i-th allocation of a generation call: the call
// says so, and the next one, with memory again, finds or makes everything that
// a first call makes.
int workspace_nomem() {
    hyperim_graph g = pairs(50000, nullptr);
    NEED(g, "graph");
    auto generate = [&]() {
        hyperim_pool p = nullptr;
        fake::fail_from = -1;
        if (hyperim_pool_create(g, nullptr, 0, 0, &p) != HYPERIM_OK) return -100;
        const int rc = hyperim_generate_rr(g, 7, 0, 0, 0, 500, p, nullptr);
        hyperim_pool_free(p);
        return rc;
    };
    NEED(generate() == HYPERIM_OK, "first run");   // (sizes the stage by a guess; later ones know the sets)
    NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
    NEED(generate() == HYPERIM_OK, "clean run");
    size_t want = 0, got = 0;
    hyperim_workspace_info(&want);
    int failed = 0;
    for (long i = 0;; ++i) {
        NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
        hyperim_pool p = nullptr;
        NEED(hyperim_pool_create(g, nullptr, 0, 0, &p) == HYPERIM_OK, "pool");
        fake::fail_from = fake::mallocs + i;
        const int rc = hyperim_generate_rr(g, 7, 0, 0, 0, 500, p, nullptr);
        fake::fail_from = -1;
        hyperim_pool_free(p);
        if (rc == HYPERIM_OK) break;
        NEED(rc == HYPERIM_ENOMEM, "allocation %ld: status %d", i, rc);
        ++failed;
        NEED(generate() == HYPERIM_OK, "after a failure of allocation %ld", i);
        hyperim_workspace_info(&got);
        NEED(got == want, "after a failure of allocation %ld: %zu bytes of workspace instead of %zu", i, got, want);
    }
    NEED(failed > 10, "%d allocations failed", failed);
    hyperim_graph_free(g);
    printf("ok %d\n", failed);
    return 0;
}

// Memory that runs out while a pool grows: the pool keeps what it held, at
// addresses that are still its own, and takes the sets when asked again.
int pool_nomem() {
    hyperim_graph g = pairs(4000, nullptr);
    NEED(g, "graph");
    int failed = 0;
    for (long i = 0;; ++i) {
        hyperim_pool p = nullptr;
        NEED(hyperim_pool_create(g, nullptr, 0, 0, &p) == HYPERIM_OK, "pool");
        NEED(hyperim_generate_rr(g, 7, 0, 0, 0, 900, p, nullptr) == HYPERIM_OK, "first ids");
        NEED(hyperim_workspace_release() == HYPERIM_OK, "release");   // freed blocks do not stay either
        fake::fail_from = fake::mallocs + i;
        const int rc = hyperim_generate_rr(g, 7, 0, 0, 900, 60000, p, nullptr);
        fake::fail_from = -1;
        NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
        const uint64_t *off = nullptr;
        const uint32_t *mem = nullptr, *roots = nullptr;
        uint64_t count = 0;
        NEED(hyperim_pool_view(p, &off, &mem, &roots, nullptr, &count) == HYPERIM_OK, "view");
        NEED(fake::live(off) && fake::live(mem) && fake::live(roots), "storage after a failure of allocation %ld", i);
        if (rc != HYPERIM_OK) {
            NEED(rc == HYPERIM_ENOMEM && count == 900, "allocation %ld: status %d, %llu sets", i, rc,
                 (unsigned long long)count);
            NEED(hyperim_generate_rr(g, 7, 0, 0, 900, 60000, p, nullptr) == HYPERIM_OK, "again");
            ++failed;
        }
        hyperim_pool_free(p);
        if (rc == HYPERIM_OK) break;
    }
    NEED(failed > 10, "%d allocations failed", failed);
    hyperim_graph_free(g);
    printf("ok %d\n", failed);
    return 0;
}

// Memory that runs out while the layer tables are built: a later call builds
// them again instead of taking what there is of them.
int tables_nomem() {
    // route: tables of a coin graph; stratify: of a stratified-setting graph,
    // which generates nothing until a call succeeds
    for (uint32_t model : {HYPERIM_MODEL_CONST, HYPERIM_MODEL_LAYERED}) {
        const bool route = model == HYPERIM_MODEL_CONST;
        size_t want = 0;
        int failed = 0;
        for (long i = -1;; ++i) {   // -1: nothing fails
            NEED(hyperim_workspace_release() == HYPERIM_OK, "release");   // no block of an earlier graph
            hyperim_graph g = pairs(4000, nullptr, model, route);
            NEED(g, "graph");
            auto call = [&]() {
                return route ? hyperim_route(g, 1, nullptr, nullptr) : hyperim_stratify(g, nullptr, nullptr);
            };
            int rc = HYPERIM_OK;
            if (i >= 0) {
                fake::fail_from = fake::mallocs + i;
                rc = call();
                fake::fail_from = -1;
            }
            const bool last = i >= 0 && rc == HYPERIM_OK;
            if (rc != HYPERIM_OK) {
                ++failed;
                NEED(rc == HYPERIM_ENOMEM, "allocation %ld: status %d", i, rc);
                if (!route) {
                    hyperim_pool p = nullptr;
                    NEED(hyperim_pool_create(g, nullptr, 0, 0, &p) == HYPERIM_OK, "pool");
                    NEED(hyperim_generate_rr(g, 7, 0, 0, 0, 5, p, nullptr) == HYPERIM_ESTATE, "allocation %ld", i);
                    hyperim_pool_free(p);
                }
            }
            if (!last) NEED(call() == HYPERIM_OK, "allocation %ld", i);
            NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
            if (i < 0) want = fake::live_blocks();
            NEED(fake::live_blocks() == want, "after a failure of allocation %ld: a graph of %zu arrays instead of %zu",
                 i, fake::live_blocks(), want);
            hyperim_graph_free(g);
            if (last) break;
        }
        NEED(failed > 5, "%d allocations failed", failed);
    }
    printf("ok both models\n");
    return 0;
}

// A session of 1 GiB answers queries on a graph of 30000 vertices, with a fresh
// workspace and with one that another call left laid out generously; it stays
// within its budget, and the next call without one lays the workspace out anew.
int small_budget() {
    const size_t budget = 1ull << 30;
    hyperim_graph g = pairs(30000, nullptr);
    NEED(g, "graph");
    size_t full = 0, now = 0;
    for (int warm = 0; warm < 2; ++warm) {
        NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
        if (warm) {
            hyperim_pool p = nullptr;
            NEED(hyperim_pool_create(g, nullptr, 0, 0, &p) == HYPERIM_OK, "pool");
            NEED(hyperim_generate_rr(g, 7, 0, 0, 0, 500, p, nullptr) == HYPERIM_OK, "generate");
            hyperim_pool_free(p);
            hyperim_workspace_info(&full);
            NEED(full > budget, "%zu bytes", full);
        }
        fake::peak = 0;
        hyperim_session s = nullptr;
        NEED(hyperim_session_create(budget, nullptr, nullptr, &s) == HYPERIM_OK, "session");
        uint64_t ticket = 0;
        hyperim_query q{g, 2, 0, 0.5, 1.0, 7};
        NEED(hyperim_session_submit(s, &q, &ticket) == HYPERIM_OK, "submit");
        int rc = HYPERIM_PENDING;
        uint32_t seeds[2];
        for (int i = 0; i < 100 && rc == HYPERIM_PENDING; ++i) {
            hyperim_session_stats st;
            NEED(hyperim_session_step(s, &st) == HYPERIM_OK, "step");
            NEED(st.bytes_resident <= budget, "%zu bytes resident", st.bytes_resident);
            rc = hyperim_session_poll(s, ticket, seeds, nullptr, nullptr);
        }
        NEED(rc == HYPERIM_OK, "warm %d: status %d: %s", warm, rc, hyperim_strerror(rc));
        NEED(fake::peak <= budget, "warm %d: %zu bytes allocated", warm, fake::peak.load());
        hyperim_session_free(s);
    }
    uint32_t seeds[2];
    NEED(hyperim_select_seeds(g, 2, 0.5, 1.0, 7, 0, nullptr, nullptr, seeds, nullptr, nullptr) == HYPERIM_OK, "alone");
    hyperim_workspace_info(&now);
    NEED(now >= full, "%zu bytes laid out, %zu before", now, full);
    hyperim_graph_free(g);
    printf("ok %zu\n", now);
    return 0;
}

// A pool whose storage has the size of `ids` ids.
hyperim_pool pool_of(hyperim_graph g, uint64_t ids) {
    hyperim_pool p = nullptr;
    if (hyperim_pool_create(g, nullptr, 0, 0, &p) != HYPERIM_OK) return nullptr;
    if (hyperim_generate_rr(g, 7, 0, 0, 0, ids, p, nullptr) != HYPERIM_OK) return nullptr;
    return p;
}

hyperim_pool freed_meanwhile = nullptr;
std::future<void> other;
bool stuck = false;

// Freed blocks: a thread that waits for the device keeps nobody else from
// freeing; what is freed during the wait is waited for again before it serves;
// freeing needs no memory of the host.
int blocks() {
    hyperim_graph g = pairs(4000, nullptr);
    NEED(g, "graph");
    hyperim_pool a = pool_of(g, 40000), b = pool_of(g, 90000);
    NEED(a && b, "pools");
    NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
    hyperim_pool_free(a);
    freed_meanwhile = b;
    fake::on_device_sync = [] {
        fake::on_device_sync = nullptr;
        other = std::async(std::launch::async, [] { hyperim_pool_free(freed_meanwhile); });
        stuck = other.wait_for(std::chrono::seconds(5)) != std::future_status::ready;
    };
    long syncs = fake::device_syncs;
    a = pool_of(g, 40000);   // in a's blocks: the device is waited for, b is freed meanwhile
    NEED(a && fake::device_syncs > syncs, "no wait");
    NEED(!stuck, "a free waited for another thread's wait for the device");
    syncs = fake::device_syncs;
    const long mallocs = fake::mallocs;
    b = pool_of(g, 90000);
    // pool_create waits once by itself
    NEED(b && fake::device_syncs > syncs + 1, "a block freed during a wait served without one");
    NEED(fake::mallocs - mallocs < 8, "%ld allocations", fake::mallocs - mallocs);
    std::vector<hyperim_pool> many;
    for (int i = 0; i < 200; ++i) {
        many.push_back(nullptr);
        NEED(hyperim_pool_create(g, nullptr, 0, 0, &many.back()) == HYPERIM_OK, "pool");
    }
    no_memory = true;
    for (hyperim_pool p : many) hyperim_pool_free(p);
    no_memory = false;
    // blocks are given back at the latest by the release
    hyperim_pool_free(a);
    hyperim_pool_free(b);
    hyperim_graph_free(g);
    NEED(hyperim_workspace_release() == HYPERIM_OK && fake::live_blocks() == 0, "%zu blocks left", fake::live_blocks());
    printf("ok %ld waits\n", fake::device_syncs.load());
    return 0;
}

// A batch of supersteps that does not finish within the wait limit: the call
// says so without waiting on, the next one leaves the workspace alone, and once
// the work is done everything goes on.
int wait_limit() {
    setenv("HYPERIM_WAIT_LIMIT_S", "0.01", 1);
    hyperim_graph g = pairs(50000, stream(0)), h = pairs(40000, stream(1));
    hyperim_pool p = nullptr, q = nullptr;
    NEED(g && h, "graphs");
    NEED(hyperim_pool_create(g, nullptr, 0, 0, &p) == HYPERIM_OK, "pool");
    NEED(hyperim_pool_create(h, nullptr, 0, 0, &q) == HYPERIM_OK, "pool");
    fake::stalled = true;
    NEED(hyperim_generate_rr(g, 7, 0, 0, 0, 100, p, stream(0)) == HYPERIM_EHIP, "the stalled call");
    NEED(fake::blocked == 0, "it waited on");
    const long launches = fake::launches;
    NEED(hyperim_generate_rr(h, 7, 0, 0, 0, 100, q, stream(1)) == HYPERIM_EHIP, "the next call");
    NEED(fake::launches == launches, "it used the workspace");
    fake::stalled = false;
    NEED(hyperim_generate_rr(h, 7, 0, 0, 0, 100, q, stream(1)) == HYPERIM_OK, "afterwards: %s", hyperim_strerror(-5));
    NEED(hyperim_generate_rr(g, 7, 0, 0, 0, 100, p, stream(0)) == HYPERIM_OK, "afterwards");
    NEED(hyperim_workspace_release() == HYPERIM_OK, "release");
    printf("ok %ld launches\n", fake::launches.load());
    return 0;
}

}  // namespace

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "streams")) return streams();
    if (!strcmp(what, "workspace_nomem")) return workspace_nomem();
    if (!strcmp(what, "pool_nomem")) return pool_nomem();
    if (!strcmp(what, "tables_nomem")) return tables_nomem();
    if (!strcmp(what, "small_budget")) return small_budget();
    if (!strcmp(what, "blocks")) return blocks();
    if (!strcmp(what, "wait_limit")) return wait_limit();
    printf("unknown scenario '%s'\n", what);
    return 2;
}
