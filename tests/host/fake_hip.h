// Controls and counters of the stand-in HIP runtime (fake_hip.cpp).
#pragma once

#include <stddef.h>

#include <atomic>

namespace fake {
extern std::atomic<size_t> total, used, peak;   // device memory: capacity, allocated, most ever
extern std::atomic<long> mallocs;               // calls of hipMalloc so far
extern std::atomic<long> fail_from;             // hipMalloc fails from this call on (-1: never)
extern std::atomic<long> launches, device_syncs;
extern std::atomic<bool> watch;                 // count `overlaps` ...
extern std::atomic<long> overlaps;              // ... work queued while another stream had some left
extern std::atomic<int> sync_us;                // how long waiting for a busy stream takes
extern std::atomic<bool> stalled;               // no event completes, and a wait for a busy stream ...
extern std::atomic<long> blocked;               // ... would not have ended
extern std::atomic<void (*)()> on_device_sync;  // called within every hipDeviceSynchronize
size_t live_blocks();                           // blocks not freed yet
bool live(const void *p);                       // whether p is the start of a block not freed yet
}  // namespace fake
