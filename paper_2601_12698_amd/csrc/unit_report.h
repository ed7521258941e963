// How launches whose workgroups meet in units of device memory (slot_map.h) say that they are done with them, and how the host
// comes to know it.  Device code.
//
// A launch's last word is one in device memory.  Host memory is written by a later launch that is asked to tell (slot_pool.h), and
// by a workgroup of its own at its beginning, where the write is over long before the launch is.  As the last access of the launch
// itself that write took 0.7-1.5 us, in which the next launch of the stream waits.
//
// Which GPU a launch ran on is not asked here either: each GPU tells a number once, the one that only it has found new, and a
// place has its next launch, with another number, only after that has arrived.  So what was told never goes back.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace addrms {

constexpr uint32_t kUnitDone = 1u << 31;
template <int UNITS>
struct UnitReports {
    uint64_t state[UNITS];                                   // of the launch with units from here on: its number, then kUnitDone once it is done
    uint32_t told[UNITS];                                    // number that this GPU has told last
};
// The launch is done.  By the one thread that knows.
__device__ __forceinline__ void unit_done(uint64_t* state, uint32_t number)
{
    __hip_atomic_store(state, static_cast<uint64_t>(number) << 32 | kUnitDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One of `all` (up to 2^31) pieces of the launch is done; piece: which.  Two operations on one word, in that order, and nobody waits
// for them: the first to come sets the count to 0, since numbers of a place only grow, and what is added is kUnitDone in all, but
// short of it for less than all pieces.
__device__ __forceinline__ void unit_piece_done(uint64_t* state, uint32_t number, uint32_t piece, uint32_t all)
{
    (void)__hip_atomic_fetch_max(state, static_cast<uint64_t>(number) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    (void)__hip_atomic_fetch_add(state, static_cast<uint64_t>(piece == 0u ? kUnitDone - (all - 1u) : 1u), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
}
// By a workgroup of `threads`: the numbers of launches that are done and not told yet go to the host's words.
template <int UNITS>
__device__ __forceinline__ void unit_tell(UnitReports<UNITS>* r, uint32_t* words, uint32_t threads)
{
    for (uint32_t u = threadIdx.x; u < static_cast<uint32_t>(UNITS); u += threads) {
        const uint64_t s = __hip_atomic_load(&r->state[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t number = static_cast<uint32_t>(s >> 32);
        if (static_cast<uint32_t>(s) != kUnitDone) continue;
        if (__hip_atomic_exchange(&r->told[u], number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != number)
            __hip_atomic_store(&words[u], number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace addrms
