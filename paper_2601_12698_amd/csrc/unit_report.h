// How launches whose workgroups meet in units of device memory (slot_map.h) say that they are done with them, and how the host
// comes to know it.  Device code.
//
// A launch's last word is one in device memory.  Host memory is written by a later launch that is asked to tell (slot_pool.h), and
// by a workgroup of its own at its beginning, where the write is over long before the launch is.  As the last access of the launch
// itself that write took 0.7-1.5 us, in which the next launch of the stream waits.
//
// A GPU tells of its own launches, into words of its own (slot_pool.h), and each number once: by the workgroup that raised `told` to
// it.  A place has its next launch, with a greater number, only after that has arrived.  So a word never goes back.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace addrms {

constexpr uint32_t kUnitDone = 1u << 31;
template <int UNITS>
struct UnitReports {
    uint64_t state[UNITS];                                   // of the launch with units from here on: its number, then kUnitDone once it is done
    uint32_t told[UNITS];                                    // greatest number that this GPU has told
};
// The launch is done.  By the one thread that knows.
__device__ __forceinline__ void unit_done(uint64_t* state, uint32_t number)
{
    __hip_atomic_store(state, static_cast<uint64_t>(number) << 32 | kUnitDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One of `all` pieces of the launch is done; piece: which.  With the number, the count of pieces comes to kUnitDone with the last one
// and not before.  Nobody waits for the additions, but they are made one after the other, 10 ns each.  Few pieces each make sure first
// that the number is this launch's (numbers of a place only grow, and the first to come starts the count at 0); of many, which would
// take twice as long, piece 0 looks at what the launch before has left and adds the step to this one's.
__device__ __forceinline__ void unit_piece_done(uint64_t* state, uint32_t number, uint32_t piece, uint32_t all)
{
    constexpr uint32_t kFew = 8;
    if (all == 1u) return unit_done(state, number);
    uint64_t more = piece == 0u ? kUnitDone - (all - 1u) : 1u;
    if (all <= kFew) {
        (void)__hip_atomic_fetch_max(state, static_cast<uint64_t>(number) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (piece == 0u) {
        const uint64_t was = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // and pieces of this launch, if any
        more += static_cast<uint64_t>(number - static_cast<uint32_t>(was >> 32)) << 32;
        more -= static_cast<uint32_t>(was) & kUnitDone;      // 0 before the first launch
    }
    (void)__hip_atomic_fetch_add(state, more, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// By a workgroup of `threads`: the numbers of launches that are done and not told yet go to the host's words.
template <int UNITS>
__device__ __forceinline__ void unit_tell(UnitReports<UNITS>* r, uint32_t* words, uint32_t threads)
{
    for (uint32_t u = threadIdx.x; u < static_cast<uint32_t>(UNITS); u += threads) {
        const uint64_t s = __hip_atomic_load(&r->state[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t number = static_cast<uint32_t>(s >> 32);
        if (static_cast<uint32_t>(s) != kUnitDone) continue;
        if (__hip_atomic_fetch_max(&r->told[u], number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < number)
            __hip_atomic_store(&words[u], number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace addrms
