// Who may use which piece of the device memory in which workgroups of one launch meet (addrms_split_body, the gate).  Host
// code only, no HIP.
//
// Such memory belongs to the loaded code object and is cut into kStreamSlots slots per GPU.  A launch needs a slot that no
// other launch in flight uses.  Launches of one stream follow each other, so a slot that is bound to a stream serves all
// of them, however many are queued; a slot whose last launch has reported itself as done is free for another stream.  A
// stream that finds no slot takes the kernels that need none.  A stream's handle names the same stream for as long as work
// of it is in flight (hipStreamDestroy waits for it: 6.9 ms behind 40 launches of 172 us).
#pragma once
#include <stdint.h>

namespace addrms {
constexpr int kStreamSlots = 4;
}  // namespace addrms

namespace addrms_host {

// The slots of one GPU.  Calls are serialised by the caller, from take() to launched().
class StreamSlots {
public:
    // done[slot * stride]: the number of the last launch that has reported itself, 0 at first.  -1: none to be had.
    int take(uintptr_t stream, const volatile uint32_t* done, int stride)
    {
        int free = -1;
        for (int i = 0; i < addrms::kStreamSlots; ++i) {
            if (slot_[i].bound && slot_[i].stream == stream) return i;
            if (free < 0 && (!slot_[i].bound || done[i * stride] == slot_[i].issued)) free = i;
        }
        if (free >= 0) slot_[free] = {stream, slot_[free].issued, true};
        return free;
    }
    // The number that the slot's next launch reports.
    uint32_t next(int slot) const { return slot_[slot].issued + 1u; }
    // That launch is in the stream's queue.  A launch that failed is not announced: the number stays the next one.
    void launched(int slot) { ++slot_[slot].issued; }

private:
    struct Slot { uintptr_t stream; uint32_t issued; bool bound; };
    Slot slot_[addrms::kStreamSlots] = {};
};

}  // namespace addrms_host
