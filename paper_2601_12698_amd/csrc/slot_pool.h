// Slots of device memory for launches whose workgroups meet in it (stream_slots.h has the rule), and the host memory in which
// these launches report that they are done with their slot.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <thread>

#include "stream_slots.h"

namespace addrms_host {

// One pool per kind of launch, for all GPUs.
class SlotPool {
public:
    // A slot, held from its choice to the launches that use it.
    class Lease {
    public:
        unsigned slot() const { return static_cast<unsigned>(slot_); }
        // What the next launch is to write, and where, when it is done with the slot (system scope, the launch's last access).
        uint32_t number() const { return slots_->next(slot_); }
        uint32_t* done() const { return done_; }
        void launched() { slots_->launched(slot_); }

    private:
        friend class SlotPool;
        std::unique_lock<std::mutex> lock_;
        StreamSlots* slots_ = nullptr;
        uint32_t* done_ = nullptr;
        int slot_ = -1;
    };

    // False: none.  A graph may be replayed on any stream and beside others, so that no slot is its own: a capturing stream
    // has none.  Nor has the per-thread default stream, one handle for as many streams as threads.
    bool take(hipStream_t stream, Lease* lease)
    {
        if (stream == hipStreamPerThread) return false;
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &capture) != hipSuccess) { (void)hipGetLastError(); return false; }
        // A launch goes to its stream's GPU and meets in that GPU's memory, whichever GPU is the current one.
        int dev = -1;
        if (capture != hipStreamCaptureStatusNone || device_of(stream, &dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
        // A launch may wait for room in its stream's queue, and that stream for something the threads waiting here have yet
        // to do: they wait some tens of microseconds, ten launches' time, and then do without.
        lease->lock_ = std::unique_lock<std::mutex>(mu_, std::try_to_lock);
        for (int i = 0; i < 200 && !lease->lock_; ++i) {
            std::this_thread::yield();
            (void)lease->lock_.try_lock();
        }
        if (!lease->lock_) return false;
        Device& d = device_[dev];
        if (!d.done && !allocate(d)) return false;
        lease->slot_ = d.slots.take(reinterpret_cast<uintptr_t>(stream), d.done, kStride);
        if (lease->slot_ < 0) return false;
        lease->slots_ = &d.slots;
        lease->done_ = d.done + lease->slot_ * kStride;
        return true;
    }

private:
    static constexpr int kMaxDevices = 64, kStride = 16;     // one 64-byte line of host memory per slot
    struct Device {
        StreamSlots slots;
        uint32_t* done = nullptr;
    };
    // The null stream's handle is the same on every GPU: it is the current one's.
    static hipError_t device_of(hipStream_t stream, int* dev)
    {
        return stream == nullptr || stream == hipStreamLegacy ? hipGetDevice(dev) : hipStreamGetDevice(stream, dev);
    }
    // 256 bytes, once per GPU, kept until the process ends.  Must not disturb a capture that another thread may be in.
    static bool allocate(Device& d)
    {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return false;
        void* p = nullptr;
        const size_t n = static_cast<size_t>(addrms::kStreamSlots) * kStride;
        const hipError_t e = hipHostMalloc(&p, n * sizeof(uint32_t), hipHostMallocDefault);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e != hipSuccess) { (void)hipGetLastError(); return false; }
        std::fill_n(static_cast<uint32_t*>(p), n, 0u);
        d.done = static_cast<uint32_t*>(p);
        return true;
    }
    std::mutex mu_;
    Device device_[kMaxDevices];
};

}  // namespace addrms_host
