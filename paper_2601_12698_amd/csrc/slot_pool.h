// Units of device memory for launches whose workgroups meet in it (slot_map.h has the rule), and the host memory in which it is
// reported that launches are done with theirs.  A launch says so in device memory (unit_report.h), and a later one, where it is
// asked to, tells the host what it finds there when it begins: a write to host memory at the end of a launch costs 1 us of it.
//
// A launch can tell of launches on its own GPU only.  So each GPU has units, counts and words of its own, and what one of them has in
// flight, or has not told yet, is nothing to the others.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <thread>

#include "slot_map.h"

namespace addrms_host {

enum class Units { taken, none, capturing };

// One pool per kind of launch, with the units of each GPU.
template <int UNITS>
class SlotPool {
    struct Gpu;

public:
    static constexpr int kMaxGpus = 64;                      // eight of them in eight partitions each; further ones have no units
    // A launch's units.  They go back where launched() is not called.
    class Lease {
    public:
        Lease() = default;
        Lease(const Lease&) = delete;
        Lease& operator=(const Lease&) = delete;
        ~Lease() { if (gpu_) give_back(*this); }
        unsigned unit() const { return static_cast<unsigned>(unit_); }
        // What is to be written, and where, once the launch is done with its units (system scope).
        uint32_t number() const { return number_; }
        uint32_t* done() const { return done_; }
        // As number(), but of all launches with any of these units: no other one of them has it.
        uint32_t tag() const { return tag_; }
        // Whether this launch is to tell what launches before it on its GPU have said, and the words of all its units for that.
        bool tells() const { return tells_; }
        uint32_t* words() const { return done_ - unit_; }
        void launched() { gpu_ = nullptr; }

    private:
        friend class SlotPool;
        Gpu* gpu_ = nullptr;
        uint32_t* done_ = nullptr;
        uint32_t number_ = 0, tag_ = 0;
        int unit_ = -1;
        bool tells_ = false;
    };

    // A graph may be replayed beside itself and others, so that no units are its own: a capturing stream has none.
    // Where launches in flight have them all, this one waits for one of them to end, as it would for room in a full queue: a
    // program that queues 400 launches of 172 us at once gets 172.5 us each, and 194.7 where those that find no units take the
    // other kernel.  But what is in flight may depend on something that the caller has yet to do.  So the wait is bounded, and
    // after one in vain nobody waits until units have been found again.
    // tell(words): queues a launch on `stream` that does nothing but tell.  Where launches have ended, but none has begun after
    // them that was to tell, it finds units for this call or for one after it.  A call that does not wait queues one only if none
    // has been for as long as a call would wait: behind a stream that waits for something they would be added to its queue.
    template <class Tell>
    Units take(hipStream_t stream, int units, Lease* lease, Tell tell)
    {
        const bool pending = hipPeekAtLastError() != hipSuccess;
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
            forget_error(pending);
            return Units::none;
        }
        if (capture != hipStreamCaptureStatusNone) return Units::capturing;
        // A launch goes to its stream's GPU and meets in that GPU's memory, whichever GPU is the current one.
        int device = -1;
        if (device_of(stream, &device) != hipSuccess) {
            forget_error(pending);
            return Units::none;
        }
        if (device < 0 || device >= kMaxGpus) return Units::none;
        Gpu& gpu = gpu_[device];
        uint32_t* done = reports(gpu, pending);
        if (!done) return Units::none;
        for (clock::time_point began{};; std::this_thread::sleep_for(std::chrono::microseconds(20))) {
            bool ask = false, waits = true;
            {
                std::lock_guard<std::mutex> lock(gpu.mu);
                int u = gpu.map.take(units, done);
                uint32_t tag = u < 0 ? 0 : *std::max_element(gpu.tag + u, gpu.tag + u + units) + 1;
                if (u >= 0 && tag == 0) {
                    gpu.map.give_back(u);
                    u = -1;
                }
                if (u >= 0) {
                    gpu.in_vain = false;
                    std::fill_n(gpu.tag + u, units, tag);
                    gpu.untold += units;
                    lease->tag_ = tag;
                    lease->gpu_ = &gpu;
                    lease->done_ = done + u;
                    lease->number_ = gpu.map.number(u);
                    lease->unit_ = u;
                    lease->tells_ = gpu.untold >= kTellEvery;
                    if (lease->tells_) gpu.untold = 0;
                    return Units::taken;
                }
                const clock::time_point now = clock::now();
                if (began == clock::time_point{}) {
                    began = now;
                    waits = !gpu.in_vain;
                    ask = waits || now - gpu.asked > kWait;
                    if (ask) gpu.asked = now;
                } else {
                    if (now - began > kWait) gpu.in_vain = true;
                    waits = !gpu.in_vain;
                }
            }
            if (ask && tell(done) != hipSuccess) forget_error(pending);
            if (!waits) return Units::none;
        }
    }
    Units take(hipStream_t stream, int units, Lease* lease)
    {
        return take(stream, units, lease, [](uint32_t*) { return hipSuccess; });
    }

private:
    using clock = std::chrono::steady_clock;
    static constexpr std::chrono::milliseconds kWait{4};
    // A call above has failed, which is nothing to the caller: the thread's error goes, unless one was pending before, for
    // whoever caused that one to find.
    static void forget_error(bool pending)
    {
        if (!pending) (void)hipGetLastError();
    }
    // The handles of the null streams and of the calling thread's are the same on every GPU: they are the current one's.
    static hipError_t device_of(hipStream_t stream, int* device)
    {
        const bool current = stream == nullptr || stream == hipStreamLegacy || stream == hipStreamPerThread;
        return current ? hipGetDevice(device) : hipStreamGetDevice(stream, device);
    }
    static void give_back(const Lease& lease)
    {
        std::lock_guard<std::mutex> lock(lease.gpu_->mu);
        lease.gpu_->map.give_back(lease.unit_);
        if (lease.tells_) lease.gpu_->untold = kTellEvery;   // the next one does
    }
    // A launch tells if so many units have been taken since the last one that does, itself included.
    static constexpr int kTellEvery = UNITS / 16;
    // One word per unit of the GPU, allocated once and kept until the process ends.  NULL: not there (yet: no thread waits for
    // the one that allocates it).  Must not disturb a capture that another thread may be in.
    static uint32_t* reports(Gpu& gpu, bool pending)
    {
        uint32_t* done = gpu.done.load(std::memory_order_acquire);
        if (done || gpu.allocating.exchange(true)) return done;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
            void* p = nullptr;
            const hipError_t e = hipHostMalloc(&p, UNITS * sizeof(uint32_t), hipHostMallocPortable);
            (void)hipThreadExchangeStreamCaptureMode(&mode);
            if (e == hipSuccess) done = static_cast<uint32_t*>(p);
            else forget_error(pending);
        }
        if (done) {
            std::fill_n(done, UNITS, 0u);
            gpu.done.store(done, std::memory_order_release);
        } else {
            gpu.allocating.store(false);
        }
        return done;
    }
    struct Gpu {
        std::mutex mu;
        SlotMap<UNITS> map;
        // Tags of the last launches with each unit, from 1.  They grow by one while all units have been taken once, or 1 ms of
        // launches, so that 2^32 of them take a month and more.  Units behind the last one are not taken any more.
        uint32_t tag[UNITS] = {};
        bool in_vain = false;
        clock::time_point asked{};                           // when the last launch that only tells was queued
        int untold = 0;                                      // units taken since a launch was asked to tell
        std::atomic<uint32_t*> done{nullptr};
        std::atomic<bool> allocating{false};
    };
    Gpu gpu_[kMaxGpus];
};

}  // namespace addrms_host
