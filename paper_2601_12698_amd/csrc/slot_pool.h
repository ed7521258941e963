// Units of device memory for launches whose workgroups meet in it (slot_map.h has the rule), and the host memory in which it is
// reported that launches are done with theirs.  A launch says so in device memory (unit_report.h), and a later one, where it is
// asked to, tells the host what it finds there when it begins: a write to host memory at the end of a launch costs 1 us of it.
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

// One pool per kind of launch, for all GPUs.
template <int UNITS>
class SlotPool {
public:
    // A launch's units.  They go back where launched() is not called.
    class Lease {
    public:
        Lease() = default;
        Lease(const Lease&) = delete;
        Lease& operator=(const Lease&) = delete;
        ~Lease() { if (pool_) pool_->give_back(*this); }
        unsigned unit() const { return static_cast<unsigned>(unit_); }
        // What is to be written, and where, once the launch is done with its units (system scope).
        uint32_t number() const { return number_; }
        uint32_t* done() const { return done_; }
        // As number(), but of all launches with any of these units: no other one of them has it.
        uint32_t tag() const { return tag_; }
        // Whether this launch is to tell what launches before it have said, and the words of all units for that.
        bool tells() const { return tells_; }
        uint32_t* words() const { return done_ - unit_; }
        void launched() { pool_ = nullptr; }

    private:
        friend class SlotPool;
        SlotPool* pool_ = nullptr;
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
    // them that was to tell, it finds units for this call or for one after it.
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
        uint32_t* done = reports(pending);
        if (!done) return Units::none;
        using clock = std::chrono::steady_clock;
        for (clock::time_point began{};; std::this_thread::sleep_for(std::chrono::microseconds(20))) {
            const bool first = began == clock::time_point{};
            {
                std::lock_guard<std::mutex> lock(mu_);
                int u = map_.take(units, done);
                uint32_t tag = u < 0 ? 0 : *std::max_element(tag_ + u, tag_ + u + units) + 1;
                if (u >= 0 && tag == 0) {
                    map_.give_back(u);
                    u = -1;
                }
                in_vain_ = in_vain_ && u < 0;
                if (u >= 0) {
                    std::fill_n(tag_ + u, units, tag);
                    untold_ += units;
                    lease->tag_ = tag;
                    lease->pool_ = this;
                    lease->done_ = done + u;
                    lease->number_ = map_.number(u);
                    lease->unit_ = u;
                    lease->tells_ = untold_ >= kTellEvery;
                    if (lease->tells_) untold_ = 0;
                    return Units::taken;
                }
                if (!first && clock::now() - began > std::chrono::milliseconds(4)) in_vain_ = true;
                if (in_vain_ && !first) return Units::none;
            }
            if (!first) continue;
            if (tell(done) != hipSuccess) forget_error(pending);
            began = clock::now();
        }
    }
    Units take(hipStream_t stream, int units, Lease* lease)
    {
        return take(stream, units, lease, [](uint32_t*) { return hipSuccess; });
    }

private:
    // A call above has failed, which is nothing to the caller: the thread's error goes, unless one was pending before, for
    // whoever caused that one to find.
    static void forget_error(bool pending)
    {
        if (!pending) (void)hipGetLastError();
    }
    void give_back(const Lease& lease)
    {
        std::lock_guard<std::mutex> lock(mu_);
        map_.give_back(lease.unit_);
        if (lease.tells_) untold_ = kTellEvery;              // the next one does
    }
    // A launch tells if so many units have been taken since the last one that does, itself included.
    static constexpr int kTellEvery = UNITS / 16;
    // One word per unit, which every GPU can write, allocated once and kept until the process ends.  NULL: not there (yet: no
    // thread waits for the one that allocates it).  Must not disturb a capture that another thread may be in.
    uint32_t* reports(bool pending)
    {
        uint32_t* done = done_.load(std::memory_order_acquire);
        if (done || allocating_.exchange(true)) return done;
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
            done_.store(done, std::memory_order_release);
        } else {
            allocating_.store(false);
        }
        return done;
    }
    std::mutex mu_;
    SlotMap<UNITS> map_;
    // Tags of the last launches with each unit, from 1.  They grow by one while all units have been taken once, or 1 ms of launches, so
    // that 2^32 of them take a month and more.  Units behind the last one are not taken any more.
    uint32_t tag_[UNITS] = {};
    bool in_vain_ = false;
    int untold_ = 0;                                         // units taken since a launch was asked to tell
    std::atomic<uint32_t*> done_{nullptr};
    std::atomic<bool> allocating_{false};
};

}  // namespace addrms_host
