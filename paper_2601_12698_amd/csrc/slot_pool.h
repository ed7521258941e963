// Units of device memory for launches whose workgroups meet in it (slot_map.h has the rule), and the host memory in which
// these launches report that they are done with theirs.
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
        ~Lease() { if (pool_) pool_->give_back(unit_); }
        unsigned unit() const { return static_cast<unsigned>(unit_); }
        // What the launch is to write, and where, when it is done with its units (system scope, its last access).
        uint32_t number() const { return number_; }
        uint32_t* done() const { return done_; }
        void launched() { pool_ = nullptr; }

    private:
        friend class SlotPool;
        SlotPool* pool_ = nullptr;
        uint32_t* done_ = nullptr;
        uint32_t number_ = 0;
        int unit_ = -1;
    };

    // A graph may be replayed beside itself and others, so that no units are its own: a capturing stream has none.
    // Where launches in flight have them all, this one waits for one of them to end, as it would for room in a full queue: a
    // program that queues 400 launches of 172 us at once gets 172.5 us each, and 194.7 where those that find no units take the
    // other kernel.  But what is in flight may depend on something that the caller has yet to do.  So the wait is bounded, and
    // after one in vain nobody waits until units have been found again.
    Units take(hipStream_t stream, int units, Lease* lease)
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
            std::lock_guard<std::mutex> lock(mu_);
            const int u = map_.take(units, done);
            in_vain_ = in_vain_ && u < 0;
            if (u >= 0) {
                lease->pool_ = this;
                lease->done_ = done + u;
                lease->number_ = map_.number(u);
                lease->unit_ = u;
                return Units::taken;
            }
            if (in_vain_) return Units::none;
            if (began == clock::time_point{}) began = clock::now();
            else if (clock::now() - began > std::chrono::milliseconds(4)) {
                in_vain_ = true;
                return Units::none;
            }
        }
    }

private:
    // A call above has failed, which is nothing to the caller: the thread's error goes, unless one was pending before, for
    // whoever caused that one to find.
    static void forget_error(bool pending)
    {
        if (!pending) (void)hipGetLastError();
    }
    void give_back(int unit)
    {
        std::lock_guard<std::mutex> lock(mu_);
        map_.give_back(unit);
    }
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
    bool in_vain_ = false;
    std::atomic<uint32_t*> done_{nullptr};
    std::atomic<bool> allocating_{false};
};

}  // namespace addrms_host
