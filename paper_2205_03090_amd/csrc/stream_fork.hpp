// stream_fork.hpp -- side streams for the independent parts of one call.
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <mutex>

#include "ptflash.h"

namespace ptf {

constexpr int kMaxDevices = 64;

// Three streams of default priority and the events that order them against the
// caller's stream.  Held by one call at a time, and only while it enqueues.
struct SideSet {
    static constexpr int kStreams = 3;
    std::mutex mu;
    bool made = false, usable = false;
    hipStream_t st[kStreams];
    hipEvent_t fork, done[kStreams];

    bool make()
    {
        // another thread may be capturing; creating streams here is no part of it
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return false;
        bool ok = hipEventCreateWithFlags(&fork, hipEventDisableTiming) == hipSuccess;
        for (int k = 0; ok && k < kStreams; ++k)
            ok = hipStreamCreateWithFlags(&st[k], hipStreamNonBlocking) == hipSuccess &&
                 hipEventCreateWithFlags(&done[k], hipEventDisableTiming) == hipSuccess;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        return ok;
    }
};
constexpr int kSideSets = 4;   // per device

struct SideSets {
    SideSet set[kSideSets];
    std::atomic<unsigned> next{0};
};

// Forks the work of one call from the caller's stream onto side streams and
// joins it back.  stream(0) is the caller's stream; the side streams come from a
// bounded set per device that is created on first use and kept, and a call holds
// its set (locked) while it enqueues.  A call under stream capture, and one for
// which no set can be had, gets one stream only.
class StreamFork {
public:
    static constexpr int kMax = 1 + SideSet::kStreams;
    // sets: of the current device; want: streams to use, at most kMax
    StreamFork(SideSets *sets, hipStream_t s, int want) : s_(s), set_(nullptr), n_(1)
    {
        if (want <= 1) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            return;
        }
        take(sets);
        const int side = (want < kMax ? want : kMax) - 1;
        if (set_->usable && hipEventRecord(set_->fork, s_) == hipSuccess)
            while (n_ - 1 < side && hipStreamWaitEvent(set_->st[n_ - 1], set_->fork, 0) == hipSuccess)
                ++n_;
        // a stream that could not be had is no error of the call
        if (n_ - 1 < side) (void)hipGetLastError();
        if (n_ == 1) {
            set_->mu.unlock();
            set_ = nullptr;
        }
    }
    ~StreamFork() { (void)join(); }   // joins what has not been joined
    StreamFork(const StreamFork &) = delete;
    StreamFork &operator=(const StreamFork &) = delete;
    int count() const { return n_; }
    hipStream_t stream(int k) const { return k == 0 ? s_ : set_->st[k - 1]; }

    // The caller's stream waits for every side stream.
    int join()
    {
        if (!set_) return PTFLASH_OK;
        int rc = PTFLASH_OK;
        for (int k = 0; k + 1 < n_; ++k) {
            if (hipEventRecord(set_->done[k], set_->st[k]) == hipSuccess &&
                hipStreamWaitEvent(s_, set_->done[k], 0) == hipSuccess)
                continue;
            // the caller's memory must not be in use past its own stream's order
            rc = PTFLASH_EHIP;
            (void)hipStreamSynchronize(set_->st[k]);
        }
        set_->mu.unlock();
        set_ = nullptr;
        return rc;
    }

private:
    // Takes (locks) a set: the first free one, or, where every set is taken, one in
    // turn, which waits for the launches of the call that holds it.  A lone caller
    // always gets the set made first, whose streams and the caller's own fall on
    // different hardware queues (there are four).  Callers on two streams may so queue
    // behind each other.  That is kept: all streams share the four queues, and both
    // sets without work left and no side streams while another call's run gain at one
    // size and lose at another (two streams, us for a call on each, nc 2-8: 2000 mixtures
    // 1070 this way, 860 with idle sets, 1040 without side streams; 30,000 1600, 1800,
    // 1750; 200,000 3250, 3350, 3600; no side streams at all 1760, 2570, 4250).
    void take(SideSets *sets)
    {
        for (int k = 0; k < kSideSets && !set_; ++k)
            if (sets->set[k].mu.try_lock()) set_ = &sets->set[k];
        if (!set_) {
            set_ = &sets->set[sets->next.fetch_add(1) % kSideSets];
            set_->mu.lock();
        }
        if (!set_->made) {
            set_->made = true;
            set_->usable = set_->make();
        }
    }

    hipStream_t s_;
    SideSet *set_;
    int n_;
};

}  // namespace ptf
