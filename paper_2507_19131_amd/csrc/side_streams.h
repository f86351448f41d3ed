// Streams of the library's own for stages that run as two chains.  Host code.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <thread>

namespace mixaq {

constexpr int MAX_DEVICES = 64;

// Side streams for stages that run as two chains (see mixaq_stage_forward).  One per stream that callers use, not one per handle:
// the runtime spreads streams over four hardware queues, and with one per handle the second chain of every fourth handle
// shared the first one's queue (six blocks on 192 windows at C = 384, three sets of handles in turn: 361 us as two chains, 358 as
// one; with a side stream per caller 300).  What is queued on a side stream only ever waits for its caller's stream, so callers
// stay independent of one another.  At most MAX of them per device; a further caller takes over an idle one (nothing queued and no
// call in progress), the one unused for longest, or runs as one chain: behind work that still waits for another caller's stream its
// second chain would wait for that stream too, for ever if that one waits for it.  They are created with a block that may use them, or on
// a caller's first call, and are given back with the last such block.
class SideStreams {
public:
    struct Side {
        hipStream_t caller = nullptr, stream = nullptr;
        std::thread::id thread;                    // of the caller, where its stream's name means another stream in every thread
        hipEvent_t fork = nullptr, join = nullptr;
        int calls = 0;                             // in progress
        unsigned long long used = 0;
        std::mutex mu;                             // an event is recorded and waited for in one piece
        // the side stream starts after the work already on `st`
        hipError_t fork_from(hipStream_t st)
        {
            std::lock_guard<std::mutex> lock(mu);
            const hipError_t e = hipEventRecord(fork, st);
            return e != hipSuccess ? e : hipStreamWaitEvent(stream, fork, 0);
        }
        // `st` goes on behind the side stream's work; where it cannot be made to wait, the host does
        hipError_t join_to(hipStream_t st)
        {
            std::lock_guard<std::mutex> lock(mu);
            hipError_t e = hipEventRecord(join, stream);
            if (e == hipSuccess) e = hipStreamWaitEvent(st, join, 0);
            if (e != hipSuccess) (void)hipStreamSynchronize(stream);
            return e;
        }
    };
    static SideStreams& of(int device)
    {
        static SideStreams all[MAX_DEVICES];
        return all[device];
    }
    // one more block that may use them; ended by release().  Its stages run as one chain where no side stream is to be had, so this
    // cannot fail
    void retain(hipStream_t caller)
    {
        std::lock_guard<std::mutex> lock(mu_);
        ++blocks_;
        if (!find(caller)) (void)fill(caller);
    }
    void release()
    {
        std::lock_guard<std::mutex> lock(mu_);
        if (--blocks_ > 0) return;
        for (Side& s : side_) {
            if (s.join) (void)hipEventDestroy(s.join);
            if (s.fork) (void)hipEventDestroy(s.fork);
            if (s.stream) (void)hipStreamDestroy(s.stream);
            s.join = s.fork = nullptr;
            s.stream = s.caller = nullptr;
        }
    }
    // the caller's side stream, or NULL; ended by done()
    Side* begin(hipStream_t caller)
    {
        std::lock_guard<std::mutex> lock(mu_);
        Side* s = find(caller);
        if (!s) s = fill(caller);
        if (!s) s = take_over(caller);
        if (s) { ++s->calls; s->used = ++clock_; }
        return s;
    }
    void done(Side* s)
    {
        std::lock_guard<std::mutex> lock(mu_);
        --s->calls;
    }

private:
    static constexpr int MAX = 4;
    static bool per_thread(hipStream_t s) { return s == hipStreamPerThread; }
    Side* find(hipStream_t caller)
    {
        for (Side& s : side_)
            if (s.stream && s.caller == caller && (!per_thread(caller) || s.thread == std::this_thread::get_id())) return &s;
        return nullptr;
    }
    // a side stream in a place that has none yet, or NULL
    Side* fill(hipStream_t caller)
    {
        for (Side& s : side_) {
            if (s.stream) continue;
            if ((!s.fork && hipEventCreateWithFlags(&s.fork, hipEventDisableTiming) != hipSuccess) ||
                (!s.join && hipEventCreateWithFlags(&s.join, hipEventDisableTiming) != hipSuccess) ||
                hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) != hipSuccess) {
                (void)hipGetLastError();                     // not to be mistaken for a launch error later
                s.stream = nullptr;
                return nullptr;
            }
            return give(s, caller);
        }
        return nullptr;
    }
    // of the idle ones of other callers the one unused for longest, or NULL
    Side* take_over(hipStream_t caller)
    {
        Side* s = nullptr;
        // asked in the relaxed mode: the stream is never captured itself, and another thread's capture is not to be broken off
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        for (Side& c : side_)
            if (c.stream && !c.calls && (!s || c.used < s->used) && hipStreamQuery(c.stream) == hipSuccess) s = &c;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        (void)hipGetLastError();                             // "not ready" is not to be mistaken for a launch error later
        return s ? give(*s, caller) : nullptr;
    }
    static Side* give(Side& s, hipStream_t caller)
    {
        s.caller = caller;
        s.thread = std::this_thread::get_id();
        return &s;
    }
    std::mutex mu_;
    Side side_[MAX];
    int blocks_ = 0;
    unsigned long long clock_ = 0;
};

}  // namespace mixaq
