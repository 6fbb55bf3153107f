// Idle sessions of the blocking calls. A session is what such a call needs
// besides its problem: device memory, a pinned staging block and the phase
// events. hipMalloc, hipFree and seven events cost a small solve as much as its
// kernels (n = 18: 200 of 430 us), so finished calls leave theirs for the next
// one: at most kIdle of them in a process, with at most kKeepBytes of device
// memory each (larger blocks are freed by the call that made them). All idle
// ones are freed by release(), which also runs when an allocation fails.
//
// A session belongs to one call at a time and comes back only after its stream
// was synchronised without an error (a failed call's is destroyed, since work of
// it may be left), so threads and streams never share one. Memory that went
// with a device reset is told by its allocation's identifier and forgotten.
//
// Dev: the device calls (tests put a counting host device in their place).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace bnk {

template <class Dev>
struct Session {
    int dev = -1;
    char *ws = nullptr;          // device memory
    size_t bytes = 0;
    char *pin = nullptr;         // pinned host memory, kPinBytes
    uint64_t ws_id = 0, pin_id = 0;
    typename Dev::Events ev{};
    bool events = false;         // all of them were created
};

template <class Dev>
class SessionPool {
   public:
    static constexpr size_t kIdle = 4;
    static constexpr size_t kKeepBytes = (size_t)64 << 20;
    static constexpr size_t kPinBytes = (size_t)1 << 20;   // larger transfers go straight
    using S = Session<Dev>;
    enum class Got { ok, no_device, no_memory };

    // a session on the current device with at least `bytes` of device memory,
    // and with the events when asked for (events stays false if they failed)
    Got take(size_t bytes, bool events, S *out) {
        S s;
        int dev = -1;
        if (!Dev::current(&dev)) return Got::no_device;
        while (pick(dev, bytes, &s)) {
            if (intact(s)) break;
            s = S{};                         // nothing of it is left to free
        }
        s.dev = dev;
        if (s.bytes < bytes) {
            free_ws(s);
            bool lost = false;
            if (!Dev::alloc(bytes, &s.ws, &s.ws_id, &lost)) {
                if (!lost) {
                    release();
                    (void)Dev::alloc(bytes, &s.ws, &s.ws_id, &lost);
                }
                if (!s.ws) {
                    destroy(s);
                    return lost ? Got::no_device : Got::no_memory;
                }
            }
            s.bytes = bytes;
        }
        if (!s.pin) (void)Dev::alloc_pinned(kPinBytes, &s.pin, &s.pin_id);   // or the caller's memory
        if (events && !s.events) s.events = Dev::make_events(s.ev);
        *out = s;
        return Got::ok;
    }

    // the session of a finished call; `clean`: its stream was synchronised and
    // nothing failed
    void give(S &s, bool clean) {
        if (!clean) {
            destroy(s);
            return;
        }
        if (s.bytes > kKeepBytes) free_ws(s);
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (n_ < kIdle) {
                idle_[n_++] = s;
                s = S{};
                return;
            }
        }
        destroy(s);
    }

    // frees every idle session
    void release() {
        S out[kIdle];
        size_t n = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (; n < n_; ++n) out[n] = idle_[n];
            n_ = 0;
        }
        for (size_t k = 0; k < n; ++k)
            if (intact(out[k])) destroy(out[k]);
    }

   private:
    // removes the smallest idle session of the device that fits, else any of the
    // device, from the pool
    bool pick(int dev, size_t bytes, S *out) {
        std::lock_guard<std::mutex> lk(mu_);
        size_t best = kIdle;
        for (size_t k = 0; k < n_; ++k) {
            const S &c = idle_[k];
            if (c.dev != dev) continue;
            if (best == kIdle) {
                best = k;
                continue;
            }
            const size_t cur = idle_[best].bytes;
            if (c.bytes >= bytes ? cur < bytes || c.bytes < cur : false) best = k;
        }
        if (best == kIdle) return false;
        *out = idle_[best];
        idle_[best] = idle_[--n_];
        return true;
    }
    static bool intact(const S &s) {
        return (!s.ws || Dev::holds(s.ws, s.ws_id)) && (!s.pin || Dev::holds(s.pin, s.pin_id));
    }
    static void free_ws(S &s) {
        if (s.ws) Dev::release(s.ws);
        s.ws = nullptr;
        s.bytes = 0;
    }
    static void destroy(S &s) {
        free_ws(s);
        if (s.pin) Dev::release_pinned(s.pin);
        Dev::destroy_events(s.ev);
        s = S{};
    }
    std::mutex mu_;
    S idle_[kIdle];
    size_t n_ = 0;
};

}  // namespace bnk
