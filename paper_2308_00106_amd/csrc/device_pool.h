// Device memory of one context, kept for reuse. A library call takes several
// workspaces and a fresh matrix about ten blocks; with calls of different sizes
// in turn, hipMallocAsync takes about 20 us a block and hipFreeAsync 60 to 100
// (9 us where only one size is ever asked for), more than most kernels here.
//
// Blocks are rounded up to an eighth of a power of two and reused by size, but
// never so that one stream waits for another's work: a block given back is
// reused on the stream of its last use, or anywhere once the event recorded
// there has passed; without such a block the call takes a new one. (Taking the
// newest block behind a wait, two streams that issued the same product in turn
// ran one after the other for good.) Blocks last used on the legacy stream
// carry no event and stay with it. What lies unused is bounded (kPoolKeep) and goes
// back to the runtime past that, when an allocation fails, and with the
// context: the oldest blocks that are free by now go first, and where they are
// not enough the block being given back, again without a stream waiting for
// another. While a stream is captured its blocks come from the runtime, as
// nodes of the graph, and so do those of the per-thread stream, whose handle
// does not say which stream it is.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <list>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace mxe {

constexpr size_t kPoolKeep = size_t(4) << 30;

class DevicePool {
  public:
    explicit DevicePool(size_t keep = kPoolKeep) : limit_(keep) {}
    DevicePool(const DevicePool &) = delete;
    DevicePool &operator=(const DevicePool &) = delete;
    // The owner has synchronized the device and made it current.
    ~DevicePool() {
        drop_all(nullptr);
        for (hipEvent_t e : events_) (void)hipEventDestroy(e);
    }

    hipError_t get(void **p, size_t bytes, hipStream_t s) {
        *p = nullptr;
        if (!ordered(s)) return hipMallocAsync(p, bytes, s);
        const size_t size = rounded(bytes);
        std::lock_guard<std::mutex> lk(mu_);
        auto by = by_size_.find(size);
        if (by != by_size_.end())
            for (auto it = by->second.rbegin(); it != by->second.rend(); ++it) {
                Free &f = **it;
                if (!free_on(f, s)) continue;
                *p = f.p;
                live_[f.p] = size;
                forget(*it);
                return hipSuccess;
            }
        hipError_t e = hipMallocAsync(p, size, s);
        if (e != hipSuccess && !free_.empty()) {             // make room
            (void)hipGetLastError();
            (void)hipDeviceSynchronize();
            drop_all(s);
            (void)hipStreamSynchronize(s);
            e = hipMallocAsync(p, size, s);
        }
        if (e == hipSuccess) live_[*p] = size;
        else *p = nullptr;
        return e;
    }

    // The block's last use was queued on s.
    void put(void *p, hipStream_t s) {
        std::lock_guard<std::mutex> lk(mu_);
        Free f{p, forget_live(p), legacy(s) ? kLegacy : kEvent, nullptr, s};
        const bool pooled = f.size > 0 && ordered(s);        // not in a capture
        if (pooled && make_room_for(f.size, s) && record(f)) keep(f);
        else if (!release(p, s) && pooled && (f.ev || record(f))) keep(f);
    }

    // No work on the block is queued any more.
    void put_idle(void *p) {
        std::lock_guard<std::mutex> lk(mu_);
        const Free f{p, forget_live(p), kIdle, nullptr, nullptr};
        if (f.size > 0 && make_room_for(f.size, nullptr)) keep(f);
        else if (!release(p, nullptr) && f.size > 0) keep(f);
    }

    // An event without timing, from those given back.
    hipError_t event(hipEvent_t *ev) {
        std::lock_guard<std::mutex> lk(mu_);
        if (events_.empty()) return hipEventCreateWithFlags(ev, hipEventDisableTiming);
        *ev = events_.back();
        events_.pop_back();
        return hipSuccess;
    }
    void put_event(hipEvent_t ev) {
        std::lock_guard<std::mutex> lk(mu_);
        events_.push_back(ev);
    }

  private:
    enum Kind { kIdle, kLegacy, kEvent };
    struct Free {
        void *p;
        size_t size;
        Kind kind;
        hipEvent_t ev;
        hipStream_t s;                                       // kEvent: where it was recorded
    };
    using Node = std::list<Free>::iterator;

    static bool legacy(hipStream_t s) { return s == nullptr || s == hipStreamLegacy; }
    static bool ordered(hipStream_t s) {
        if (legacy(s)) return true;
        if (s == hipStreamPerThread) return false;
        hipStreamCaptureStatus cs;
        if (hipStreamIsCapturing(s, &cs) == hipSuccess) return cs == hipStreamCaptureStatusNone;
        (void)hipGetLastError();
        return false;
    }
    static size_t rounded(size_t bytes) {
        size_t step = 256;
        while (step * 16 <= bytes) step *= 2;                // bytes in [8 step, 16 step)
        return (bytes + step - 1) / step * step;
    }
    // Whether s may use the block without waiting for another stream. The wait on
    // its own stream costs that stream nothing; it is there for a stream that was
    // made after the one of this handle was destroyed.
    static bool free_on(const Free &f, hipStream_t s) {
        if (f.kind == kIdle) return true;
        if (f.kind == kLegacy) return legacy(s);
        if (f.s == s) {
            if (hipStreamWaitEvent(s, f.ev, 0) == hipSuccess) return true;
            (void)hipGetLastError();                         // the next launch is not to report it
        }
        if (hipEventQuery(f.ev) == hipSuccess) return true;
        (void)hipGetLastError();                             // hipErrorNotReady
        return false;
    }
    // bytes of a block handed out, 0 for one that is not the pool's
    size_t forget_live(void *p) {
        auto it = live_.find(p);
        if (it == live_.end()) return 0;
        const size_t size = it->second;
        live_.erase(it);
        return size;
    }
    static bool release(void *p, hipStream_t s) {
        if (hipFreeAsync(p, s) == hipSuccess) return true;
        (void)hipGetLastError();
        return false;
    }
    bool record(Free &f) {
        if (f.kind != kEvent) return true;
        if (!events_.empty()) {
            f.ev = events_.back();
            events_.pop_back();
        } else if (hipEventCreateWithFlags(&f.ev, hipEventDisableTiming) != hipSuccess) {
            f.ev = nullptr;
        }
        if (f.ev && hipEventRecord(f.ev, f.s) == hipSuccess) return true;
        (void)hipGetLastError();
        if (f.ev) events_.push_back(f.ev);
        f.ev = nullptr;
        return false;
    }
    // Frees the oldest blocks until `size` more bytes stay within the limit. A
    // block of the legacy stream is freed there, any other on s if s may use it.
    bool make_room_for(size_t size, hipStream_t s) {
        if (size > limit_) return false;
        for (Node it = free_.begin(); kept_ + size > limit_ && it != free_.end();) {
            const Node at = it++;
            const hipStream_t on = at->kind == kLegacy ? nullptr : s;
            if (free_on(*at, on) && release(at->p, on)) forget(at);
        }
        return kept_ + size <= limit_;
    }
    void keep(const Free &f) {
        free_.push_back(f);
        by_size_[f.size].push_back(std::prev(free_.end()));
        kept_ += f.size;
    }
    void forget(Node at) {
        auto by = by_size_.find(at->size);
        auto &v = by->second;
        for (size_t i = 0; i < v.size(); ++i)
            if (v[i] == at) {
                v.erase(v.begin() + i);
                break;
            }
        if (v.empty()) by_size_.erase(by);
        kept_ -= at->size;
        if (at->ev) events_.push_back(at->ev);
        free_.erase(at);
    }
    // Every use of the blocks has ended.
    void drop_all(hipStream_t s) {
        for (Node it = free_.begin(); it != free_.end();) {
            const Node at = it++;
            if (release(at->p, s)) forget(at);
        }
    }

    std::mutex mu_;
    std::unordered_map<void *, size_t> live_;                // blocks handed out
    std::list<Free> free_;                                   // oldest first
    std::map<size_t, std::vector<Node>> by_size_;
    std::vector<hipEvent_t> events_;
    const size_t limit_;
    size_t kept_ = 0;                                        // bytes of free_
};

}  // namespace mxe
