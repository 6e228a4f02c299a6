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
// carry no event and stay with it. What lies unused is bounded by kPoolKeep bytes
// and goes back to the runtime past that, when an allocation fails, and with
// the context. While a stream is captured its blocks come from the runtime, as
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
    DevicePool() = default;
    DevicePool(const DevicePool &) = delete;
    DevicePool &operator=(const DevicePool &) = delete;
    // The owner has synchronized the device and made it current.
    ~DevicePool() {
        for (auto &f : free_) give_back(f, nullptr);
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
                kept_ -= size;
                if (f.ev) events_.push_back(f.ev);
                const auto node = *it;
                by->second.erase(std::next(it).base());
                free_.erase(node);
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
        auto it = live_.find(p);
        if (it == live_.end() || !ordered(s)) {              // captured, or not the pool's
            if (it != live_.end()) live_.erase(it);
            (void)hipFreeAsync(p, s);
            return;
        }
        Free f{p, it->second, kLegacy, nullptr, s};
        live_.erase(it);
        if (!legacy(s)) {
            f.kind = kEvent;
            if (!events_.empty()) {
                f.ev = events_.back();
                events_.pop_back();
            } else if (hipEventCreateWithFlags(&f.ev, hipEventDisableTiming) != hipSuccess) {
                f.ev = nullptr;
            }
            if (!f.ev || hipEventRecord(f.ev, s) != hipSuccess) {
                if (f.ev) events_.push_back(f.ev);
                (void)hipFreeAsync(p, s);
                return;
            }
        }
        keep(f, s);
    }

    // No work on the block is queued any more.
    void put_idle(void *p) {
        std::lock_guard<std::mutex> lk(mu_);
        auto it = live_.find(p);
        if (it == live_.end()) {
            (void)hipFreeAsync(p, nullptr);
            return;
        }
        Free f{p, it->second, kIdle, nullptr, nullptr};
        live_.erase(it);
        keep(f, nullptr);
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
        if ((f.s == s && hipStreamWaitEvent(s, f.ev, 0) == hipSuccess) || hipEventQuery(f.ev) == hipSuccess)
            return true;
        (void)hipGetLastError();                             // hipErrorNotReady
        return false;
    }
    void keep(const Free &f, hipStream_t s) {
        free_.push_back(f);
        by_size_[f.size].push_back(std::prev(free_.end()));
        kept_ += f.size;
        // oldest first; on a stream ordered behind each block's last use
        for (Node it = free_.begin(); kept_ > kPoolKeep && it != free_.end();) {
            const Node at = it++;
            if (at->kind == kLegacy && !legacy(s)) continue;
            if (at->kind == kEvent && hipStreamWaitEvent(s, at->ev, 0) != hipSuccess) continue;
            forget(at);
            give_back(*at, s);
            free_.erase(at);
        }
    }
    void forget(Node at) {
        auto &v = by_size_[at->size];
        for (size_t i = 0; i < v.size(); ++i)
            if (v[i] == at) {
                v.erase(v.begin() + i);
                break;
            }
        kept_ -= at->size;
    }
    void give_back(Free &f, hipStream_t s) {
        (void)hipFreeAsync(f.p, s);
        if (f.ev) events_.push_back(f.ev);
    }
    void drop_all(hipStream_t s) {
        for (auto &f : free_) give_back(f, s);
        free_.clear();
        by_size_.clear();
        kept_ = 0;
    }

    std::mutex mu_;
    std::unordered_map<void *, size_t> live_;                // blocks handed out
    std::list<Free> free_;                                   // oldest first
    std::map<size_t, std::vector<Node>> by_size_;
    std::vector<hipEvent_t> events_;
    size_t kept_ = 0;
};

}  // namespace mxe
