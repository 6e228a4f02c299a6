// Device memory of one context, kept for reuse. A library call takes several
// workspaces and a fresh matrix about ten blocks; with calls of different sizes
// in turn, hipMallocAsync takes about 20 us a block and hipFreeAsync 60 to 100
// (9 us where only one size is ever asked for), more than most kernels here.
//
// Blocks are rounded up to an eighth of a power of two, where a budget counts
// them or memory is short to whole pages only, and reused by size, but never
// so that one stream waits for another's work: a block given back is reused on
// the stream of its last use, or anywhere once the event recorded there has
// passed; without such a block the call takes a new one. (Taking the newest
// block behind a wait, two streams that issued the same product in turn ran
// one after the other for good: 400K skewed FP64 rows in their original order
// took 69 us a product on two streams and 55 on one, now 44 and 55.) Blocks
// last used on the legacy stream carry no event and stay with it. What lies
// unused is bounded (kPoolKeep) and goes back to the runtime past that, when
// an allocation fails, and with the context: the oldest blocks that are free
// by now go first, and where they are not enough the block being given back,
// again without a stream waiting for another. An allocation that fails takes
// back what lies unused in every context of the device. While a stream is
// captured its blocks come from the runtime, as nodes of the graph, and so do
// those of the per-thread stream, whose handle does not say which stream it
// is.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <list>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace mxe {

constexpr size_t kPoolKeep = size_t(4) << 30;

class DevicePool {
  public:
    explicit DevicePool(int device, size_t keep = kPoolKeep) : device_(device), limit_(keep) {
        Registry &r = registry();
        std::lock_guard<std::mutex> lk(r.mu);
        r.pools.push_back(this);
    }
    DevicePool(const DevicePool &) = delete;
    DevicePool &operator=(const DevicePool &) = delete;
    // The owner has synchronized the device and made it current.
    ~DevicePool() {
        {
            Registry &r = registry();
            std::lock_guard<std::mutex> lk(r.mu);
            r.pools.remove(this);
        }
        drop(nullptr, true);
        for (hipEvent_t e : events_) (void)hipEventDestroy(e);
    }

    // counted: the bytes are held against a budget. optional: the caller can do
    // without, so the call waits for nothing.
    hipError_t get(void **p, size_t bytes, hipStream_t s, bool counted = false, bool optional = false) {
        *p = nullptr;
        const bool pooled = ordered(s);
        size_t size = !pooled ? bytes : counted ? paged(bytes) : rounded(bytes);
        if (pooled && take(p, size, s)) return hipSuccess;
        hipError_t e = hipMallocAsync(p, size, s);
        // a capture neither waits nor frees
        if (e == hipErrorOutOfMemory && (pooled || s == hipStreamPerThread) && !capturing(s)) {
            (void)hipGetLastError();
            if (optional) drop_unused(s);
            else make_room(s);
            e = hipMallocAsync(p, size, s);
            if (e == hipErrorOutOfMemory && pooled && size > paged(bytes)) {
                (void)hipGetLastError();
                size = paged(bytes);
                e = hipMallocAsync(p, size, s);
            }
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();                         // the next launch is not to report it
            *p = nullptr;
        } else if (pooled && !hand_out(*p, size)) {
            (void)release(*p, s);
            *p = nullptr;
            e = hipErrorOutOfMemory;
        }
        return e;
    }

    // The block's last use was queued on s.
    void put(void *p, hipStream_t s) {
        std::lock_guard<std::mutex> lk(mu_);
        Free f{p, forget_live(p), legacy(s) ? kLegacy : kEvent, nullptr, s};
        const bool pooled = f.size > 0 && ordered(s);        // not in a capture
        if (pooled && make_room_for(f.size, s) && record(f) && keep(f)) return;
        if (!release(p, s) && pooled && (f.ev || record(f)) && keep(f)) return;
        if (f.ev) give_event(f.ev);
    }

    // No work on the block is queued any more.
    void put_idle(void *p) {
        std::lock_guard<std::mutex> lk(mu_);
        const Free f{p, forget_live(p), kIdle, nullptr, nullptr};
        if (f.size > 0 && make_room_for(f.size, nullptr) && keep(f)) return;
        if (!release(p, nullptr) && f.size > 0) (void)keep(f);
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
        give_event(ev);
    }

    static bool legacy(hipStream_t s) { return s == nullptr || s == hipStreamLegacy; }
    static bool capturing(hipStream_t s) {
        if (legacy(s)) return false;                         // it cannot be captured
        hipStreamCaptureStatus cs;
        if (hipStreamIsCapturing(s, &cs) == hipSuccess) return cs != hipStreamCaptureStatusNone;
        (void)hipGetLastError();
        return true;
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
    // every context's pool; never destroyed, contexts may outlive static objects
    struct Registry {
        std::mutex mu;                                       // taken before any pool's
        std::list<DevicePool *> pools;
    };
    static Registry &registry() {
        static Registry *r = new Registry;
        return *r;
    }

    static bool ordered(hipStream_t s) {
        if (legacy(s)) return true;
        return s != hipStreamPerThread && !capturing(s);
    }
    static size_t paged(size_t bytes) {                      // small blocks to 256 bytes
        const size_t step = bytes < 32768 ? 256 : 4096;
        return (bytes + step - 1) / step * step;
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
        return passed(f.ev);
    }
    // The thread's relaxed capture mode: in the others asking for an event or
    // waiting ends a capture that is under way on any stream.
    class Relaxed {
      public:
        Relaxed() : set_(hipThreadExchangeStreamCaptureMode(&mode_) == hipSuccess) {}
        ~Relaxed() {
            if (set_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
        }
        Relaxed(const Relaxed &) = delete;
        Relaxed &operator=(const Relaxed &) = delete;

      private:
        hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
        const bool set_;
    };
    static bool passed(hipEvent_t ev) {
        const Relaxed r;
        if (hipEventQuery(ev) == hipSuccess) return true;
        (void)hipGetLastError();                             // hipErrorNotReady
        return false;
    }
    // A block of this size that s may use without waiting, the newest.
    bool take(void **p, size_t size, hipStream_t s) {
        std::lock_guard<std::mutex> lk(mu_);
        auto by = by_size_.find(size);
        if (by == by_size_.end()) return false;
        for (auto it = by->second.rbegin(); it != by->second.rend(); ++it) {
            if (!free_on(**it, s)) continue;
            try {
                live_[(*it)->p] = size;
            } catch (const std::bad_alloc &) {
                return false;
            }
            *p = (*it)->p;
            forget(*it);
            return true;
        }
        return false;
    }
    // Gives the device back what lies unused in its pools, for an allocation on s,
    // and then what the runtime itself holds unused. Waits for the blocks' last
    // uses, not for the device.
    void make_room(hipStream_t s) {
        const Relaxed relaxed;
        Registry &r = registry();
        {
            std::lock_guard<std::mutex> lk(r.mu);
            for (DevicePool *q : r.pools)
                if (q->device_ == device_) q->drop(s, false);
        }
        hipMemPool_t runtime;
        if (hipStreamSynchronize(nullptr) != hipSuccess || hipStreamSynchronize(s) != hipSuccess ||
            hipDeviceGetDefaultMemPool(&runtime, device_) != hipSuccess || hipMemPoolTrimTo(runtime, 0) != hipSuccess)
            (void)hipGetLastError();
    }
    // The unused blocks that s, or the legacy stream, may free without waiting.
    void drop_unused(hipStream_t s) {
        std::lock_guard<std::mutex> lk(mu_);
        for (Node it = free_.begin(); it != free_.end();) {
            const Node at = it++;
            const hipStream_t on = at->kind == kLegacy ? nullptr : s;
            if (free_on(*at, on) && release(at->p, on)) forget(at);
        }
    }
    // Every unused block; ended: no use of one is still running.
    void drop(hipStream_t s, bool ended) {
        std::lock_guard<std::mutex> lk(mu_);
        for (Node it = free_.begin(); it != free_.end();) {
            const Node at = it++;
            if (!ended && at->kind == kEvent && hipEventSynchronize(at->ev) != hipSuccess) (void)hipGetLastError();
            else if (release(at->p, at->kind == kLegacy ? nullptr : s)) forget(at);
        }
    }
    // Calls end matrices and workspaces on their way out, so nothing here throws:
    // without host memory for its bookkeeping a block goes back to the runtime.
    bool hand_out(void *p, size_t size) {
        std::lock_guard<std::mutex> lk(mu_);
        try {
            live_[p] = size;
        } catch (const std::bad_alloc &) {
            return false;
        }
        return true;
    }
    bool keep(const Free &f) {
        try {
            free_.push_back(f);
        } catch (const std::bad_alloc &) {
            return false;
        }
        try {
            by_size_[f.size].push_back(std::prev(free_.end()));
        } catch (const std::bad_alloc &) {
            free_.pop_back();
            return false;
        }
        kept_ += f.size;
        return true;
    }
    void give_event(hipEvent_t ev) {
        try {
            events_.push_back(ev);
        } catch (const std::bad_alloc &) {
            (void)hipEventDestroy(ev);
        }
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
        if (f.ev) give_event(f.ev);
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
        if (at->ev) give_event(at->ev);
        free_.erase(at);
    }

    std::mutex mu_;
    std::unordered_map<void *, size_t> live_;                // blocks handed out
    std::list<Free> free_;                                   // oldest first
    std::map<size_t, std::vector<Node>> by_size_;
    std::vector<hipEvent_t> events_;
    const int device_;
    const size_t limit_;
    size_t kept_ = 0;                                        // bytes of free_
};

}  // namespace mxe
