// A stand-in for the few HIP calls that the device memory pool makes, so that
// its bookkeeping is tested on the CPU: streams with a count of work queued and
// done, events that remember a point of one, memory that is counted. Tests
// steer it through namespace sim.
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>

#include <map>
#include <utility>
#include <vector>

enum hipError_t {
    hipSuccess = 0,
    hipErrorInvalidValue = 1,
    hipErrorOutOfMemory = 2,
    hipErrorNotReady = 600,
    hipErrorStreamCaptureUnsupported = 900
};
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
enum hipStreamCaptureMode {
    hipStreamCaptureModeGlobal = 0,
    hipStreamCaptureModeThreadLocal = 1,
    hipStreamCaptureModeRelaxed = 2
};
constexpr unsigned hipEventDisableTiming = 2;

struct SimStream {
    uint64_t queued = 0, done = 0;                     // work items
    bool capturing = false;
    std::vector<const SimStream *> waited_for;         // streams whose unfinished work it was made to wait for
};
struct SimEvent {
    const SimStream *s = nullptr;
    uint64_t at = 0;
};
using hipStream_t = SimStream *;
using hipEvent_t = SimEvent *;
using hipMemPool_t = int *;

namespace sim {
inline SimStream legacy, per_thread;
inline size_t capacity = ~size_t(0), held = 0;         // bytes of the device, bytes allocated
inline std::map<void *, size_t> blocks;
inline std::vector<std::pair<void *, SimStream *>> freed_on;
inline int mallocs = 0, frees = 0, bad_frees = 0, device_syncs = 0, event_waits = 0, events = 0, trims = 0;
inline bool fail_free = false, fail_wait = false;
inline int device = 0, unsafe_calls = 0;               // calls that would end a capture
inline hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
inline hipError_t last = hipSuccess;
inline hipError_t err(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}
inline SimStream *of(SimStream *s);
int pause_host_failures();                             // the stand-in's own memory does not fail
void resume_host_failures(int left);
}  // namespace sim

#define hipStreamLegacy (&sim::legacy)
#define hipStreamPerThread (&sim::per_thread)
inline SimStream *sim::of(SimStream *s) { return s ? s : &legacy; }

inline hipError_t hipGetLastError() {
    const hipError_t e = sim::last;
    sim::last = hipSuccess;
    return e;
}
inline hipError_t hipGetDevice(int *d) {
    *d = sim::device;
    return hipSuccess;
}
inline hipError_t hipMallocAsync(void **p, size_t bytes, hipStream_t) {
    if (bytes > sim::capacity - sim::held) return sim::err(hipErrorOutOfMemory);
    *p = malloc(1);
    const int left = sim::pause_host_failures();
    sim::blocks[*p] = bytes;
    sim::resume_host_failures(left);
    sim::held += bytes;
    ++sim::mallocs;
    return hipSuccess;
}
inline hipError_t hipFreeAsync(void *p, hipStream_t s) {
    if (sim::fail_free) return sim::err(hipErrorStreamCaptureUnsupported);
    auto it = sim::blocks.find(p);
    if (it == sim::blocks.end()) {
        ++sim::bad_frees;
        return sim::err(hipErrorInvalidValue);
    }
    sim::held -= it->second;
    sim::blocks.erase(it);
    sim::freed_on.push_back({p, sim::of(s)});
    ++sim::frees;
    return hipSuccess;                                 // the address is not reused: p stays allocated
}
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *cs) {
    *cs = sim::of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
    if (sim::mode != hipStreamCaptureModeRelaxed) ++sim::unsafe_calls;
    sim::of(s)->done = sim::of(s)->queued;
    return hipSuccess;
}
inline hipError_t hipDeviceSynchronize() {
    ++sim::device_syncs;
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    const int left = sim::pause_host_failures();
    *e = new SimEvent();
    sim::resume_host_failures(left);
    ++sim::events;
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    --sim::events;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    *e = SimEvent{sim::of(s), sim::of(s)->queued};
    return hipSuccess;
}
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
    std::swap(*m, sim::mode);
    return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) {
    if (sim::mode != hipStreamCaptureModeRelaxed) ++sim::unsafe_calls;
    return !e->s || e->s->done >= e->at ? hipSuccess : sim::err(hipErrorNotReady);
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    if (sim::mode != hipStreamCaptureModeRelaxed) ++sim::unsafe_calls;
    ++sim::event_waits;
    if (e->s && e->s->done < e->at) const_cast<SimStream *>(e->s)->done = e->at;
    return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (sim::fail_wait) return sim::err(hipErrorInvalidValue);
    if (e->s && e->s != sim::of(s) && e->s->done < e->at) sim::of(s)->waited_for.push_back(e->s);
    return hipSuccess;
}
inline hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *, int) { return hipSuccess; }
inline hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
    if (sim::mode != hipStreamCaptureModeRelaxed) ++sim::unsafe_calls;
    ++sim::trims;
    return hipSuccess;
}
