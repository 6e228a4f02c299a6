// Bookkeeping of the device memory pool, on the CPU: `pool_test NAME` runs one
// test of the table below and returns 0 when it holds.
#include "device_pool.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

using mxe::DevicePool;

// the host's own allocations fail once `allocations_left` has run out (-1: never)
static int allocations_left = -1;
void *operator new(size_t n) {
    if (allocations_left == 0) throw std::bad_alloc();
    if (allocations_left > 0) --allocations_left;
    if (void *p = malloc(n)) return p;
    throw std::bad_alloc();
}
int sim::pause_host_failures() {
    const int left = allocations_left;
    allocations_left = -1;
    return left;
}
void sim::resume_host_failures(int left) { allocations_left = left; }
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

#define CHECK(c)                                                     \
    do {                                                             \
        if (!(c)) {                                                  \
            fprintf(stderr, "line %d: %s\n", __LINE__, #c);          \
            return false;                                            \
        }                                                            \
    } while (0)

namespace {

constexpr size_t kMiB = size_t(1) << 20;

void work(SimStream &s) { ++s.queued; }
void finish(SimStream &s) { s.done = s.queued; }

// A call on s that takes a workspace.
void *call(DevicePool &pool, SimStream &s, size_t bytes) {
    void *p = nullptr;
    if (pool.get(&p, bytes, &s) != hipSuccess) return nullptr;
    work(s);
    pool.put(p, &s);
    return p;
}

// Two streams that issue calls of the same size in turn, none of them finished:
// neither waits for the other, and after the first two no memory is taken.
bool streams_in_turn() {
    DevicePool pool(0);
    SimStream a, b;
    void *pa = call(pool, a, kMiB), *pb = call(pool, b, kMiB);
    CHECK(pa && pb && pa != pb);
    for (int i = 0; i < 10; ++i) {
        CHECK(call(pool, a, kMiB) == pa);
        CHECK(call(pool, b, kMiB) == pb);
    }
    CHECK(a.waited_for.empty() && b.waited_for.empty());
    CHECK(sim::mallocs == 2 && sim::last == hipSuccess);
    return true;
}

// A block whose last use has finished goes to any stream, behind a newer one
// that is still in use; so does an idle one.
bool finished_blocks_go_anywhere() {
    DevicePool pool(0);
    SimStream a, b, c;
    void *pa = call(pool, a, kMiB), *pb = call(pool, b, kMiB);
    CHECK(pa != pb);
    finish(a);
    CHECK(call(pool, c, kMiB) == pa);
    CHECK(c.waited_for.empty());
    void *p;
    CHECK(pool.get(&p, 2 * kMiB, &a) == hipSuccess);
    pool.put_idle(p);
    CHECK(call(pool, c, 2 * kMiB) == p);
    return true;
}

// What was last used on the legacy stream stays with it.
bool legacy_blocks_stay() {
    DevicePool pool(0);
    SimStream a;
    void *p = call(pool, sim::legacy, kMiB);
    CHECK(call(pool, a, kMiB) != p);
    CHECK(call(pool, sim::legacy, kMiB) == p);
    return true;
}

// What lies unused stays within the limit whatever stream gives blocks back,
// and none waits for another: legacy blocks go on the legacy stream, blocks in
// use elsewhere are left alone.
bool limit_of_unused_blocks() {
    DevicePool pool(0, 4 * kMiB);
    SimStream a, b;
    std::vector<void *> taken(8);
    for (auto &p : taken) CHECK(pool.get(&p, kMiB, nullptr) == hipSuccess);
    work(sim::legacy);
    for (int i = 0; i < 3; ++i) pool.put(taken[i], nullptr);
    for (int i = 3; i < 8; ++i) pool.put(taken[i], &a);
    CHECK(sim::held <= 4 * kMiB);
    for (size_t i = 0; i < sim::freed_on.size(); ++i)
        if (sim::freed_on[i].first == taken[0]) CHECK(sim::freed_on[i].second == &sim::legacy);
    for (int i = 0; i < 6; ++i) {                      // more of another stream, a's not finished
        work(a);
        void *p;
        CHECK(pool.get(&p, (i % 3 + 1) * kMiB, &b) == hipSuccess);
        work(b);
        pool.put(p, &b);
        CHECK(sim::held <= 4 * kMiB);
    }
    CHECK(a.waited_for.empty() && b.waited_for.empty() && sim::legacy.waited_for.empty());
    void *big;                                         // larger than the limit: not kept, nothing else dropped
    const size_t before = sim::held;
    CHECK(pool.get(&big, 16 * kMiB, &b) == hipSuccess);
    pool.put(big, &b);
    CHECK(sim::held == before);
    return true;
}

// Blocks of the legacy stream that fill the limit make way for those of others.
bool legacy_blocks_make_way() {
    DevicePool pool(0, 4 * kMiB);
    SimStream a;
    void *p[4];
    for (auto &q : p) CHECK(pool.get(&q, kMiB, nullptr) == hipSuccess);
    for (auto &q : p) pool.put(q, nullptr);
    void *first = call(pool, a, kMiB);
    CHECK(call(pool, a, kMiB) == first && sim::held == 4 * kMiB);
    CHECK(sim::freed_on.size() == 1 && sim::freed_on[0] == std::make_pair(p[0], &sim::legacy));
    return true;
}

// The limit holds for blocks given back idle too, and where every older block
// is still in use.
bool limit_where_all_are_in_use() {
    DevicePool pool(0, 2 * kMiB);
    SimStream a, b;
    void *p[4];
    for (auto &q : p) CHECK(pool.get(&q, kMiB, &a) == hipSuccess);
    work(a);
    pool.put(p[0], &a);
    pool.put(p[1], &a);
    CHECK(sim::held == 4 * kMiB);
    work(b);
    pool.put(p[2], &b);
    CHECK(sim::held == 3 * kMiB);
    CHECK(sim::freed_on.back() == std::make_pair(p[2], &b));
    pool.put_idle(p[3]);
    CHECK(sim::held == 2 * kMiB && b.waited_for.empty() && sim::legacy.waited_for.empty());
    return true;
}

// A failing runtime call leaves no error behind and loses no block.
bool failing_calls() {
    DevicePool pool(0, 2 * kMiB);
    SimStream a;
    void *p[3];
    for (auto &q : p) CHECK(pool.get(&q, kMiB, &a) == hipSuccess);
    pool.put(p[0], &a);
    pool.put(p[1], &a);
    finish(a);
    sim::fail_free = true;
    pool.put(p[2], &a);
    CHECK(sim::last == hipSuccess);
    sim::fail_free = false;
    sim::fail_wait = true;
    void *q = nullptr;
    CHECK(pool.get(&q, kMiB, &a) == hipSuccess && sim::last == hipSuccess && sim::mallocs == 3);
    sim::fail_wait = false;
    pool.put(q, &a);
    work(a);                                           // at the limit, and the runtime refuses the block
    sim::fail_free = true;
    CHECK(pool.get(&q, 2 * kMiB, &a) == hipSuccess);
    pool.put(q, &a);
    sim::fail_free = false;
    CHECK(call(pool, a, 2 * kMiB) == q && sim::last == hipSuccess);
    return true;
}

// An allocation that fails gets back what lies unused in every context of its
// device, in use or not, but not another device's, and leaves no error behind.
bool room_from_other_contexts() {
    DevicePool one(0), two(0), other(1);
    SimStream a, b;
    call(one, a, 4 * kMiB);
    call(two, b, 3 * kMiB);
    call(two, sim::legacy, 2 * kMiB);
    call(other, a, kMiB);
    sim::capacity = 10 * kMiB;
    void *p = nullptr;
    CHECK(one.get(&p, 8 * kMiB, &a) == hipSuccess && p);
    CHECK(sim::held == 9 * kMiB && sim::device_syncs == 0 && sim::trims == 1);
    CHECK(sim::freed_on.size() == 3 && sim::freed_on.back().second == &sim::legacy);
    void *q = p;
    CHECK(two.get(&q, 8 * kMiB, &b) == hipErrorOutOfMemory && !q && sim::last == hipSuccess);
    one.put(p, &a);
    CHECK(two.get(&q, 8 * kMiB, hipStreamPerThread) == hipSuccess);        // not a pooled stream
    CHECK(sim::held == 9 * kMiB);
    two.put(q, hipStreamPerThread);
    CHECK(sim::held == kMiB);
    return true;
}

// A block that the caller can do without waits for nothing: it gets back what
// is free by now and no more.
bool optional_blocks_wait_for_nothing() {
    DevicePool pool(0);
    SimStream a, b;
    call(pool, a, 4 * kMiB);
    call(pool, b, 2 * kMiB);
    finish(a);
    sim::capacity = 8 * kMiB;
    void *p;
    CHECK(pool.get(&p, 5 * kMiB, &a, false, true) == hipSuccess && sim::held == 7 * kMiB);
    pool.put(p, &a);
    CHECK(pool.get(&p, 8 * kMiB, &a, false, true) == hipErrorOutOfMemory && sim::last == hipSuccess);
    CHECK(sim::event_waits == 0 && sim::device_syncs == 0 && sim::trims == 0 && a.waited_for.empty());
    return true;
}

// A call in a capture takes its block from the runtime and asks for no room.
bool no_room_in_a_capture() {
    DevicePool pool(0);
    SimStream a, b;
    call(pool, a, 4 * kMiB);
    sim::capacity = 4 * kMiB;
    b.capturing = true;
    void *p;
    CHECK(pool.get(&p, 4 * kMiB, &b) == hipErrorOutOfMemory && sim::last == hipSuccess);
    CHECK(sim::frees == 0 && sim::event_waits == 0 && sim::trims == 0);
    return true;
}

// Memory of a budget takes no more than its pages, and so does any block where
// the device has no room for the rounded size.
bool counted_blocks_fit() {
    for (size_t bytes : {size_t(1), size_t(255), size_t(257), size_t(5000), size_t(100'001), 9 * kMiB + 1, 1000 * kMiB + 77}) {
        DevicePool pool(0);
        SimStream a;
        void *p, *q;
        CHECK(pool.get(&p, bytes, &a, true) == hipSuccess);
        CHECK(sim::held >= bytes && sim::held - bytes < (bytes < 32768 ? 256 : 4096));
        pool.put(p, &a);
        CHECK(pool.get(&q, bytes, &a, true) == hipSuccess && p == q);
        pool.put(q, &a);
    }
    CHECK(sim::held == 0);
    DevicePool pool(0);
    SimStream a;
    sim::capacity = 9 * kMiB + 4096;
    void *p = nullptr;
    CHECK(pool.get(&p, 9 * kMiB + 1, &a) == hipSuccess && sim::held == 9 * kMiB + 4096);
    pool.put(p, &a);
    finish(a);
    CHECK(pool.get(&p, 9 * kMiB + 1, &a) == hipSuccess && sim::last == hipSuccess);
    pool.put(p, &a);
    return true;
}

// Without host memory for the bookkeeping nothing throws and no block is lost.
bool no_host_memory() {
    for (int left = 0; left < 12; ++left) {
        {
            DevicePool pool(0);
            SimStream a;
            void *p[3], *q = nullptr;
            for (auto &x : p) CHECK(pool.get(&x, kMiB, &a) == hipSuccess);
            hipEvent_t ev;
            CHECK(pool.event(&ev) == hipSuccess);
            sim::freed_on.reserve(100);
            allocations_left = left;
            pool.put(p[0], &a);
            pool.put(p[1], nullptr);
            pool.put_idle(p[2]);
            pool.put_event(ev);
            allocations_left = -1;
            work(a);
            for (int i = 0; i < 2; ++i) {
                allocations_left = left;
                const bool got = pool.get(&q, kMiB, &a) == hipSuccess;
                allocations_left = -1;
                CHECK(got == (q != nullptr));
                if (got) pool.put(q, &a);
            }
        }
        CHECK(sim::held == 0 && sim::events == 0);
    }
    return true;
}

// Everything goes back with the pool, events too.
bool all_returned() {
    {
        DevicePool pool(0);
        SimStream a;
        for (size_t i = 1; i < 6; ++i) call(pool, a, i * kMiB);
        call(pool, sim::legacy, kMiB);
        CHECK(sim::held > 0);
    }
    CHECK(sim::held == 0 && sim::events == 0);
    return true;
}

const struct {
    const char *name;
    bool (*run)();
} kTests[] = {
    {"streams_in_turn", streams_in_turn},
    {"finished_blocks_go_anywhere", finished_blocks_go_anywhere},
    {"legacy_blocks_stay", legacy_blocks_stay},
    {"limit_of_unused_blocks", limit_of_unused_blocks},
    {"legacy_blocks_make_way", legacy_blocks_make_way},
    {"limit_where_all_are_in_use", limit_where_all_are_in_use},
    {"failing_calls", failing_calls},
    {"room_from_other_contexts", room_from_other_contexts},
    {"optional_blocks_wait_for_nothing", optional_blocks_wait_for_nothing},
    {"no_room_in_a_capture", no_room_in_a_capture},
    {"counted_blocks_fit", counted_blocks_fit},
    {"no_host_memory", no_host_memory},
    {"all_returned", all_returned},
};

}  // namespace

int main(int argc, char **argv) {
    for (const auto &t : kTests) {
        if (argc < 2) puts(t.name);
        else if (!strcmp(argv[1], t.name)) return t.run() && sim::bad_frees == 0 && sim::unsafe_calls == 0 && sim::mode == hipStreamCaptureModeGlobal ? 0 : 1;
    }
    return argc < 2 ? 0 : 2;
}
