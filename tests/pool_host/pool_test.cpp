// Bookkeeping of the device memory pool, on the CPU: `pool_test NAME` runs one
// test of the table below and returns 0 when it holds.
#include "device_pool.h"

#include <cstdio>
#include <cstring>

using mxe::DevicePool;

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
    DevicePool pool;
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
    DevicePool pool;
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
    DevicePool pool;
    SimStream a;
    void *p = call(pool, sim::legacy, kMiB);
    CHECK(call(pool, a, kMiB) != p);
    CHECK(call(pool, sim::legacy, kMiB) == p);
    return true;
}

const struct {
    const char *name;
    bool (*run)();
} kTests[] = {
    {"streams_in_turn", streams_in_turn},
    {"finished_blocks_go_anywhere", finished_blocks_go_anywhere},
    {"legacy_blocks_stay", legacy_blocks_stay},
};

}  // namespace

int main(int argc, char **argv) {
    for (const auto &t : kTests) {
        if (argc < 2) puts(t.name);
        else if (!strcmp(argv[1], t.name)) return t.run() && sim::bad_frees == 0 ? 0 : 1;
    }
    return argc < 2 ? 0 : 2;
}
