/* Stands before hipMallocAsync in a process that loads it first, globally: lets
 * the next allocations of at least `least` bytes fail as if the device were
 * full, `times` of them (-1: all), and counts them. */
#include <dlfcn.h>
#include <stddef.h>

#define OUT_OF_MEMORY 2                                 /* hipErrorOutOfMemory */

static int (*real)(void **, size_t, void *);
static size_t least;
static int times, failed;

int shim_runtime(const char *path) {
    void *h = dlopen(path, RTLD_LAZY | RTLD_NOLOAD);
    if (h) real = (int (*)(void **, size_t, void *))dlsym(h, "hipMallocAsync");
    return real != NULL;
}
void shim_fail(size_t bytes, int n) {
    least = bytes;
    times = n;
    failed = 0;
}
int shim_failed(void) { return failed; }

int hipMallocAsync(void **p, size_t bytes, void *stream) {
    if (times != 0 && bytes >= least) {
        if (times > 0) --times;
        ++failed;
        return OUT_OF_MEMORY;
    }
    return real(p, bytes, stream);
}
