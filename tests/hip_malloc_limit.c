/* Device allocations above a limit, or a chosen one, fail, for tests of what the
 * library does then.  Loaded with RTLD_GLOBAL before libpm.so, whose hipMalloc then resolves
 * here; the runtime's own makes the allocation. */
#include <dlfcn.h>
#include <stddef.h>

static size_t limit = ~(size_t)0, largest;

void malloc_limit(size_t bytes) {
    limit = bytes;
    largest = 0;
}
size_t malloc_largest(void) { return largest; } /* since the limit was set */

static long until = -1;
void malloc_fail(long nth) { until = nth; } /* 0: the next allocation */

int hipMalloc(void **p, size_t bytes) {
    static int (*real)(void **, size_t);
    if (bytes > limit || until-- == 0) return 2; /* hipErrorOutOfMemory */
    if (!real) {
        void *hip = dlopen("libamdhip64.so.7", RTLD_LAZY);
        if (!hip) return 1;
        *(void **)&real = dlsym(hip, "hipMalloc");
        if (!real) return 1;
    }
    if (bytes > largest) largest = bytes;
    return real(p, bytes);
}
