/* Refuses device allocations of one size, FAIL_BYTES, and counts them: loaded
 * before the library with global symbols, its hipMalloc is the one that the
 * library calls; every other size goes on to the runtime. */
#include <dlfcn.h>
#include <stddef.h>

int refused = 0;

int hipMalloc(void** ptr, size_t bytes)
{
    static int (*real)(void**, size_t) = NULL;
    if (bytes == (size_t)FAIL_BYTES) {
        ++refused;
        return 2; /* hipErrorOutOfMemory */
    }
    if (!real) {
        void* h = dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_LOCAL);
        if (h) *(void**)&real = dlsym(h, "hipMalloc");
        if (!real) return 999;
    }
    return real(ptr, bytes);
}
