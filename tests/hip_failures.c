/* Stands between libftk.so and the HIP runtime and lets chosen calls fail: for tests of the library's error paths.  Loaded
 * (RTLD_GLOBAL) before the runtime, so that the library's references find it first. */
#include <dlfcn.h>

enum { kOutOfMemory = 2, kUnknown = 999 };
static int create_at = 0, record_at = 0; /* the n-th call from now fails; 0: none does */

void hip_failures_set(int create, int record) {
    create_at = create;
    record_at = record;
}

static void* runtime;
int hip_failures_runtime(const char* path) { return (runtime = dlopen(path, RTLD_LAZY)) != 0; }
static void* next(const char* name) { return dlsym(runtime, name); }

int hipEventCreateWithFlags(void** event, unsigned flags) {
    static int (*real)(void**, unsigned);
    if (!real) *(void**)&real = next("hipEventCreateWithFlags");
    if (create_at > 0 && --create_at == 0) return kOutOfMemory;
    return real(event, flags);
}

int hipEventRecord(void* event, void* stream) {
    static int (*real)(void*, void*);
    if (!real) *(void**)&real = next("hipEventRecord");
    if (record_at > 0 && --record_at == 0) return kUnknown;
    return real(event, stream);
}
