// Host side of dd_levelize without a GPU: launches do nothing, device memory
// is host memory, and the allocations past a limit fail.  Exit status 0 =
// every check held.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "dd_internal.h"

static size_t held = 0, limit = ~(size_t)0;

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace dd {
hipError_t dalloc(void **p, size_t bytes, hipStream_t) {
    *p = nullptr;
    if (held + bytes > limit) return hipErrorOutOfMemory;
    held += bytes;
    *p = malloc(16);                          // (never touched)
    return hipSuccess;
}
void dfree(void *p, hipStream_t) { free(p); }
hipError_t direct_buf(void **h, void **d) {
    static char buf[kDirectBytes];
    *h = *d = buf;
    return hipSuccess;
}
hipError_t scan_exclusive(const int64_t *, int64_t *, int64_t, hipStream_t) { return hipSuccess; }
ReadBack::ReadBack(hipStream_t s, size_t) : s_(s) {}
hipError_t ReadBack::add(void *, const void *, size_t) { return hipSuccess; }
hipError_t ReadBack::finish() { return hipSuccess; }
}  // namespace dd

static int bad = 0;
#define EXPECT(c)                                                                      \
    do {                                                                               \
        if (!(c)) {                                                                    \
            fprintf(stderr, "FAILED: %s (line %d, %d threads)\n", #c, __LINE__, threads); \
            bad++;                                                                     \
        }                                                                              \
    } while (0)

int main() {
    for (const int threads : {1, 16, 64, 300}) {
        dd_graph g;
        g.n = 100000;
        g.n_threads = threads;
        g.n_cross = 30000;
        char msg[64];
        // with room for everything: the one-variant kernel's records are there
        dd_sched all, some, none;
        held = 0;
        limit = ~(size_t)0;
        EXPECT(dd::levelize_device(&g, 1, DD_PHASES, &all, nullptr, msg, sizeof(msg)) == DD_OK && all.so_rec);
        // not quite: a schedule all the same
        const size_t most = held, recs = sizeof(dd::SoloRec) * (size_t)g.n;
        held = 0;
        limit = most - recs / 2;
        EXPECT(dd::levelize_device(&g, 1, DD_PHASES, &some, nullptr, msg, sizeof(msg)) == DD_OK && !some.so_rec);
        EXPECT(some.rec);
        // no more than that is given up
        held = 0;
        limit = most - recs * 2;
        EXPECT(dd::levelize_device(&g, 1, DD_PHASES, &none, nullptr, msg, sizeof(msg)) == DD_ENOMEM);
    }
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}
