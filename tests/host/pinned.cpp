// Pinned host memory of the C-ABI's host layer, without a GPU: the HIP calls
// that the layer makes are replaced by host memory that is counted.  Exit
// status 0 = every check held.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <condition_variable>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "dd_internal.h"

static std::mutex mu;
static std::set<void *> pinned;
static size_t most = 0, made = 0;

extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    std::lock_guard<std::mutex> lk(mu);
    *p = calloc(1, n);
    pinned.insert(*p);
    made++;
    if (pinned.size() > most) most = pinned.size();
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> lk(mu);
    if (!pinned.erase(p)) abort();
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipErrorInvalidValue; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorInvalidValue; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace dd {
#define STUB return hipErrorNoDevice
dd_status levelize_device(const dd_graph *, uint64_t, int32_t, dd_sched *, hipStream_t, char *, size_t) { return DD_EHIP; }
hipError_t launch_simulate(const dd_graph *, const dd_sched *, const dd_variants *, int64_t *, int64_t *, int64_t *, int,
                           hipStream_t) { STUB; }
hipError_t simulate_noalloc(const dd_graph *, const dd_sched *, const dd_variants *, int64_t *, int64_t *, int64_t *,
                            hipStream_t, size_t *, size_t *) { STUB; }
int split_width(const dd_sched *, const dd_variants *) { return 0; }
hipError_t launch_split(const dd_graph *, const dd_sched *, const dd_variants *, int64_t *, int64_t *, int64_t *, int,
                        hipStream_t) { STUB; }
void split_set_polls(int32_t) {}
hipError_t launch_breakdown(const dd_graph *, const dd_variants *, const uint8_t *, const int64_t *, const int64_t *,
                            int64_t *, hipStream_t) { STUB; }
hipError_t build_event_lists(const dd_graph *, EventLists *, hipStream_t) { STUB; }
void free_event_lists(EventLists *, hipStream_t) {}
hipError_t launch_sim_event(const dd_graph *, const EventLists &, const dd_variants *, int32_t, const uint8_t *,
                            const int32_t *, int32_t *, int64_t *, uint32_t **, int64_t *, int64_t *, int64_t *,
                            uint32_t *, hipStream_t) { STUB; }
}  // namespace dd

static int bad = 0;
#define EXPECT(c)                                                                  \
    do {                                                                           \
        if (!(c)) {                                                                \
            fprintf(stderr, "FAILED: %s (line %d): %zu made, %zu at once, %zu live\n", #c, __LINE__, made, most, \
                    pinned.size());                                                \
            bad++;                                                                 \
        }                                                                          \
    } while (0)

static void call() {
    int64_t ptr[1] = {0};
    dd_graph *g = nullptr;
    if (dd_graph_load(0, 1, ptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, &g) != DD_OK)
        abort();
    dd_graph_free(g);
}

int main() {
    // threads that come and go hand one block on
    for (int i = 0; i < 100; i++) std::thread(call).join();
    EXPECT(made <= 1 && pinned.size() <= 1);
    // as many blocks as threads that are in the library at once
    std::condition_variable cv;
    std::mutex m;
    int in = 0;
    std::vector<std::thread> ts;
    for (int i = 0; i < 8; i++)
        ts.emplace_back([&] {
            call();
            std::unique_lock<std::mutex> lk(m);
            if (++in == 8) cv.notify_all();
            cv.wait(lk, [&] { return in == 8; });
        });
    for (auto &t : ts) t.join();
    EXPECT(pinned.size() <= 8);
    for (int i = 0; i < 50; i++) std::thread(call).join();
    EXPECT(made <= 8);
    // given back on request, but for the blocks of living threads
    call();
    EXPECT(dd_release_cache() == DD_OK);
    EXPECT(pinned.size() == 1);
    call();
    EXPECT(pinned.size() == 1);
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}
