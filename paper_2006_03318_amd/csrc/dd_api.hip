// C-ABI of the dd library: handle management, argument checks, and the
// order in which the device passes of each call run.

#include <atomic>
#include <map>
#include <math.h>
#include <mutex>
#include <unordered_map>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "dd_internal.h"

namespace {

thread_local char g_err[512] = "";
std::atomic<uint64_t> g_next_id{1};

dd_status fail(dd_status s, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return s;
}

dd_status hip_fail(hipError_t e, const char *what) {
    return fail(e == hipErrorOutOfMemory ? DD_ENOMEM : DD_EHIP, "%s: %s", what,
                hipGetErrorString(e));
}

dd_status map_err_bits(uint32_t e) {
    using namespace dd;
    if (e & ERR_THREAD_RANGE) return fail(DD_EINVAL, "thread_id outside [0, n_threads)");
    if (e & ERR_PREV_RANGE) return fail(DD_EINVAL, "thread_prev outside [-1, n) or naming the task itself");
    if (e & ERR_NEG_TIME) return fail(DD_EINVAL, "negative duration or gap");
    if (e & ERR_PTR_ORDER) return fail(DD_EINVAL, "in_ptr is not non-decreasing");
    if (e & ERR_SRC_RANGE) return fail(DD_EINVAL, "in_src outside [0, n)");
    if (e & ERR_EDGE_CLS) return fail(DD_EINVAL, "edge class >= 64");
    if (e & ERR_SCALE) return fail(DD_EINVAL, "scale with p < 0 or q < 1");
    if (e & ERR_BIG_TIME) return fail(DD_ERANGE, "duration or gap >= 2^62 ns");
    if (e & ERR_PREV_THREAD) return fail(DD_ECHAIN, "thread_prev names a task on another thread");
    if (e & ERR_SUCC) return fail(DD_ECHAIN, "two tasks name the same thread_prev");
    if (e & ERR_HEADS) return fail(DD_ECHAIN, "a thread has more than one first task");
    if (e & ERR_CHAIN_CYCLE) return fail(DD_ECHAIN, "thread order loops");
    if (e & ERR_SELF_LOOP) return fail(DD_ECYCLE, "dependency from a task to itself");
    if (e & ERR_BACK_EDGE) return fail(DD_ECYCLE, "dependency goes backwards along one thread");
    if (e & ERR_KAHN_CYCLE) return fail(DD_ECYCLE, "dependencies plus thread order contain a cycle");
    return DD_OK;
}

template <class T>
hipError_t copy_in(T **dst, const T *src, size_t count, hipStream_t s) {
    hipError_t e = dd::dalloc_n(dst, count, s);
    if (e != hipSuccess) return e;
    if (count == 0) return hipSuccess;
    if (src) return hipMemcpyAsync(*dst, src, count * sizeof(T), hipMemcpyDefault, s);
    return hipMemsetAsync(*dst, 0, count * sizeof(T), s);
}

// memory that kernels on the current device may read in place: a copy queued
// on the call's stream would read it no earlier
// (align: their elements, as a copy would not have minded)
bool on_device(const void *p, size_t align = 1) {
    if (!p || reinterpret_cast<uintptr_t>(p) % align) return false;
    hipPointerAttribute_t at;
    int dev = 0;
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();             // host memory the runtime does not know
        return false;
    }
    return at.type == hipMemoryTypeDevice && hipGetDevice(&dev) == hipSuccess && at.device == dev;
}

void free_graph_arrays(dd_graph *g) {
    hipStream_t s = g->stream;
    dd::join_uses(g->uses, s);
    dd::dfree(g->thread_prev, s); dd::dfree(g->thread_id, s); dd::dfree(g->dur, s);
    dd::dfree(g->gap, s); dd::dfree(g->cls, s); dd::dfree(g->rank, s);
    dd::dfree(g->thread_base, s); dd::dfree(g->order, s); dd::dfree(g->xin_ptr, s);
    dd::dfree(g->xin_src, s); dd::dfree(g->xin_cls, s);
    dd::free_event_lists(&g->ev, s);
}

void free_sched_arrays(dd_sched *x) {
    hipStream_t s = x->stream;
    dd::join_uses(x->uses, s);
    dd::dfree(x->step_ptr, s); dd::dfree(x->pos_node, s); dd::dfree(x->node_step, s);
    dd::dfree(x->gat_rng, s); dd::dfree(x->gat_src, s); dd::dfree(x->gat_spos, s);
    dd::dfree(x->gat_cls, s); dd::dfree(x->gat_gap, s); dd::dfree(x->rec, s);
    dd::dfree(x->bat, s); dd::dfree(x->nbat, s); dd::dfree(x->so_rec, s);
}

}  // namespace

namespace dd {

// Device memory cache.  Released blocks wait in a free list keyed by
// (device, stream) and serve later requests on that stream only: work on
// one stream runs in order, so a block released there can be handed out
// again at once.  A cached block serves a request of up to its size and at
// least half of it.  New blocks come from hipMalloc; when that fails, every
// cached block of the device is returned and the allocation retried.
namespace {

struct CacheKey {
    int dev;
    hipStream_t s;
    bool operator<(const CacheKey &o) const { return dev != o.dev ? dev < o.dev : s < o.s; }
};
struct LiveBlock {
    size_t bytes;
    int dev;
};

std::mutex g_mu;
std::map<CacheKey, std::multimap<size_t, void *>> g_free;
std::unordered_map<void *, LiveBlock> g_live;

void release_cached(int dev) {   // caller holds g_mu; dev is the current device
    (void)hipDeviceSynchronize();  // work queued before a release may still read a block
    for (auto it = g_free.begin(); it != g_free.end();) {
        if (it->first.dev == dev) {
            for (auto &b : it->second) (void)hipFree(b.second);
            it = g_free.erase(it);
        } else {
            ++it;
        }
    }
}

}  // namespace

hipError_t dalloc(void **p, size_t bytes, hipStream_t s) {
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    bytes = (bytes + 511) & ~(size_t)511;
    if (bytes == 0) bytes = 512;
    std::lock_guard<std::mutex> lk(g_mu);
    auto fit = g_free.find(CacheKey{dev, s});
    if (fit != g_free.end()) {
        auto it = fit->second.lower_bound(bytes);
        if (it != fit->second.end() && it->first / 2 <= bytes) {
            *p = it->second;
            g_live[*p] = LiveBlock{it->first, dev};
            fit->second.erase(it);
            return hipSuccess;
        }
    }
    e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        release_cached(dev);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        return e;
    }
    g_live[*p] = LiveBlock{bytes, dev};
    return hipSuccess;
}

void dfree(void *p, hipStream_t s) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_live.find(p);
    if (it == g_live.end()) return;
    g_free[CacheKey{it->second.dev, s}].emplace(it->second.bytes, p);
    g_live.erase(it);
}

hipError_t note_use(ForeignUses &u, hipStream_t own, hipStream_t s) {
    if (s == own) return hipSuccess;
    std::lock_guard<std::mutex> lk(u.mu);
    hipEvent_t ev = nullptr;
    for (auto &x : u.ev)
        if (x.first == s) ev = x.second;
    if (!ev) {
        hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e != hipSuccess) return e;
        u.ev.emplace_back(s, ev);
    }
    // re-recording keeps the latest use: earlier work on s precedes it
    return hipEventRecord(ev, s);
}

void join_uses(ForeignUses &u, hipStream_t own) {
    std::lock_guard<std::mutex> lk(u.mu);
    for (auto &x : u.ev) {
        (void)hipStreamWaitEvent(own, x.second, 0);
        (void)hipEventDestroy(x.second);
    }
    u.ev.clear();
}

namespace {
// Pinned host memory, a block per host thread that calls the library: results
// that kernels write (kDirectBytes), then read-backs (kStageBytes).  A thread
// that ends leaves its block to later ones (every call waits for its work
// before it returns), so there are as many as threads ran at once;
// dd_release_cache frees those that no thread holds.
constexpr size_t kStageBytes = 4096;
struct HostBlock {
    char *host = nullptr, *dev = nullptr;
};
struct HostBlocks {
    std::mutex mu;
    std::vector<HostBlock> left;
};
HostBlocks &host_blocks() {
    static HostBlocks *const b = new HostBlocks;   // (threads may end after static objects)
    return *b;
}
struct ThreadBlock {
    HostBlock b;
    ~ThreadBlock() {
        if (!b.host) return;
        HostBlocks &all = host_blocks();
        std::lock_guard<std::mutex> lk(all.mu);
        try {
            all.left.push_back(b);
        } catch (...) {
            (void)hipHostFree(b.host);
        }
    }
};

hipError_t host_block(HostBlock *out) {
    thread_local ThreadBlock mine;
    if (!mine.b.host) {
        HostBlocks &all = host_blocks();
        std::lock_guard<std::mutex> lk(all.mu);
        if (!all.left.empty()) {
            mine.b = all.left.back();
            all.left.pop_back();
        } else {
            void *h = nullptr, *d = nullptr;
            hipError_t e = hipHostMalloc(&h, kDirectBytes + kStageBytes, hipHostMallocPortable | hipHostMallocMapped);
            if (e != hipSuccess) return e;
            e = hipHostGetDevicePointer(&d, h, 0);
            if (e != hipSuccess) {
                (void)hipHostFree(h);
                return e;
            }
            mine.b = HostBlock{static_cast<char *>(h), static_cast<char *>(d)};
        }
    }
    *out = mine.b;
    return hipSuccess;
}

void release_host_blocks() {
    HostBlocks &all = host_blocks();
    std::lock_guard<std::mutex> lk(all.mu);
    for (const HostBlock &b : all.left) (void)hipHostFree(b.host);
    all.left.clear();
}
}  // namespace

hipError_t release_cache() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    release_host_blocks();
    std::lock_guard<std::mutex> lk(g_mu);
    release_cached(dev);
    return hipGetLastError();
}

hipError_t direct_buf(void **host, void **dev) {
    HostBlock b;
    const hipError_t e = host_block(&b);
    *host = b.host;
    *dev = b.dev;
    return e;
}

ReadBack::ReadBack(hipStream_t s, size_t cap) : s_(s) {
    cap_ = cap + 8 * 16;                  // room for aligning up to 16 items
    HostBlock b;
    err_ = cap_ > kStageBytes ? hipErrorInvalidValue : host_block(&b);
    if (err_ == hipSuccess) buf_ = b.host + kDirectBytes;
}

hipError_t ReadBack::add(void *dst, const void *src, size_t n) {
    if (err_ != hipSuccess) return err_;
    const size_t off = (used_ + 7) & ~size_t(7);
    if (off + n > cap_) return err_ = hipErrorInvalidValue;
    err_ = hipMemcpyAsync(buf_ + off, src, n, hipMemcpyDefault, s_);
    if (err_ == hipSuccess) {
        items_.push_back(Item{dst, off, n});
        used_ = off + n;
    }
    return err_;
}

hipError_t ReadBack::finish() {
    if (err_ == hipSuccess) err_ = hipStreamSynchronize(s_);
    if (err_ == hipSuccess)
        for (const Item &it : items_) memcpy(it.dst, buf_ + it.off, it.n);
    items_.clear();
    used_ = 0;
    return err_;
}

}  // namespace dd

#define TRY(x, what)                                           \
    do {                                                       \
        hipError_t e_ = (x);                                   \
        if (e_ != hipSuccess) { st = hip_fail(e_, what); goto fail_out; } \
    } while (0)

extern "C" {

const char *dd_status_str(dd_status s) {
    // callers may pass any integer: read it as one, not as the enum
    int code;
    memcpy(&code, &s, sizeof(code));
    switch (code) {
        case DD_OK: return "DD_OK";
        case DD_EINVAL: return "DD_EINVAL";
        case DD_ECYCLE: return "DD_ECYCLE";
        case DD_ECHAIN: return "DD_ECHAIN";
        case DD_ERANGE: return "DD_ERANGE";
        case DD_ENOMEM: return "DD_ENOMEM";
        case DD_EHIP: return "DD_EHIP";
        case DD_EMISMATCH: return "DD_EMISMATCH";
        case DD_ELIMIT: return "DD_ELIMIT";
    }
    return "DD_UNKNOWN";
}

const char *dd_last_error(void) { return g_err; }

dd_status dd_graph_load(int32_t n, int32_t n_threads, const int64_t *in_ptr, const int32_t *in_src,
                        const uint8_t *edge_cls, const int32_t *thread_prev,
                        const int32_t *thread_id, const int64_t *dur_ns, const int64_t *gap_ns,
                        const uint16_t *node_cls, void *stream, dd_graph **out) {
    return dd_graph_load_ex(n, n_threads, in_ptr, in_src, edge_cls, thread_prev, thread_id,
                            dur_ns, gap_ns, node_cls, 0u, stream, out);
}

dd_status dd_graph_load_ex(int32_t n, int32_t n_threads, const int64_t *in_ptr,
                           const int32_t *in_src, const uint8_t *edge_cls,
                           const int32_t *thread_prev, const int32_t *thread_id,
                           const int64_t *dur_ns, const int64_t *gap_ns, const uint16_t *node_cls,
                           uint32_t flags, void *stream, dd_graph **out) {
    g_err[0] = 0;
    if (!out) return fail(DD_EINVAL, "out is NULL");
    *out = nullptr;
    if (flags & ~DD_LOAD_SHARED_THREADS) return fail(DD_EINVAL, "unknown load flags 0x%x", flags);
    if (n < 0) return fail(DD_EINVAL, "n < 0");
    if (n_threads < 1) return fail(DD_EINVAL, "n_threads < 1");
    if (!in_ptr) return fail(DD_EINVAL, "in_ptr is NULL");
    if (n > 0 && (!thread_prev || !thread_id || !dur_ns || !gap_ns))
        return fail(DD_EINVAL, "thread_prev, thread_id, dur_ns and gap_ns are required");
    hipStream_t s = (hipStream_t)stream;
    dd_status st = DD_OK;
    dd_graph *g = new dd_graph();
    g->n = n;
    g->n_threads = n_threads;
    g->shared = (flags & DD_LOAD_SHARED_THREADS) != 0;
    g->stream = s;
    g->id = g_next_id.fetch_add(1);
    (void)hipGetDevice(&g->device);
    int64_t *d_in_ptr = nullptr;
    int32_t *d_in_src = nullptr;
    uint8_t *d_ecls = nullptr;
    dd::LoadOut *lo = nullptr, *lo_dev = nullptr;
    dd::LoadIn in;
    const size_t N = (size_t)n;
    // the call's own copy of an array: kernels make it from device memory
    // while they check it, anything else is copied here and checked in place
    auto own = [&](auto **dst, const auto *src, size_t count, const auto **from) -> hipError_t {
        *from = nullptr;
        hipError_t e = dd::dalloc_n(dst, count, s);
        if (e != hipSuccess || !src) return e;
        if (on_device(src, sizeof(*src))) {
            *from = src;
            return e;
        }
        *from = *dst;
        return hipMemcpyAsync(*dst, src, count * sizeof(*src), hipMemcpyDefault, s);
    };
    // the edge arrays, once their length is known
    auto edges = [&](int64_t e_count) -> hipError_t {
        if (e_count < 0 || e_count >= (int64_t(1) << 31)) {
            st = lo && lo->ends[0] != 0 ? fail(DD_EINVAL, "in_ptr[0] != 0")
                                        : fail(DD_EINVAL, "edge count outside [0, 2^31)");
            return hipErrorInvalidValue;
        }
        if (e_count > 0 && !in_src) {
            st = fail(DD_EINVAL, "in_src is NULL");
            return hipErrorInvalidValue;
        }
        g->n_edges = e_count;
        const size_t E = (size_t)e_count;
        hipError_t e = own(&d_in_src, E ? in_src : nullptr, E, &in.in_src);
        in.own_src = d_in_src;
        if (e == hipSuccess && edge_cls && E) {
            e = own(&d_ecls, edge_cls, E, &in.ecls);
            in.own_ecls = d_ecls;
        } else if (e == hipSuccess && g->shared) {
            e = copy_in(&d_ecls, (const uint8_t *)nullptr, E, s);   // (the graph keeps every edge's class)
        }
        if (e == hipSuccess && !g->shared) e = dd::dalloc_n(&g->xin_src, E + 1, s);
        if (e == hipSuccess && !g->shared) e = dd::dalloc_n(&g->xin_cls, E + 1, s);
        if (e != hipSuccess) st = hip_fail(e, "copy edges");
        return e;
    };

    {
        void *h = nullptr, *d = nullptr;
        TRY(dd::direct_buf(&h, &d), "alloc read-back buffer");
        lo = static_cast<dd::LoadOut *>(h);
        lo_dev = static_cast<dd::LoadOut *>(d);
    }
    *lo = dd::LoadOut{};
    TRY(dd::dalloc_n(&g->rank, N + 1, s), "alloc rank");
    if (!g->shared) {
        TRY(dd::dalloc_n(&g->thread_base, (size_t)n_threads + 1, s), "alloc");
        TRY(dd::dalloc_n(&g->order, N + 1, s), "alloc");
        TRY(dd::dalloc_n(&g->xin_ptr, N + 1, s), "alloc");
    }
    TRY(own(&g->thread_prev, thread_prev, N, &in.prev), "copy thread_prev");
    TRY(own(&g->thread_id, thread_id, N, &in.tid), "copy thread_id");
    TRY(own(&g->dur, dur_ns, N, &in.dur), "copy dur");
    TRY(own(&g->gap, gap_ns, N, &in.gap), "copy gap");
    TRY(own(&g->cls, node_cls, N, &in.cls), "copy node_cls");
    {
        TRY(own(&d_in_ptr, in_ptr, N + 1, &in.in_ptr), "copy in_ptr");
        in.own_ptr = d_in_ptr;
        if (n == 0) {
            dd::ReadBack rb(s, sizeof(int64_t));
            TRY(rb.add(&lo->ends[0], in.in_ptr, sizeof(int64_t)), "read in_ptr");
            TRY(rb.finish(), "sync");
            if (lo->ends[0] != 0) { st = fail(DD_EINVAL, "in_ptr[0] != 0"); goto fail_out; }
            if (edges(0) != hipSuccess) goto fail_out;
            TRY(hipMemsetAsync(g->shared ? d_in_ptr : g->xin_ptr, 0, sizeof(int64_t), s), "memset");
            if (!g->shared) {
                TRY(hipMemsetAsync(g->thread_base, 0, sizeof(int64_t) * ((size_t)n_threads + 1), s), "memset");
            }
            TRY(hipStreamSynchronize(s), "sync");
        } else {
            TRY(dd::load_device(g, in, lo, lo_dev, s, edges), "load");
            if (st != DD_OK) goto fail_out;
        }
    }
    if (lo->err[0]) { st = map_err_bits(lo->err[0]); goto fail_out; }
    g->n_cross = lo->n_cross;
    if (g->shared) {
        // several chains per thread: no thread-major order and no dropped
        // edges; every dependency edge stays for the schedule-rule path
        g->xin_ptr = d_in_ptr; d_in_ptr = nullptr;
        g->xin_src = d_in_src; d_in_src = nullptr;
        g->xin_cls = d_ecls; d_ecls = nullptr;
        g->n_cross = g->n_edges;
    }
    {
        const dd::LoadStats hs = lo->st;
        g->dsum = ((__int128)hs.dsum_hi << 32) + (__int128)hs.dsum_lo;
        const __int128 gs = ((__int128)hs.gsum_hi << 32) + (__int128)hs.gsum_lo;
        g->gsum = gs >= ((__int128)1 << 62) ? ((int64_t)1 << 62) : (int64_t)gs;
        g->dmax = (int64_t)hs.dmax;
        g->gmax = (int64_t)hs.gmax;
        g->max_cls = (int32_t)hs.cls_max;
        g->cross_mask = hs.cross_mask;
    }
    if (g->dsum + (__int128)g->gsum >= ((__int128)1 << 62)) {
        st = fail(DD_ERANGE, "sum of durations and gaps reaches 2^62 ns");
        goto fail_out;
    }
    dd::dfree(d_in_ptr, s); dd::dfree(d_in_src, s); dd::dfree(d_ecls, s);
    *out = g;
    return DD_OK;
fail_out:
    (void)hipStreamSynchronize(s);
    dd::dfree(d_in_ptr, s); dd::dfree(d_in_src, s); dd::dfree(d_ecls, s);
    free_graph_arrays(g);
    delete g;
    return st;
}

dd_status dd_levelize(const dd_graph *g, uint64_t active_edge_classes, int32_t mode, void *stream,
                      dd_sched **out, int64_t *n_steps_out) {
    g_err[0] = 0;
    if (!out) return fail(DD_EINVAL, "out is NULL");
    *out = nullptr;
    if (!g) return fail(DD_EINVAL, "graph is NULL");
    if (mode != DD_LEVELS && mode != DD_PHASES) return fail(DD_EINVAL, "mode must be DD_LEVELS or DD_PHASES");
    if (g->shared)
        return fail(DD_EINVAL, "the graph was loaded with shared threads: simulate it with dd_simulate_policy");
    hipStream_t s = (hipStream_t)stream;
    dd_sched *x = new dd_sched();
    x->graph_id = g->id;
    x->stream = s;
    char msg[256] = "";
    dd_status st = dd::levelize_device(g, active_edge_classes, mode, x, s, msg, sizeof(msg));
    if (st != DD_OK) {
        fail(st, "%s", msg);
        (void)hipStreamSynchronize(s);
        free_sched_arrays(x);
        delete x;
        return st;
    }
    if (hipError_t e = dd::note_use(g->uses, g->stream, s)) {
        st = hip_fail(e, "record stream use");
        free_sched_arrays(x);
        delete x;
        return st;
    }
    if (n_steps_out) *n_steps_out = x->n_steps;
    *out = x;
    return DD_OK;
}

dd_status dd_apply_transforms(const dd_graph *g, int32_t n_variants, int32_t n_cls,
                              const dd_ratio *scale, const uint32_t *remove_bits,
                              const uint64_t *edge_on, void *stream, dd_variants **out) {
    g_err[0] = 0;
    if (!out) return fail(DD_EINVAL, "out is NULL");
    *out = nullptr;
    if (!g) return fail(DD_EINVAL, "graph is NULL");
    if (n_variants < 1) return fail(DD_EINVAL, "n_variants < 1");
    if (!scale) n_cls = g->max_cls + 1;
    if (n_cls < 1 || n_cls <= g->max_cls)
        return fail(DD_EINVAL, "n_cls (%d) must exceed the largest task class (%d)", n_cls, g->max_cls);
    if ((int64_t)n_cls * n_variants >= (int64_t(1) << 31))
        return fail(DD_EINVAL, "n_cls * n_variants too large");
    hipStream_t s = (hipStream_t)stream;
    dd_status st = DD_OK;
    dd_variants *x = new dd_variants();
    x->graph_id = g->id;
    x->n = g->n;
    x->V = n_variants;
    x->W = (n_variants + 31) / 32;
    x->n_cls = n_cls;
    x->stream = s;
    dd_ratio *d_scale = nullptr;
    dd::TransformOut *o = nullptr, *o_dev = nullptr;
    dd::TransformIn t{n_cls, n_variants, nullptr, nullptr, nullptr, nullptr, nullptr, 0};
    const size_t cv = (size_t)n_cls * n_variants;
    const size_t rmw = (size_t)g->n * x->W;
    {
        void *h = nullptr, *d = nullptr;
        TRY(dd::direct_buf(&h, &d), "alloc read-back buffer");
        o = static_cast<dd::TransformOut *>(h);
        o_dev = static_cast<dd::TransformOut *>(d);
        static_assert(sizeof(dd::TransformOut) <= dd::kDirectBytes, "results fit the buffer");
    }
    TRY(dd::dalloc_n(&x->table, cv, s), "alloc table");
    if (scale && !on_device(scale, alignof(dd_ratio))) {
        TRY(copy_in(&d_scale, scale, cv, s), "copy scale");
        t.scale = d_scale;
    } else {
        t.scale = scale;
    }
    // removal bits: with the rest where they are few (a copy of its own
    // costs a launch), else by the runtime's copy
    if ((!remove_bits || on_device(remove_bits, sizeof(uint32_t))) && rmw <= ((size_t)2 << 20)) {
        TRY(dd::dalloc_n(&x->rm_bits, rmw, s), "alloc remove_bits");
        t.rm_src = remove_bits;
        t.rm_dst = x->rm_bits;
        t.rm_words = (int64_t)rmw;
    } else {
        TRY(copy_in(&x->rm_bits, remove_bits, rmw, s), "copy remove_bits");
    }
    TRY(dd::dalloc_n(&x->edge_on, (size_t)n_variants, s), "alloc edge_on");
    t.on_dst = x->edge_on;
    if (edge_on && !on_device(edge_on, sizeof(uint64_t))) {
        TRY(hipMemcpyAsync(x->edge_on, edge_on, sizeof(uint64_t) * (size_t)n_variants, hipMemcpyDefault, s),
            "copy edge_on");
        t.on_src = x->edge_on;
    } else {
        t.on_src = edge_on;
    }
    TRY(dd::transforms_device(t, x->table, o, o_dev, s), "transforms");
    x->used_mask = o->used_mask;
    x->all_mask = o->all_mask;
    x->any_magic = o->magic != 0;
    if (o->err) { st = map_err_bits(o->err); goto fail_out; }
    {
        const uint64_t pmax = (uint64_t)o->pmax;
        double rmax;
        memcpy(&rmax, &o->rmax_bits, 8);
        // d * p must stay below 2^62, and so must every time in the simulation
        if ((__int128)g->dmax * (__int128)pmax >= ((__int128)1 << 62)) {
            st = fail(DD_ERANGE, "largest duration times largest p reaches 2^62");
            goto fail_out;
        }
        long double bound = (long double)g->dsum * (long double)rmax + (long double)g->gsum;
        if (bound >= 4.0e18L) {   // 2^62 = 4.61e18, kept a margin for rounding
            st = fail(DD_ERANGE, "scaled durations could sum past 2^62 ns");
            goto fail_out;
        }
        // every simulated time is a sum of weights along a path, so below
        // the bound; 2^51 = 2.25e15 (a margin for rounding again)
        x->f64_ok = bound < 2.0e15L &&
                    (__int128)g->dmax * (__int128)pmax < ((__int128)1 << 53);
        x->quot_ok = x->f64_ok && (__int128)g->dmax * (__int128)pmax < ((__int128)1 << 50);
    }
    TRY(dd::note_use(g->uses, g->stream, s), "record stream use");
    dd::dfree(d_scale, s);
    *out = x;
    return DD_OK;
fail_out:
    (void)hipStreamSynchronize(s);
    dd::dfree(d_scale, s);
    dd::dfree(x->table, s); dd::dfree(x->rm_bits, s); dd::dfree(x->edge_on, s);
    delete x;
    return st;
}

}  // extern "C"

namespace {

dd_status simulate_impl(const dd_graph *g, const dd_sched *sched, const dd_variants *var,
                        int64_t *d_finish, int64_t *d_start, int64_t *d_makespan, int vs,
                        void *stream) {
    if (!g || !sched || !var) return fail(DD_EINVAL, "NULL handle");
    if (!d_makespan || (!d_finish && g->n > 0))
        return fail(DD_EINVAL, "d_finish and d_makespan are required");
    if (sched->graph_id != g->id || var->graph_id != g->id)
        return fail(DD_EMISMATCH, "handles come from different graphs");
    const uint64_t missing = var->used_mask & g->cross_mask & ~sched->mask;
    if (missing)
        return fail(DD_EMISMATCH, "variants switch on edge classes 0x%llx that the schedule was not built for",
                    (unsigned long long)missing);
    hipStream_t s = (hipStream_t)stream;
    // few variants over few long steps: each step cut across workgroups
    const int sw = vs < 0 ? -vs : vs == 0 ? dd::split_width(sched, var) : 0;
    if (sw > 0 && (int64_t)sched->h_step_ptr.size() != sched->n_steps + 1)
        return fail(DD_EINVAL, "the split path needs a schedule of at most %lld steps (this one has %lld)",
                    (long long)dd::kSplitMaxSteps, (long long)sched->n_steps);
    hipError_t e = sw > 0 ? dd::launch_split(g, sched, var, d_finish, d_start, d_makespan, sw, s)
                          : dd::launch_simulate(g, sched, var, d_finish, d_start, d_makespan, vs, s);
    if (e != hipSuccess) return hip_fail(e, "simulate launch");
    e = dd::note_use(g->uses, g->stream, s);
    if (e == hipSuccess) e = dd::note_use(sched->uses, sched->stream, s);
    if (e == hipSuccess) e = dd::note_use(var->uses, var->stream, s);
    if (e != hipSuccess) return hip_fail(e, "record stream use");
    return DD_OK;
}

}  // namespace

extern "C" {

dd_status dd_simulate_batch(const dd_graph *g, const dd_sched *sched, const dd_variants *var,
                            int64_t *d_finish, int64_t *d_start, int64_t *d_makespan, void *stream) {
    g_err[0] = 0;
    return simulate_impl(g, sched, var, d_finish, d_start, d_makespan, 0, stream);
}

dd_status dd_simulate_batch_vs(const dd_graph *g, const dd_sched *sched, const dd_variants *var,
                               int64_t *d_finish, int64_t *d_start, int64_t *d_makespan,
                               int32_t variants_per_wg, void *stream) {
    g_err[0] = 0;
    const int w = variants_per_wg < 0 ? -variants_per_wg : variants_per_wg;
    if (!(w == 0 || w == 1 || w == 2 || w == 4 || w == 8 || (w == 16 && variants_per_wg > 0)))
        return fail(DD_EINVAL, "variants_per_wg must be 0, 1, 2, 4, 8, 16, -1, -2, -4 or -8 (got %d)",
                    (int)variants_per_wg);
    return simulate_impl(g, sched, var, d_finish, d_start, d_makespan, variants_per_wg, stream);
}

void dd_set_lookback_polls(int32_t polls) { dd::split_set_polls(polls); }

dd_status dd_runtime_breakdown(const dd_graph *g, const dd_variants *var, const uint8_t *role,
                               const int64_t *d_finish, const int64_t *d_makespan,
                               int64_t *d_out, void *stream) {
    g_err[0] = 0;
    if (!g || !var) return fail(DD_EINVAL, "NULL handle");
    if (!d_makespan || !d_out || (g->n > 0 && (!d_finish || !role)))
        return fail(DD_EINVAL, "role, d_finish, d_makespan and d_out are required");
    if (var->graph_id != g->id) return fail(DD_EMISMATCH, "handles come from different graphs");
    if (g->shared)
        return fail(DD_EINVAL, "the graph was loaded with shared threads: its thread order is "
                               "decided by the schedule rule, not recorded");
    hipStream_t s = (hipStream_t)stream;
    dd_status st = DD_OK;
    uint8_t *d_role = nullptr;
    if (!on_device(role)) TRY(copy_in(&d_role, role, (size_t)g->n, s), "copy role");
    TRY(dd::launch_breakdown(g, var, d_role ? d_role : role, d_finish, d_makespan, d_out, s), "breakdown");
    TRY(dd::note_use(g->uses, g->stream, s), "record stream use");
    TRY(dd::note_use(var->uses, var->stream, s), "record stream use");
fail_out:
    dd::dfree(d_role, s);
    return st;
}

dd_status dd_simulate_policy(const dd_graph *g, const dd_variants *var, int32_t policy,
                             const uint8_t *pp, const int32_t *prio, int64_t *d_finish,
                             int64_t *d_start, int64_t *d_makespan, void *stream) {
    g_err[0] = 0;
    if (!g || !var) return fail(DD_EINVAL, "NULL handle");
    if (policy != DD_POLICY_EARLIEST && policy != DD_POLICY_PRIORITY)
        return fail(DD_EINVAL, "policy must be DD_POLICY_EARLIEST or DD_POLICY_PRIORITY");
    if (policy == DD_POLICY_PRIORITY && g->n > 0 && (!pp || !prio))
        return fail(DD_EINVAL, "DD_POLICY_PRIORITY needs pp and prio");
    if (!d_makespan || (!d_finish && g->n > 0))
        return fail(DD_EINVAL, "d_finish and d_makespan are required");
    if (var->graph_id != g->id) return fail(DD_EMISMATCH, "handles come from different graphs");
    if (g->n >= (1 << dd::kEventIdBits))
        return fail(DD_ELIMIT, "the schedule-rule path takes n < 2^%d tasks", dd::kEventIdBits);
    if (g->n_threads > dd::kEventMaxThreads)
        return fail(DD_ELIMIT, "the schedule-rule path takes at most %d threads", dd::kEventMaxThreads);
    if (g->n_cross + (int64_t)g->n >= (int64_t(1) << 31))
        return fail(DD_ELIMIT, "too many edges for the schedule-rule path");
    hipStream_t s = (hipStream_t)stream;
    dd_status st = DD_OK;
    uint8_t *d_pp = nullptr;
    int32_t *d_prio = nullptr, *ref = nullptr;
    int64_t *est = nullptr;
    uint32_t *err = nullptr, *keep = nullptr;
    uint32_t h_err = 0;
    const size_t nv = (size_t)g->n * (size_t)var->V;
    {
        std::lock_guard<std::mutex> lk(g->ev_mu);
        if (!g->ev.rec) {
            hipError_t e = dd::build_event_lists(g, &g->ev, s);
            if (e != hipSuccess) {
                dd::free_event_lists(&g->ev, s);
                return hip_fail(e, "build out-edge lists");
            }
            // the lists belong to the graph and are released on its stream
            e = dd::note_use(g->uses, g->stream, s);
            if (e != hipSuccess) return hip_fail(e, "record stream use");
        }
    }
    if (policy == DD_POLICY_PRIORITY) {
        TRY(copy_in(&d_pp, pp, (size_t)g->n, s), "copy pp");
        TRY(copy_in(&d_prio, prio, (size_t)g->n, s), "copy prio");
    }
    TRY(copy_in(&err, (const uint32_t *)nullptr, 1, s), "alloc");
    {
        const hipError_t e = dd::launch_sim_event(g, g->ev, var, policy, d_pp, d_prio, nullptr, nullptr, &keep,
                                                  d_finish, d_start, d_makespan, err, s);
        if (e != hipErrorNotSupported) {
            TRY(e, "simulate");
            dd::ReadBack rb(s, sizeof(uint32_t));
            TRY(rb.add(&h_err, err, sizeof(uint32_t)), "read err");
            TRY(rb.finish(), "sync");
        } else {
            h_err = 4u;
            dd::dfree(keep, s);
            keep = nullptr;
        }
    }
    if (h_err & 4u) {
        h_err = 0;
        TRY(hipMemsetAsync(err, 0, sizeof(uint32_t), s), "memset");
        hipError_t e = dd::dalloc_n(&ref, nv, s);
        if (e == hipSuccess) e = dd::dalloc_n(&est, nv, s);
        if (e == hipErrorOutOfMemory && keep) {  // (from the start, then)
            (void)hipGetLastError();
            dd::dfree(keep, s);
            dd::dfree(ref, s);
            keep = nullptr;
            ref = nullptr;
            e = dd::dalloc_n(&ref, nv, s);
            if (e == hipSuccess) e = dd::dalloc_n(&est, nv, s);
        }
        TRY(e, "alloc reference counts and start times");
        TRY(dd::launch_sim_event(g, g->ev, var, policy, d_pp, d_prio, ref, est, &keep, d_finish, d_start,
                                 d_makespan, err, s), "simulate");
        dd::ReadBack rb(s, sizeof(uint32_t));
        TRY(rb.add(&h_err, err, sizeof(uint32_t)), "read err");
        TRY(rb.finish(), "sync");
    }
    TRY(dd::note_use(g->uses, g->stream, s), "record stream use");
    TRY(dd::note_use(var->uses, var->stream, s), "record stream use");
    if (h_err & 2u)
        st = fail(DD_ELIMIT, "more than %d tasks were ready at once in some variant",
                  dd::kEventQueue);
    else if (h_err & 1u)
        st = fail(DD_ECYCLE, "the active dependencies and thread chains contain a cycle");
fail_out:
    dd::dfree(d_pp, s);
    dd::dfree(d_prio, s);
    dd::dfree(ref, s);
    dd::dfree(est, s);
    dd::dfree(err, s);
    dd::dfree(keep, s);
    return st;
}

dd_status dd_simulate_batch_noalloc(const dd_graph *g, const dd_sched *sched, const dd_variants *var,
                                    int64_t *d_finish, int64_t *d_start, int64_t *d_makespan,
                                    void *stream) {
    g_err[0] = 0;
    if (!g || !sched || !var) return fail(DD_EINVAL, "NULL handle");
    if (!d_makespan || (!d_finish && g->n > 0))
        return fail(DD_EINVAL, "d_finish and d_makespan are required");
    if (sched->graph_id != g->id || var->graph_id != g->id)
        return fail(DD_EMISMATCH, "handles come from different graphs");
    const uint64_t missing = var->used_mask & g->cross_mask & ~sched->mask;
    if (missing)
        return fail(DD_EMISMATCH, "variants switch on edge classes 0x%llx that the schedule was not built for",
                    (unsigned long long)missing);
    size_t need = 0, limit = 0;
    hipError_t e = dd::simulate_noalloc(g, sched, var, d_finish, d_start, d_makespan,
                                        (hipStream_t)stream, &need, &limit);
    if (need > limit)
        return fail(DD_EINVAL, "this batch needs %zu bytes of scratch; the allocation-free entry "
                               "point has %zu (use dd_simulate_batch)", need, limit);
    if (e != hipSuccess) return hip_fail(e, "simulate launch");
    return DD_OK;
}

dd_status dd_release_cache(void) {
    g_err[0] = 0;
    hipError_t e = dd::release_cache();
    if (e != hipSuccess) return hip_fail(e, "release cache");
    return DD_OK;
}

dd_status dd_sched_task_steps(const dd_sched *sched, int32_t *steps_out, void *stream) {
    g_err[0] = 0;
    if (!sched || !steps_out) return fail(DD_EINVAL, "NULL argument");
    hipStream_t s = (hipStream_t)stream;
    if (sched->n == 0) return DD_OK;
    hipError_t e = hipMemcpyAsync(steps_out, sched->node_step, sizeof(int32_t) * (size_t)sched->n,
                                  hipMemcpyDefault, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "copy steps");
    return DD_OK;
}

dd_status dd_simulate_plan(const dd_sched *sched, const dd_variants *var,
                           int32_t *variants_per_wg) {
    g_err[0] = 0;
    if (!sched || !var || !variants_per_wg) return fail(DD_EINVAL, "NULL argument");
    const int sw = dd::split_width(sched, var);
    *variants_per_wg = sw > 0 ? -sw : dd::solo_chosen(sched, var) ? 1 : dd::strip_width(var->V);
    return DD_OK;
}

dd_status dd_sched_info(const dd_sched *sched, int64_t *n_steps, int64_t *n_segments,
                        int64_t *max_step_width, int64_t *n_gathers) {
    g_err[0] = 0;
    if (!sched) return fail(DD_EINVAL, "NULL schedule");
    if (n_steps) *n_steps = sched->n_steps;
    if (n_segments) *n_segments = sched->n_segments;
    if (max_step_width) *max_step_width = sched->max_width;
    if (n_gathers) *n_gathers = sched->n_gathers;
    return DD_OK;
}

void dd_graph_free(dd_graph *g) {
    if (!g) return;
    free_graph_arrays(g);
    delete g;
}

void dd_sched_free(dd_sched *x) {
    if (!x) return;
    free_sched_arrays(x);
    delete x;
}

void dd_variants_free(dd_variants *x) {
    if (!x) return;
    hipStream_t s = x->stream;
    dd::join_uses(x->uses, s);
    dd::dfree(x->table, s);
    dd::dfree(x->rm_bits, s);
    dd::dfree(x->edge_on, s);
    delete x;
}

}  // extern "C"
