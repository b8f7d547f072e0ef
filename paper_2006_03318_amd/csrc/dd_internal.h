// Internal declarations shared by the HIP sources of the dd library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <functional>
#include <mutex>
#include <utility>
#include <vector>

#include "dd.h"

namespace dd {

// ---------------------------------------------------------------------------
// error bits raised by device-side validation (one 32-bit word per check run)
enum : uint32_t {
    ERR_THREAD_RANGE = 1u << 0,   // thread id outside [0, n_threads)       EINVAL
    ERR_PREV_RANGE = 1u << 1,     // thread_prev outside [-1, n) or == self  EINVAL
    ERR_PREV_THREAD = 1u << 2,    // thread_prev on another thread           ECHAIN
    ERR_NEG_TIME = 1u << 3,       // negative duration or gap                EINVAL
    ERR_BIG_TIME = 1u << 4,       // duration or gap >= 2^62                 ERANGE
    ERR_PTR_ORDER = 1u << 5,      // in_ptr decreasing                       EINVAL
    ERR_SRC_RANGE = 1u << 6,      // in_src outside [0, n)                   EINVAL
    ERR_SELF_LOOP = 1u << 7,      // edge u -> u                             ECYCLE
    ERR_EDGE_CLS = 1u << 8,       // edge class >= 64                        EINVAL
    ERR_SUCC = 1u << 9,           // two tasks name the same thread_prev     ECHAIN
    ERR_HEADS = 1u << 10,         // a thread with two first tasks           ECHAIN
    ERR_CHAIN_CYCLE = 1u << 11,   // thread order loops                      ECHAIN
    ERR_BACK_EDGE = 1u << 12,     // same-thread dependency points backwards ECYCLE
    ERR_KAHN_CYCLE = 1u << 13,    // Kahn rounds stall before the end        ECYCLE
    ERR_SCALE = 1u << 14,         // p < 0 or q < 1                          EINVAL
};

constexpr int64_t kTimeLimit = int64_t(1) << 62;

// Per-(class, variant) shrink/scale entry: floor(d * p / q) evaluated as
// a = d * p; q a power of two: a >> shift; otherwise the high 64 bits of
// a * magic shifted right by `shift` (Granlund & Montgomery, PLDI 1994,
// round-up method; exact for every a < 2^62).
struct alignas(16) ScaleEntry {
    uint64_t magic;   // 0 when q is a power of two
    uint32_t p;
    uint32_t shift;
};

// One schedule position as the simulation reads it: the task, its
// duration, gap and class, and up to two of its gathers inline (source task,
// the source's schedule position, edge class).  Gathers beyond two stay in
// the gather arrays (gat_rng).
struct alignas(16) Rec {
    int64_t dur, gap;
    int32_t node, g0_src, g1_src, g0_spos;
    int32_t g1_spos;
    uint32_t cls;     // bits 0..15 task class, 16..23 / 24..31 edge class of gather 0 / 1
    uint32_t flags;   // bit0: first task of a thread run; bit1: last task of a run;
                      // bits 2..7: thread (graphs with at most 64 threads);
                      // bits 8..31: gathers beyond two (saturating)
    uint32_t g0_gap32;  // gap of gather 0's source, low 32 bits (whole when gaps < 2^32)
};
static_assert(sizeof(Rec) == 48, "record size");

// Schedules of at most this many steps keep a host copy of their step
// offsets: the few-variant path launches one kernel per step.
constexpr int64_t kSplitMaxSteps = 512;

// Graphs with at most this many threads keep each thread's latest release in
// LDS during the simulation instead of gathering the previous task of a run.
constexpr int kMaxCarryThreads = 64;

// Batches of the one-variant-per-workgroup kernel (k_solo.hip): steps of at
// most kSoloNarrow positions are grouped by the kSoloGroup-aligned span they
// start in (so a group has fewer than kSoloPos positions), wider ones cut
// into parts of kSoloPos positions.
constexpr int kSoloNarrow = 128;
constexpr int kSoloGroup = 384;
constexpr int kSoloPos = 512;
static_assert(kSoloGroup + kSoloNarrow <= kSoloPos, "a group of narrow steps is one batch");
constexpr int kSoloCls = 2048;    // scale entries it keeps in LDS (16 bytes each)
constexpr int kSoloRing = 32768;  // releases of recent positions it keeps per variant at most

// A schedule position as that kernel reads it (durations and gaps below
// 2^32).
struct alignas(16) SoloRec {
    uint32_t dur, gap;
    int32_t node, g0_spos;    // task; schedule position of its first parent (-1: none)
    uint32_t cls;             // as Rec::cls
    uint32_t flags;           // bits 0..7 as Rec::flags; kSoG1; 16..31 parents beyond two (saturating)
    int32_t g1_spos, pad;
};
constexpr uint32_t kSoG1 = 1u << 8;   // a second parent on another thread

// Streams other than its own on which a handle's device memory was used.
// A handle's blocks go back to the cache of the stream it was created on;
// before that, its own stream waits for the last use on each other stream,
// so a later allocation there cannot overwrite memory a kernel still reads.
struct ForeignUses {
    std::mutex mu;
    std::vector<std::pair<hipStream_t, hipEvent_t>> ev;
};
// record the point after the work just queued on s (no-op when s == own)
hipError_t note_use(ForeignUses &u, hipStream_t own, hipStream_t s);
// make `own` wait for every recorded use; the events are released
void join_uses(ForeignUses &u, hipStream_t own);

// Statistics reduced on the device while loading (hi/lo split sums cannot
// overflow for n < 2^31 values below 2^62).
struct LoadStats {
    unsigned long long dsum_hi, dsum_lo, gsum_hi, gsum_lo;
    unsigned long long dmax, cls_max, cross_mask, gmax;
};

}  // namespace dd

namespace dd {
// Out-edge lists for the task-by-task simulation under a schedule rule:
// every dependency edge and every thread-order link as (child << 8 | class),
// class 255 for thread order (always present), grouped by parent.
struct EventLists {
    int4 *rec = nullptr;        // [n] {first out-edge, out-edge count, thread, task class}
    uint4 *e4 = nullptr;        // [n] the first four out-edges (0 past the count)
    uint32_t *edges = nullptr;  // [n_edges]
    int64_t n_edges = 0;
    uint64_t cls_mask = 0;      // edge classes present
};
constexpr uint32_t kEdgeAlways = 255;
}  // namespace dd

struct dd_graph {
    int32_t n = 0, n_threads = 0;
    bool shared = false;          // threads may hold several chains (DD_LOAD_SHARED_THREADS);
                                  // then xin_* hold every dependency edge
    int64_t n_edges = 0, n_cross = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    uint64_t id = 0;
    // statistics (host)
    int64_t dmax = 0, gmax = 0, gsum = 0;
    __int128 dsum = 0;
    int32_t max_cls = 0;
    uint64_t cross_mask = 0;      // edge classes present among cross-thread edges
    // device arrays
    int32_t *thread_prev = nullptr, *thread_id = nullptr;
    int64_t *dur = nullptr, *gap = nullptr;
    uint16_t *cls = nullptr;
    int32_t *rank = nullptr;      // position of each task on its thread
    int64_t *thread_base = nullptr;  // [T+1]
    int32_t *order = nullptr;     // [n] tasks thread-major in thread order
    int64_t *xin_ptr = nullptr;   // [n+1] cross-thread in-edges
    int32_t *xin_src = nullptr;
    uint8_t *xin_cls = nullptr;
    mutable dd::ForeignUses uses;
    mutable std::mutex ev_mu;     // guards ev, built on first use
    mutable dd::EventLists ev;
};

struct dd_sched {
    uint64_t graph_id = 0;
    int32_t n = 0, mode = 0;
    uint64_t mask = 0;
    int64_t n_steps = 0, n_segments = 0, max_width = 0, n_gathers = 0;
    hipStream_t stream = nullptr;
    int32_t *step_ptr = nullptr;  // [n_steps+1] position offsets
    int32_t *pos_node = nullptr;  // [n]
    uint64_t *gat_rng = nullptr;  // [n] gathers of each position: first entry | entries << 32
    int32_t *gat_src = nullptr;   // source task of each gather
    uint8_t *gat_cls = nullptr;   // edge class; 255 = always present (thread order)
    int64_t *gat_gap = nullptr;   // gap of the source task
    int32_t *gat_spos = nullptr;  // schedule position of the source task
    int32_t *node_step = nullptr; // [n]
    dd::Rec *rec = nullptr;       // [n] per position
    int4 *bat = nullptr;          // batches of k_solo.hip
    int32_t *nbat = nullptr;      // [1] how many
    dd::SoloRec *so_rec = nullptr;    // [n] its records
    bool thread_carry = false;    // thread predecessors come from per-thread carries
    std::vector<int32_t> h_step_ptr;  // host copy of step_ptr (schedules of at most
                                      // kSplitMaxSteps steps; empty otherwise)
    mutable dd::ForeignUses uses;
};

struct dd_variants {
    uint64_t graph_id = 0;
    int32_t n = 0, V = 0, W = 0, n_cls = 0;
    uint64_t used_mask = 0;       // OR of edge_on over all variants
    uint64_t all_mask = 0;        // AND of edge_on over all variants
    bool any_magic = false;       // some scale has q not a power of two
    bool f64_ok = false;          // every simulated time below 2^51 and every d * p below
                                  // 2^53: the double form of the time arithmetic is exact
    bool quot_ok = false;         // f64_ok and every d * p below 2^50: so are quotients by any q
    hipStream_t stream = nullptr;
    dd::ScaleEntry *table = nullptr;  // [n_cls][V]
    uint32_t *rm_bits = nullptr;      // [n][W]
    uint64_t *edge_on = nullptr;      // [V]
    mutable dd::ForeignUses uses;
};

namespace dd {

// Read-backs of small results (below 4,000 bytes) through a pinned host buffer.  A copy from the device into
// pageable memory waits for its stream by itself (about 10 us each); into
// pinned memory it is a plain DMA, so the queued copies of one read-back
// cost one synchronization.  cap = the bytes that will be queued.
class ReadBack {
public:
    ReadBack(hipStream_t s, size_t cap);
    // queue a copy of n bytes from src (device or host) into dst
    hipError_t add(void *dst, const void *src, size_t n);
    // wait for the stream, then fill every queued dst
    hipError_t finish();
private:
    struct Item { void *dst; size_t off, n; };
    hipStream_t s_;
    char *buf_ = nullptr;
    size_t cap_ = 0, used_ = 0;
    hipError_t err_ = hipSuccess;
    std::vector<Item> items_;
};

// device memory (cache of blocks kept per device and stream)
hipError_t dalloc(void **p, size_t bytes, hipStream_t s);
void dfree(void *p, hipStream_t s);
// return every cached block of the current device (waits for the device)
hipError_t release_cache();
template <class T>
hipError_t dalloc_n(T **p, size_t count, hipStream_t s) {
    return dalloc(reinterpret_cast<void **>(p), count * sizeof(T) + 16, s);
}

// exclusive prefix sum: out[i] = sum_{j<i} in[j] for i in [0, n]; in/out may alias
hipError_t scan_exclusive(const int64_t *in, int64_t *out, int64_t n, hipStream_t s);
// the same with the caller's temporaries: tmp holds scan_temp_count(n) int64
int64_t scan_temp_count(int64_t n);
hipError_t scan_exclusive_ws(const int64_t *in, int64_t *out, int64_t n, int64_t *tmp,
                             hipStream_t s);

inline int grid_for(int64_t n, int bs) {
    int64_t g = (n + bs - 1) / bs;
    if (g < 1) g = 1;
    if (g > (int64_t(1) << 30)) g = int64_t(1) << 30;
    return (int)g;
}

// Passes over n > 0 tasks cut them into at most kChunks chunks, of whole
// workgroups of `bs` threads (in 64 bits: n + kChunks passes 2^31).
constexpr int kChunks = 1024;
inline int64_t chunk_len(int64_t n, int bs) {
    return ((n + kChunks - 1) / kChunks + bs - 1) / bs * bs;
}

// Results that kernels write straight into host memory (a pinned buffer of
// this host thread; read after the stream has been waited for): no copy, and no launch for one.  *dev receives the address
// kernels use.
constexpr size_t kDirectBytes = 64 << 10;
hipError_t direct_buf(void **host, void **dev);

// Device passes that only the full library has: weak, so that the API layer
// links (and its host-side checks run) without them.
#define DD_PASS __attribute__((weak))

// graph load (k_graph.hip)
struct LoadIn {                   // the caller's arrays where kernels can read them (or the
                                  // copies themselves, of arrays they cannot)
    const int64_t *in_ptr = nullptr;
    const int32_t *in_src = nullptr;
    const uint8_t *ecls = nullptr;
    const int32_t *prev = nullptr, *tid = nullptr;
    const int64_t *dur = nullptr, *gap = nullptr;
    const uint16_t *cls = nullptr;
    // the copies that the passes check and use (own_ecls null: all class 0)
    int64_t *own_ptr = nullptr;
    int32_t *own_src = nullptr;
    uint8_t *own_ecls = nullptr;
};
struct LoadOut {
    int64_t ends[2];              // in_ptr[0], in_ptr[n]
    int64_t n_cross;
    uint32_t err[2];
    LoadStats st;
};
// All passes of a load with n > 0, complete on return.  edges(E), called with
// the edge count once in_ptr's ends are read (-1: in_ptr[0] != 0), checks it
// and provides the edge arrays of in and the lists of g that it sizes, or
// fails, and nothing more runs.  out: results (host memory, see direct_buf).
DD_PASS hipError_t load_device(dd_graph *g, const LoadIn &in, LoadOut *out, LoadOut *out_dev, hipStream_t s,
                               const std::function<hipError_t(int64_t)> &edges);

// levelization (k_levelize.hip)
struct LevelizeOut {
    int64_t n_steps, n_segments, max_width, n_gathers;
    uint32_t err, pad;
    int32_t steps[kSplitMaxSteps + 1];   // step offsets, of at most kSplitMaxSteps steps
};
dd_status levelize_device(const dd_graph *g, uint64_t mask, int32_t mode, dd_sched *sch,
                          hipStream_t s, char *msg, size_t msg_len);

// transforms (k_transform.hip): everything dd_apply_transforms does on the
// device, complete on return
constexpr int kTransformBlocks = 512, kMaskBlocks = 64;
struct TransformIn {
    int32_t n_cls, V;
    const dd_ratio *scale;        // device, or null: 1/1
    const uint64_t *on_src;       // device, or null: all classes
    uint64_t *on_dst;
    const uint32_t *rm_src;       // device, or null: none removed
    uint32_t *rm_dst;
    int64_t rm_words;             // 0: copied elsewhere
};
struct TransformOut {
    uint64_t used_mask, all_mask; // OR and AND of the edge-class masks
    uint32_t err, magic;          // error bits; some q is not a power of two
    int64_t pmax, rmax_bits;      // largest p, largest p / q (bits of a double)
    struct Block {
        uint32_t err, magic;
        int64_t pmax, rmax_bits;
    } blk[kTransformBlocks];
    uint64_t used[kMaskBlocks], all[kMaskBlocks];   // the masks, per block
};
DD_PASS hipError_t transforms_device(const TransformIn &t, ScaleEntry *table, TransformOut *out,
                                     TransformOut *out_dev, hipStream_t s);

// few-variant simulation (k_split.hip): every step cut across several
// workgroups per variant, one launch per step.  split_width() gives the
// variants per workgroup (1, 2, 4 or 8) when the schedule and variants suit
// it, else 0; launch_split() takes that width.
int split_width(const dd_sched *sch, const dd_variants *var);
// look-back polls of one slot before a lane folds that chunk itself
// (negative: the default)
void split_set_polls(int32_t polls);
hipError_t launch_split(const dd_graph *g, const dd_sched *sch, const dd_variants *var,
                        int64_t *finish, int64_t *start, int64_t *makespan, int vg, hipStream_t s);

// variants per workgroup of the one-workgroup-per-strip kernel when the
// caller leaves it to the library: the fewest with which all workgroups run
// at once (one per compute unit).  A workgroup of twice the variants takes
// 1.0 to 1.3 times as long, a second pass twice as long: 5 transformer
// iterations, 1,000 variants: 1,634 us four to a workgroup, 3,247 two.
inline int strip_width(int64_t V) {
    int vs = 1;
    while (vs < 16 && (V + vs - 1) / vs > 256) vs *= 2;
    return vs;
}

// simulation (k_simulate.hip)
hipError_t launch_simulate(const dd_graph *g, const dd_sched *sch, const dd_variants *var,
                           int64_t *finish, int64_t *start, int64_t *makespan, int vs_hint,
                           hipStream_t s);
// the same in the library's per-GPU scratch array, allocating nothing:
// *need = bytes this call needs, *limit = the array's size;
// hipErrorInvalidValue when need > limit (nothing launched)
hipError_t simulate_noalloc(const dd_graph *g, const dd_sched *sch, const dd_variants *var,
                            int64_t *finish, int64_t *start, int64_t *makespan, hipStream_t s,
                            size_t *need, size_t *limit);

// one variant per workgroup (k_solo.hip): the most entries the batch list of
// n positions can have (a wide step has at least kSoloNarrow + 1 positions and
// ends a group of narrow ones; a group starts in each kSoloGroup-aligned
// span), and the launch (hipErrorOutOfMemory when its scratch, mostly
// V * kSoloRing * 8 bytes, cannot be had)
inline int64_t solo_batch_max(int64_t n) {
    return 2 * (n / kSoloNarrow) + n / kSoloPos + n / kSoloGroup + 8;
}
hipError_t launch_solo(const dd_graph *g, const dd_sched *sch, const dd_variants *var,
                       int64_t *finish, int64_t *start, int64_t *makespan, hipStream_t s);

// removal bits [n][W] as one bit string per variant, [V][stride] words, in
// the order of `order`.  rm_stride: whole pairs of words that hold bits 0 to n
// (a lane of k_solo.hip without a position looks at bit n, where the next
// position would be)
inline int64_t rm_stride(int64_t n) { return (n / 64 + 1) * 2; }
hipError_t launch_rm_bits(int64_t n, int32_t V, int32_t W, int64_t stride, const int32_t *order,
                          const uint32_t *rm, uint32_t *rmb, hipStream_t s);

// whether that kernel takes these handles: times and durations fit its
// arithmetic (the schedule then has its records), the scales fit LDS
inline bool solo_fits(const dd_sched *sch, const dd_variants *var) {
    return sch->so_rec && sch->n > 0 && var->quot_ok && var->n_cls <= kSoloCls;
}

// Whether dd_simulate_batch takes it.  Two of its workgroups run on a compute
// unit, so up to 512 variants run at once, at 0.35 to 0.4 us per narrow step
// and 1.1 to 1.8 us per 512 positions of a wide one; the strip kernel costs
// 1.5 us per step and 1.7 us per 512 positions, but packs up to 16 variants
// into a workgroup.  Measured, us (solo / strip): 5 transformer iterations
// (163,840 tasks in 256 steps) 565 / 1,073 at 256 variants, 819 / 1,402 at
// 333, 916 / 1,390 at 512, 1,401 / 1,461 at 768, 2,108 / 1,490 at 1,024;
// the offloading CNN (1,932 tasks in 173 steps) 70 / 284 at 256, 148 / 308
// at 1,024.  Beyond 2,048 variants its passes add up on any schedule.
inline bool solo_chosen(const dd_sched *sch, const dd_variants *var) {
    if (!solo_fits(sch, var) || var->V > 2048) return false;
    return var->V <= 768 || (int64_t)sch->n <= 32 * sch->n_steps;
}

// runtime breakdown (k_breakdown.hip): out [V][4]
hipError_t launch_breakdown(const dd_graph *g, const dd_variants *var, const uint8_t *role_dev,
                            const int64_t *finish, const int64_t *makespan, int64_t *out, hipStream_t s);

// simulation under a schedule rule (k_event.hip)
// out-edge lists of g (dependencies in xin_*, thread order in thread_prev)
hipError_t build_event_lists(const dd_graph *g, EventLists *ev, hipStream_t s);
void free_event_lists(EventLists *ev, hipStream_t s);
// err: uint32, zeroed by the caller (bit 0: a cycle, bit 1: frontier capacity
// exceeded).  First with ref == nullptr (est is not used), the kernel that
// keeps its frontier in registers: hipErrorNotSupported where it does not take
// the call, and err bit 2 when a variant outgrew it; *keep then holds where
// each variant stopped (the caller frees it, whatever is returned).  After
// either of the two with ref: int32 [V][n] and est: int64 [V][n] as working
// memory: every variant goes on from *keep, or from the start if it is null.
hipError_t launch_sim_event(const dd_graph *g, const EventLists &ev, const dd_variants *var,
                            int32_t policy, const uint8_t *pp, const int32_t *prio, int32_t *ref,
                            int64_t *est, uint32_t **keep, int64_t *finish, int64_t *start,
                            int64_t *makespan, uint32_t *err, hipStream_t s);
constexpr int kEventQueue = 1024;      // ready tasks one variant may hold
constexpr int kEventIdBits = 22;       // tasks: n < 2^22
constexpr int kEventMaxThreads = 4096;

}  // namespace dd
