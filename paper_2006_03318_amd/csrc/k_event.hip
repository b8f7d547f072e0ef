// Simulation under an overridden schedule() (Sec. 4.4, "Schedule"; the P3
// model of the appendix).
//
// When a thread holds tasks with no recorded order among them (the push and
// pull slices a what-if recipe puts on a communication channel), the start
// times depend on which ready task schedule() picks, so the max-plus form of
// the batch kernel no longer applies.  This path runs Algorithm 1 task by
// task for every variant: the reference counts, the frontier Q of ready
// tasks, schedule(Q), the thread progress P and the children's start times.
//
// Design (one wavefront per variant, 64 threads per workgroup):
//  * the frontier lives in LDS (up to kEventQueue entries of 18 bytes,
//    structure of arrays): what schedule() reads -- id, push/pull and
//    removal flags, thread, priority, start so far.  The dispatched task's
//    record (out-edges, duration, gap, class) is read when it is picked;
//  * schedule(Q) is a wave reduction: the least time max(P[t], start), then
//    the least id among those (Q is in trace order, so that is Q's first),
//    then, for the priority rule when that task is a push/pull task, the
//    highest priority (least id among equals) over the push/pull tasks of
//    least time -- the task the paper's scan over Q ends with;
//  * the dispatched task's children are handled one per lane: a device
//    atomic decrement of the child's reference count and an atomic max of
//    its start (two edges from one parent, e.g. a dependency that repeats
//    the thread order, stay correct), with the child's metadata loaded at
//    the same time; children whose count reaches zero join Q;
//  * reference counts and starts are per-variant arrays [V][n] in device
//    memory; P for every thread and the variant's scale column (when it has
//    at most kLdsCls classes) sit in LDS.
// Each step is a chain of dependent latencies (LDS, reductions, the picked
// task's record, the children's atomics), so the rate is set by how many
// variants run at once: every variant is one wave of ~20 KB of LDS, eight
// per CU, so about 2,000 variants are resident together.
//
// Two kernels.  k_sim_event_reg, below, serves what fits it (at most 64
// threads, 512 classes, 32-bit durations, every edge class on); k_sim_event
// (described above) everything else.
#include "dd_common.h"
#include "dd_internal.h"
#include "dd_time.h"

#include <type_traits>

namespace dd {
namespace {

constexpr int kBS = 256;
constexpr int kQ = kEventQueue;
constexpr int kLdsCls = 64;        // scale columns cached in LDS up to this many classes

__device__ __forceinline__ int64_t scaled(int64_t d, const ScaleEntry &se) {
    const uint64_t a = (uint64_t)d * (uint64_t)se.p;
    return (int64_t)(se.magic ? (__umul64hi(a, se.magic) >> se.shift) : (a >> se.shift));
}

// Wave-wide minima: butterflies inside each row of 16 lanes with DPP (quad
// permutations, half-row and row mirrors), then the four row results read
// into scalar registers.  All 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
    const uint32_t lo = dpp32<CTRL>((uint32_t)x);
    const uint32_t hi = dpp32<CTRL>((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
template <class T>
__device__ __forceinline__ T tmin(T a, T b) { return b < a ? b : a; }

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t x) {
    x = tmin(x, dpp64<0xB1>(x));     // quad_perm [1,0,3,2]
    x = tmin(x, dpp64<0x4E>(x));     // quad_perm [2,3,0,1]
    x = tmin(x, dpp64<0x141>(x));    // row_half_mirror
    x = tmin(x, dpp64<0x140>(x));    // row_mirror
    return tmin(tmin(readlane_u64(x, 0), readlane_u64(x, 16)),
                tmin(readlane_u64(x, 32), readlane_u64(x, 48)));
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
    x = tmin(x, dpp32<0xB1>(x));
    x = tmin(x, dpp32<0x4E>(x));
    x = tmin(x, dpp32<0x141>(x));
    x = tmin(x, dpp32<0x140>(x));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32);
    const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return tmin(tmin(a, b), tmin(c, d));
}

__device__ __forceinline__ uint32_t pick4(const uint4 &e, int k) {
    return k == 0 ? e.x : k == 1 ? e.y : k == 2 ? e.z : e.w;
}

// ---------------------------------------------------------------------------
// out-edge lists: count per parent, scan, fill, per-task records
__global__ __launch_bounds__(kBS) void k_ev_count(int32_t n, const int64_t *__restrict__ in_ptr,
                                                  const int32_t *__restrict__ in_src,
                                                  const int32_t *__restrict__ prev,
                                                  unsigned long long *__restrict__ cnt) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u >= n) return;
    for (int64_t e = in_ptr[u]; e < in_ptr[u + 1]; e++) atomicAdd(&cnt[in_src[e]], 1ull);
    if (prev[u] >= 0) atomicAdd(&cnt[prev[u]], 1ull);
}

__global__ __launch_bounds__(kBS) void k_ev_fill(int32_t n, const int64_t *__restrict__ in_ptr,
                                                 const int32_t *__restrict__ in_src,
                                                 const uint8_t *__restrict__ in_cls,
                                                 const int32_t *__restrict__ prev,
                                                 const int64_t *__restrict__ beg,
                                                 unsigned long long *__restrict__ cur,
                                                 uint32_t *__restrict__ edges,
                                                 unsigned long long *__restrict__ mask) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u >= n) return;
    uint64_t cm = 0;
    for (int64_t e = in_ptr[u]; e < in_ptr[u + 1]; e++) {
        const int32_t s = in_src[e];
        const int64_t at = beg[s] + (int64_t)atomicAdd(&cur[s], 1ull);
        edges[at] = ((uint32_t)u << 8) | (in_cls ? (uint32_t)in_cls[e] : 0u);
        cm |= 1ull << (in_cls ? in_cls[e] : 0);
    }
    if (cm) atomic_or_hot(mask, (unsigned long long)cm);
    const int32_t p = prev[u];
    if (p >= 0) {
        const int64_t at = beg[p] + (int64_t)atomicAdd(&cur[p], 1ull);
        edges[at] = ((uint32_t)u << 8) | kEdgeAlways;
    }
}

__global__ __launch_bounds__(kBS) void k_ev_rec(int32_t n, const int64_t *__restrict__ beg,
                                                const int32_t *__restrict__ tid,
                                                const uint16_t *__restrict__ cls,
                                                const uint32_t *__restrict__ edges,
                                                int4 *__restrict__ rec, uint4 *__restrict__ e4) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u >= n) return;
    const int64_t b = beg[u];
    const int32_t k = (int32_t)(beg[u + 1] - b);
    rec[u] = make_int4((int32_t)b, k, tid[u], cls ? (int32_t)cls[u] : 0);
    e4[u] = make_uint4(k > 0 ? edges[b] : 0u, k > 1 ? edges[b + 1] : 0u,
                       k > 2 ? edges[b + 2] : 0u, k > 3 ? edges[b + 3] : 0u);
}

// ---------------------------------------------------------------------------
struct EvArgs {
    int32_t n, V, W, T, n_cls, policy;
    const int4 *__restrict__ rec;
    const uint4 *__restrict__ e4;
    const uint32_t *__restrict__ edges;
    const int64_t *__restrict__ in_ptr;    // dependency in-edges (for the first counts)
    const uint8_t *__restrict__ in_cls;
    const int32_t *__restrict__ tprev;
    const int32_t *__restrict__ tid;
    const int64_t *__restrict__ dur;
    const int64_t *__restrict__ gap;
    const ScaleEntry *__restrict__ table;  // [n_cls][V]
    const uint32_t *__restrict__ rm;       // [n][W]
    const uint64_t *__restrict__ edge_on;  // [V]
    const uint8_t *__restrict__ pp;
    const int32_t *__restrict__ prio;
    int32_t *ref;                          // [V][n]
    unsigned long long *est;               // [V][n] (times >= 0: unsigned order is the order)
    int64_t *finish, *start, *makespan;
    uint32_t *err;
    const uint32_t *keep;                  // what k_sim_event_reg left, or null (then from the start)
    int64_t keep_stride;
};

// What a variant's wave of k_sim_event_reg leaves when it stops, in words:
//   0 tasks dispatched, 1 ready tasks (kFresh: it has not begun), 2 ready and
//   waiting tasks, 4 and 5 base, 6 and 7 makespan so far, from kKeepP the
//   threads' progress, from kKeepEnt the tasks, the ready ones first:
//   { word, parents left (ready: 0), time or start so far }
// (times as differences to the base; one before it counts as it: whatever
// depends on it starts no earlier)
constexpr int kKeepP = 8, kKeepEnt = kKeepP + 64;
constexpr uint32_t kFresh = ~0u;

// A frontier entry is 18 bytes: what schedule(Q) reads.  The rest of a task
// (out-edges, duration, gap, class) is read when it is dispatched.
constexpr int kSlotBits = 10;
static_assert((1 << kSlotBits) == kQ, "slot bits");
constexpr uint32_t kIdMask = (1u << kEventIdBits) - 1u;
constexpr uint32_t kPPb = 1u << kEventIdBits;          // push/pull task
constexpr uint32_t kRMb = 1u << (kEventIdBits + 1);    // removed in this variant
static_assert(kEventIdBits + kSlotBits <= 32, "id and slot share one word");

struct Frontier {
    uint32_t a[kQ];     // id | flags
    uint16_t th[kQ];    // thread
    int32_t pr[kQ];     // priority
    int64_t est[kQ];    // start so far (final once the task is ready)
};

__device__ __forceinline__ void push_entry(Frontier &q, int32_t slot, uint32_t u, bool ppf,
                                           bool rmv, int32_t th, int32_t pr, int64_t est) {
    q.a[slot] = u | (ppf ? kPPb : 0u) | (rmv ? kRMb : 0u);
    q.th[slot] = (uint16_t)th;
    q.pr[slot] = pr;
    q.est[slot] = est;
}

template <bool TLDS>
__global__ __launch_bounds__(64) void k_sim_event(EvArgs a) {
    extern __shared__ int64_t sP[];           // [T] thread progress
    __shared__ Frontier q;
    __shared__ ScaleEntry sTab[TLDS ? kLdsCls : 1];
    const int lane = threadIdx.x;
    const int v = blockIdx.x;
    const int32_t n = a.n;
    const int64_t V = a.V;
    const uint64_t on = a.edge_on[v];
    int32_t *ref = a.ref + (int64_t)v * n;
    unsigned long long *est = a.est + (int64_t)v * n;
    const uint64_t lt = (1ull << lane) - 1ull;
    const uint32_t vbit = 1u << (v & 31);
    const int vw = v >> 5;

    const uint32_t *const kept = a.keep ? a.keep + (int64_t)v * a.keep_stride : nullptr;
    const bool resume = kept && kept[1] != kFresh;
    const int32_t before = resume ? (int32_t)kept[0] : 0;

    for (int t = lane; t < a.T; t += 64) sP[t] = 0;
    if (TLDS)
        for (int c = lane; c < a.n_cls; c += 64) sTab[c] = a.table[(int64_t)c * V + v];
    uint32_t err = 0;

    // reference counts over the active parents; tasks with none are ready
    // (a variant that has none left needs no counts)
    int32_t qn = 0;
    for (int64_t base = 0; base < n && !(resume && kept[1] == 0u); base += 64) {
        const int64_t u = base + lane;
        bool root = false;
        if (u < n) {
            int32_t r = a.tprev[u] >= 0 ? 1 : 0;
            for (int64_t e = a.in_ptr[u]; e < a.in_ptr[u + 1]; e++) {
                const uint32_t c = a.in_cls ? a.in_cls[e] : 0u;
                r += (int32_t)((on >> c) & 1ull);
            }
            ref[u] = r;
            est[u] = 0ull;
            root = r == 0 && !resume;
        }
        const uint64_t b = __ballot(root);
        if (root) {
            const int32_t slot = qn + __popcll(b & lt);
            if (slot < kQ)
                push_entry(q, slot, (uint32_t)u, a.pp ? a.pp[u] != 0 : false,
                           (a.rm[u * a.W + vw] & vbit) != 0u, a.tid[u], a.prio ? a.prio[u] : 0, 0);
            else
                err |= 2u;
        }
        qn += __popcll(b);
        if (qn > kQ) qn = kQ;
    }
    __threadfence();   // the counts are in memory before the first atomic on them
    __syncthreads();

    int64_t ms = 0;
    if (resume) {
        const int64_t base = (int64_t)((uint64_t)kept[5] << 32 | kept[4]);
        ms = (int64_t)((uint64_t)kept[7] << 32 | kept[6]);
        qn = (int32_t)kept[1];
        const int32_t cnt = (int32_t)kept[2];
        for (int32_t i = lane; i < cnt; i += 64) {
            const uint32_t *const e = kept + kKeepEnt + 3 * i;
            const int64_t u = e[0] >> 10;
            const int64_t t = base + e[2];
            if (i < qn) {
                push_entry(q, i, (uint32_t)u, a.pp ? a.pp[u] != 0 : false, (a.rm[u * a.W + vw] & vbit) != 0u,
                           a.tid[u], a.prio ? a.prio[u] : 0, t);
            } else {
                ref[u] = (int32_t)e[1];
                est[u] = (unsigned long long)t;
            }
        }
        for (int t = lane; t < a.T; t += 64) sP[t] = base + kept[kKeepP + t];
        __threadfence();
        __syncthreads();
    }
    int32_t done = 0;
    int32_t bu = 0;                 // this lane's buffered result: task, finish, start
    int64_t bf = 0, bs = 0;
    while (qn > 0) {
        // ---- schedule(Q) ----
        // One pass: per lane, the least time among its entries, the least
        // (id, slot) among its entries of that time, and the best push/pull
        // key (highest priority, then least id) among them.  Times are
        // nonnegative, so they compare as unsigned.
        uint64_t tb = ~0ull;
        uint32_t kb = 0xffffffffu;           // id << kSlotBits | slot
        uint64_t pb = ~0ull;                 // ~priority << 32 | id << kSlotBits | slot
        for (int j = 0; j * 64 < qn; j++) {
            const int i = j * 64 + lane;
            if (i < qn) {
                const int64_t p = sP[q.th[i]];
                const int64_t e = q.est[i];
                const uint64_t t = (uint64_t)(p > e ? p : e);
                const uint32_t ai = q.a[i];
                const uint32_t k = ((ai & kIdMask) << kSlotBits) | (uint32_t)i;
                const uint64_t pk = (ai & kPPb)
                    ? ((uint64_t)(~((uint32_t)q.pr[i] ^ 0x80000000u)) << 32) | k : ~0ull;
                if (t < tb) {
                    tb = t;
                    kb = k;
                    pb = pk;
                } else if (t == tb) {
                    kb = tmin(kb, k);
                    pb = tmin(pb, pk);
                }
            }
        }
        const uint64_t T0 = wave_min_u64(tb);
        const bool at = tb == T0;
        const uint32_t m1 = wave_min_u32(at ? kb : 0xffffffffu);
        int32_t ws = (int32_t)(m1 & (uint32_t)(kQ - 1));
        if (a.policy == 1 && (q.a[ws] & kPPb)) {
            // the push/pull tasks of least time: highest priority, then least id
            const uint64_t pk = wave_min_u64(at ? pb : ~0ull);
            ws = (int32_t)(pk & (uint64_t)(kQ - 1));
        }
        // ---- dispatch ----
        const uint32_t wa = __builtin_amdgcn_readfirstlane(q.a[ws]);
        const int32_t th = __builtin_amdgcn_readfirstlane((int32_t)q.th[ws]);
        const int64_t eu = q.est[ws];
        const int32_t u = (int32_t)(wa & kIdMask);
        const bool rmv = (wa & kRMb) != 0u;
        const int4 ur = a.rec[u];
        const uint4 ue4 = a.e4[u];
        const int64_t dd = a.dur[u];
        const int64_t gg = a.gap[u];
        const ScaleEntry se = TLDS ? sTab[ur.w] : a.table[(int64_t)ur.w * V + v];
        const int64_t du = rmv ? 0 : scaled(dd, se);
        const int64_t gu = rmv ? 0 : gg;
        const int64_t pt = sP[th];
        const int64_t s = pt > eu ? pt : eu;
        const int64_t f = s + du;
        const int64_t rel = f + gu;
        if (!rmv) ms = f > ms ? f : ms;
        const int32_t last = qn - 1;
        if (lane == 0) {
            // the last entry fills the dispatched one's slot
            q.a[ws] = q.a[last];
            q.th[ws] = q.th[last];
            q.pr[ws] = q.pr[last];
            q.est[ws] = q.est[last];
            sP[th] = rel;
        }
        // results go out 64 at a time, one per lane: a store in every step
        // would make each step's wait for its loads wait for the store too
        // (vector memory operations complete in order)
        if (lane == (done & 63)) {
            bu = u;
            bf = f;
            bs = s;
        }
        qn = last;
        done++;
        if ((done & 63) == 0) {
            a.finish[(int64_t)bu * V + v] = bf;
            if (a.start) a.start[(int64_t)bu * V + v] = bs;
        }
        // ---- children ----
        for (int32_t base = 0; base < ur.y; base += 64) {
            const int32_t k = base + lane;
            bool act = false;
            uint32_t pk = 0;
            if (k < ur.y) {
                pk = k < 4 ? pick4(ue4, k) : a.edges[(int64_t)ur.x + k];
                const uint32_t c = pk & 255u;
                act = c == kEdgeAlways || ((on >> c) & 1ull);
            }
            bool ready = false;
            int64_t ce = 0;
            int32_t cth = 0, cp = 0;
            bool cpp = false, crm = false;
            const int32_t c = (int32_t)(pk >> 8);
            if (act) {
                const int32_t old = atomicSub(&ref[c], 1);
                const unsigned long long oe = atomicMax(&est[c], (unsigned long long)rel);
                // what the frontier entry needs, if this was the child's last parent
                cth = a.tid[c];
                cp = a.prio ? a.prio[c] : 0;
                cpp = a.pp ? a.pp[c] != 0 : false;
                crm = (a.rm[(int64_t)c * a.W + vw] & vbit) != 0u;
                ready = old == 1;
                ce = (int64_t)oe > rel ? (int64_t)oe : rel;
            }
            const uint64_t b = __ballot(ready);
            if (ready) {
                const int32_t slot = qn + __popcll(b & lt);
                if (slot < kQ)
                    push_entry(q, slot, (uint32_t)c, cpp, crm, cth, cp, ce);
                else
                    err |= 2u;
            }
            qn += __popcll(b);
            if (qn > kQ) qn = kQ;
        }
    }
    if (lane < (done & 63)) {
        a.finish[(int64_t)bu * V + v] = bf;
        if (a.start) a.start[(int64_t)bu * V + v] = bs;
    }
    if (before + done != n) err |= 1u;
    for (int o = 32; o > 0; o >>= 1) err |= (uint32_t)__shfl_xor((int)err, o, 64);
    if (lane == 0) {
        a.makespan[v] = ms;
        if (err) atomicOr(a.err, err);
    }
}

// ---------------------------------------------------------------------------
// The same simulation with its state in registers and the task records in
// LDS: one wave per variant, up to eight variants per workgroup, which share
// one window of records.  What a step costs is the chain of latencies when
// few variants run, and the instructions of its wave when 2,048 do (two
// waves per SIMD), so both are kept short:
//   * a lane holds up to kRegK ready tasks, each as its time max(P[thread],
//     start) and one word with its id, thread and push/pull flag; dispatching
//     raises the times of its thread's other ready tasks.  Dispatch times
//     never fall, so all times are 32-bit differences to a base that moves up
//     when they pass 2^31, and schedule(Q) is a 32-bit minimum over the lanes,
//     resolved by a ballot (ties: by id, or by the priority rule);
//   * while that minimum is taken, every lane reads the record of its own
//     least task, so the winner's is there when the winner is known;
//   * after S steps S tasks are done, and tasks that become ready lie near
//     the S-th (they are numbered in trace order): the window holds
//     [S - size / 2, S + size / 2) and moves on every kRegStage steps, with
//     one barrier for all waves.  A record outside of it is read from memory;
//   * an out-edge carries its child's word and number of parents, so nothing
//     of a child is read before the child is dispatched.  A child with one
//     parent is ready at once, the first in its parent's place; the others
//     wait in kPendM places per lane (word, parents left, start so far),
//     found by a ballot; the threads' progress is one register.
// Capacity (ready and waiting tasks, times 2^31 ahead of the last dispatch)
// is not known beforehand: a wave that runs out sets error bit 2 and stops, as
// do the others when they see it, and the caller runs k_sim_event, which goes
// on from the last move of the window: at each, every wave leaves its state in
// memory.  (4,400 tasks of which the 3,990th releases 400:
// 7.2 ms in k_sim_event alone, 12.6 when it began again, 6.2 now, 30 variants.)
// What bounds it: the instructions of one wave, about 2,000 cycles a step
// (choosing the task 560, the priority rule up to 700 more, dispatch and
// raised times 620, children 750); at 2,048 variants another 650, in which a
// workgroup waits for its slowest wave.  VGG-19 with P3's slices, P3 rule,
// 14,688 tasks x 2,048 variants: 21.1 ms a call (33.7 with k_sim_event); 918
// tasks x 30 variants, default rule: 0.81 ms (1.43).
constexpr int kRegK = 4;              // ready tasks per lane
constexpr int kPendM = 4;             // waiting tasks per lane
constexpr int kRegCls = 512;          // scale entries in LDS at most (per wave)
constexpr int kRegT = 64;             // threads at most
constexpr int kRegWaves = 8;          // variants per workgroup at most
constexpr int kRegStage = 256;        // steps between moves of the window
constexpr size_t kRegLds = 160 * 1024 - 64;   // LDS of a compute unit, less the static part

// a task's word: id << 10 | thread << 4 | push/pull << 3, in the order of the
// ids; in an out-edge, with the task's parents in the low bits (kMany: that
// many or more)
static_assert(kEventIdBits + 10 <= 32 && kRegT <= 64, "the word holds them");
constexpr uint32_t kMany = 7, kWordPP = 8, kWordTh = 63u << 4;

// a task's record:
//   a = { duration, gap (below 2^32), class, priority }
//   b = { its first two out-edges, first out-edge, out-edges }
struct alignas(32) EvTask {
    uint4 a, b;
};

// (a thread per out-edge, and one per task: a task may have any number of them)
__global__ __launch_bounds__(kBS) void k_ev_task(int32_t n, int64_t n_edges, const int4 *__restrict__ rec,
                                                 const uint32_t *__restrict__ edges,
                                                 const int64_t *__restrict__ dur,
                                                 const int64_t *__restrict__ gap,
                                                 const int64_t *__restrict__ in_ptr,
                                                 const int32_t *__restrict__ prev,
                                                 const uint8_t *__restrict__ pp,
                                                 const int32_t *__restrict__ prio,
                                                 EvTask *__restrict__ out, uint32_t *__restrict__ words,
                                                 uint32_t *__restrict__ parents,
                                                 uint32_t *__restrict__ roots) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    auto count = [&](uint32_t c) {
        return (uint32_t)(in_ptr[c + 1] - in_ptr[c]) + (prev[c] >= 0 ? 1u : 0u);
    };
    auto word = [&](uint32_t c) { return c << 10 | (uint32_t)rec[c].z << 4 | ((pp && pp[c]) ? kWordPP : 0u); };
    auto edge = [&](int64_t j) {
        const uint32_t c = edges[j] >> 8, k = count(c);
        return word(c) | (k < kMany ? k : kMany);
    };
    if (u < n_edges) words[u] = edge(u);
    if (u >= n) return;
    const int4 r = rec[u];
    EvTask t;
    t.a = make_uint4((uint32_t)dur[u], (uint32_t)gap[u], (uint32_t)r.w, prio ? (uint32_t)prio[u] : 0u);
    t.b = make_uint4(r.y > 0 ? edge(r.x) : 0u, r.y > 1 ? edge((int64_t)r.x + 1) : 0u, (uint32_t)r.x, (uint32_t)r.y);
    out[u] = t;
    const uint32_t k = count((uint32_t)u);
    parents[u] = k;
    if (k == 0) roots[1 + atomicAdd(&roots[0], 1u)] = word((uint32_t)u);
}

struct EvRegArgs {
    int32_t n, V, W, n_cls, win;           // win: records of the window, a power of two
    const EvTask *__restrict__ task;
    const uint32_t *__restrict__ words;    // out-edges
    const uint32_t *__restrict__ parents;  // [n]
    const uint32_t *__restrict__ roots;    // count, then the tasks without parents
    const ScaleEntry *__restrict__ table;  // [n_cls][V]
    const uint32_t *__restrict__ rm;       // [n][W]
    int64_t *finish, *start, *makespan;
    uint32_t *err;
    uint32_t *keep;                        // [V][keep_stride]
    int64_t keep_stride;
};

// LDS of a workgroup: the window, then each wave's scale entries and removal
// bits of the window
inline size_t reg_lds(int win, int waves, int n_cls) {
    return (size_t)win * sizeof(EvTask) + (size_t)waves * (sizeof(double2) * (size_t)n_cls + (size_t)win / 8);
}

// orders by `hi`, then by `lo`
__device__ __forceinline__ uint64_t pair(uint32_t hi, uint32_t lo) {
    return (uint64_t)join64((int)lo, (int)hi);
}

template <bool START, bool PRIO>
__global__ __launch_bounds__(64 * kRegWaves) void k_sim_event_reg(EvRegArgs a) {
    extern __shared__ uint4 sWin[];           // [win][2], then per wave
    __shared__ uint32_t sStop;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    double2 *const sTab = reinterpret_cast<double2 *>(sWin + 2 * a.win) +
                          wave * (a.n_cls + a.win / 128);         // [n_cls] {p, 1/q}
    uint32_t *const sRm = reinterpret_cast<uint32_t *>(sTab + a.n_cls);   // [win / 32]
    const int v = blockIdx.x * waves + wave;
    const bool mine = v < a.V;
    const int64_t V = a.V;
    const uint32_t vbit = 1u << (v & 31);
    const uint32_t *const rmv = a.rm + (mine ? v >> 5 : 0);
    for (int c = lane; c < a.n_cls; c += 64) {
        const ScaleEntry e = a.table[(int64_t)c * V + (mine ? v : 0)];
        sTab[c] = make_double2((double)e.p, inv_quotient(e));
    }
    // tasks [t0, t1) come into the window (both multiples of 64)
    auto stage = [&](int32_t t0, int32_t t1) {
#pragma unroll 4
        for (int32_t t = t0 + (int32_t)threadIdx.x; t < t1 && t < a.n; t += (int32_t)blockDim.x) {
            const EvTask r = a.task[t];
            const int at = 2 * (t & (a.win - 1));
            sWin[at] = r.a;
            sWin[at + 1] = r.b;
        }
#pragma unroll 4
        for (int32_t t = t0; t < t1 && t < a.n; t += 64) {
            const int32_t u = t + lane;
            const uint64_t gone = __ballot(u < a.n && (rmv[(int64_t)(u < a.n ? u : 0) * a.W] & vbit));
            if (lane < 2) sRm[((t & (a.win - 1)) >> 5) + lane] = (uint32_t)(gone >> (32 * lane));
        }
    };

    uint32_t t[kRegK], key[kRegK];            // ready tasks: time, word (both ~0: free)
    uint32_t pr[kRegK];                       // priority, descending (PRIO, push/pull tasks)
    uint32_t pid[kPendM], left[kPendM];       // waiting tasks: word (~0: free), parents left,
    uint32_t pst[kPendM];                     // start so far
    uint32_t P = 0;                           // progress of thread `lane`
#pragma unroll
    for (int k = 0; k < kRegK; k++) t[k] = key[k] = pr[k] = ~0u;
#pragma unroll
    for (int m = 0; m < kPendM; m++) {
        pid[m] = ~0u;
        left[m] = pst[m] = 0u;
    }
    uint32_t err = 0;                         // (uniform)
    const bool whole = a.n <= a.win;          // the window holds every task
    int32_t lo = whole ? 0 : -(a.win / 2);    // first task of the window
    const uint32_t wmask = (uint32_t)(a.win - 1);

    // task `w`, ready at x, into place pk of lane pl; pl < 0: any free one
    auto put = [&](uint32_t w, uint32_t x, int pl, int pk) {
        if (pl < 0) {
            int fk = -1;
#pragma unroll
            for (int k = kRegK - 1; k >= 0; k--) fk = key[k] == ~0u ? k : fk;
            const uint64_t f = __ballot(fk >= 0);
            if (f == 0) {
                err = 4u;
                return;
            }
            pl = __ffsll((unsigned long long)f) - 1;
            pk = __builtin_amdgcn_readlane(fk, pl);
        }
        const int at = lane == pl ? pk : -1;
#pragma unroll
        for (int k = 0; k < kRegK; k++) {
            t[k] = at == k ? x : t[k];
            key[k] = at == k ? w : key[k];
        }
        if (PRIO && (w & kWordPP)) {
            const uint32_t c = w >> 10;
            const uint32_t d =
                c - (uint32_t)lo < (uint32_t)a.win ? sWin[2 * (c & wmask)].w : a.task[c].a.w;
#pragma unroll
            for (int k = 0; k < kRegK; k++) pr[k] = at == k ? ~(d ^ 0x80000000u) : pr[k];
        }
    };
    // one more parent of task `w` is done, at rel (it has k of them); true
    // when it was the last, est then its start
    auto arrive = [&](uint32_t w, uint32_t k, uint32_t rel, uint32_t &est) -> bool {
        est = rel;
        if (k == 1u) return true;
        int hm = -1;
        uint32_t lf = 0, ps = 0;
#pragma unroll
        for (int m = 0; m < kPendM; m++) {
            const bool h = pid[m] == w;
            hm = h ? m : hm;
            lf = h ? left[m] : lf;
            ps = h ? pst[m] : ps;
        }
        const uint64_t hit = __ballot(hm >= 0);
        if (hit == 0) {
            int fm = -1;
#pragma unroll
            for (int m = kPendM - 1; m >= 0; m--) fm = pid[m] == ~0u ? m : fm;
            const uint64_t f = __ballot(fm >= 0);
            if (f == 0) {
                err = 4u;
                return false;
            }
            if (k == kMany) k = __builtin_amdgcn_readfirstlane(a.parents[w >> 10]);
            const int at = lane == __ffsll((unsigned long long)f) - 1 ? fm : -1;
#pragma unroll
            for (int m = 0; m < kPendM; m++) {
                pid[m] = at == m ? w : pid[m];
                left[m] = at == m ? k - 1u : left[m];
                pst[m] = at == m ? rel : pst[m];
            }
            return false;
        }
        const int l = __ffsll((unsigned long long)hit) - 1;
        const uint32_t now_left = __builtin_amdgcn_readlane(lf, l) - 1u;
        const uint32_t p = __builtin_amdgcn_readlane(ps, l);
        est = p > rel ? p : rel;
        const uint32_t nw = now_left == 0u ? ~0u : w;
#pragma unroll
        for (int m = 0; m < kPendM; m++) {    // (hm: the lane that holds it only)
            pid[m] = hm == m ? nw : pid[m];
            left[m] = hm == m ? now_left : left[m];
            pst[m] = hm == m ? est : pst[m];
        }
        return now_left == 0u;
    };
    // the same for an out-edge; a child that becomes ready goes to place pk of
    // lane pl (pl < 0: any), and true is returned
    auto child = [&](uint32_t e, uint32_t rel, int pl, int pk) -> bool {
        const uint32_t w = e & ~7u;
        uint32_t est;
        if (!arrive(w, e & 7u, rel, est)) return false;
        const uint32_t p = __builtin_amdgcn_readlane(P, (w & kWordTh) >> 4);
        put(w, p > est ? p : est, pl, pk);
        return true;
    };

    int64_t base = 0, ms = 0;       // time of the 32-bit zero; makespan
    int32_t done = 0;
    // where the variant stands, for k_sim_event to go on from
    uint32_t *const kp = a.keep + (int64_t)(mine ? v : 0) * a.keep_stride;
    auto keep = [&]() {
        uint32_t c = 0;
        auto list = [&](bool is, uint32_t w, uint32_t l, uint32_t x) {
            const uint64_t b = __ballot(is);
            uint32_t *const e = kp + kKeepEnt + 3 * (c + (uint32_t)__popcll(b & ((1ull << lane) - 1ull)));
            if (is) {
                e[0] = w;
                e[1] = l;
                e[2] = x;
            }
            c += (uint32_t)__popcll(b);
        };
#pragma unroll
        for (int k = 0; k < kRegK; k++) list(key[k] != ~0u, key[k], 0u, t[k]);
        const uint32_t r = c;
#pragma unroll
        for (int m = 0; m < kPendM; m++) list(pid[m] != ~0u, pid[m], left[m], pst[m]);
        kp[kKeepP + lane] = P;
        if (lane == 0) {
            kp[0] = (uint32_t)done;
            kp[1] = r;
            kp[2] = c;
            kp[4] = (uint32_t)base;
            kp[5] = (uint32_t)((uint64_t)base >> 32);
            kp[6] = (uint32_t)ms;
            kp[7] = (uint32_t)((uint64_t)ms >> 32);
        }
    };

    stage(0, whole ? (a.n + 63) & ~63 : a.win / 2);
    __syncthreads();
    if (mine) {
        const uint32_t nr = __builtin_amdgcn_readfirstlane(a.roots[0]);
        if (lane == 0) kp[1] = kFresh;
        for (uint32_t i = 0; i < nr && !err; i++) put(__builtin_amdgcn_readfirstlane(a.roots[1 + i]), 0u, -1, 0);
    }

    uint32_t bu = 0;                // this lane's buffered result: task, finish, start
    int64_t bf = 0, bs = 0;
    bool run = mine && !err;        // (uniform per wave)
    for (int32_t S = 0; S < a.n; S += kRegStage) {
        // ---- the window moves on; every wave has done S steps or has ended ----
        if (S > 0) {
            if (mine && !err) keep();
            if (threadIdx.x == 0) sStop = load_coherent(a.err) & 4u;
            if (!whole) {
                __syncthreads();
                lo = S - a.win / 2;
                stage(S + a.win / 2 - kRegStage, S + a.win / 2);
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(sStop)) break;   // some wave ran out of room: this run is thrown away
            __syncthreads();
        }
        for (int i = 0; i < kRegStage && run; i++) {
            // ---- schedule(Q): this lane's least task, and its record ----
            uint32_t bt = t[0], bk = key[0];
            int kk = 0;
#pragma unroll
            for (int k = 1; k < kRegK; k++) {
                const bool less = pair(t[k], key[k]) < pair(bt, bk);
                bt = less ? t[k] : bt;
                bk = less ? key[k] : bk;
                kk = less ? k : kk;
            }
            uint4 ra, rb;
            uint32_t rw;
            double2 sc;
            auto record = [&](uint32_t w) {               // (one outside of the window: any other)
                const uint32_t i = (w >> 10) & wmask;
                ra = sWin[2 * i];
                rb = sWin[2 * i + 1];
                rw = sRm[i >> 5];
            };
            auto scale = [&] { sc = sTab[ra.z < (uint32_t)a.n_cls ? ra.z : 0u]; };
            record(bk);
            // ---- the least of all ----
            const uint32_t T0 = __builtin_amdgcn_readfirstlane(wave_min_u32(bt));
            if (T0 == ~0u) {                              // the frontier is empty
                run = false;
                break;
            }
            scale();
            int wl;                                       // the winner's lane
            {
                uint64_t at = __ballot(bt == T0);
                if (at & (at - 1)) at = __ballot(bk == wave_min_u32(bt == T0 ? bk : ~0u));
                wl = __ffsll((unsigned long long)at) - 1;
            }
            uint32_t wkey = __builtin_amdgcn_readlane(bk, wl);
            int wk = __builtin_amdgcn_readlane(kk, wl);
            if (PRIO && (wkey & kWordPP)) {
                // a push/pull task: of those of least time, the one of highest
                // priority, least id among equals
                uint32_t bd = ~0u, bw = ~0u;
                int bi = 0;
#pragma unroll
                for (int k = 0; k < kRegK; k++) {
                    const bool less = t[k] == T0 && (key[k] & kWordPP) &&
                                      pair(pr[k], key[k]) < pair(bd, bw);
                    bd = less ? pr[k] : bd;
                    bw = less ? key[k] : bw;
                    bi = less ? k : bi;
                }
                record(bw);
                uint64_t at = __ballot(bw != ~0u);
                const uint32_t b0 = wave_min_u32(bd);
                if (at & (at - 1)) at = __ballot(bd == b0 && bw != ~0u);
                scale();
                if (at & (at - 1)) at = __ballot(bw == wave_min_u32(bd == b0 ? bw : ~0u));
                wl = __ffsll((unsigned long long)at) - 1;
                wk = __builtin_amdgcn_readlane(bi, wl);
                wkey = __builtin_amdgcn_readlane(bw, wl);
            }
            const uint32_t id = wkey >> 10;
            if (id - (uint32_t)lo >= (uint32_t)a.win) {   // not in the window
                ra = a.task[id].a;
                rb = a.task[id].b;
                rw = (rmv[(int64_t)id * a.W] & vbit) ? ~0u : 0u;
                scale();
            }
            // ---- dispatch ----
            const bool gone = (__builtin_amdgcn_readlane(rw, wl) >> (id & 31u)) & 1u;
            const double kTop = 4294967295.0;
            const double fd = gone ? 0.0 : scale_f64((double)ra.x, sc.x, sc.y);
            const double fl = __builtin_fmin(fd + (double)T0, kTop);
            const double rl = __builtin_fmin(fl + (gone ? 0.0 : (double)ra.y), kTop);
            const uint32_t f = __builtin_amdgcn_readlane((uint32_t)fl, wl);
            const uint32_t rel = __builtin_amdgcn_readlane((uint32_t)rl, wl);
            const uint32_t ecnt = __builtin_amdgcn_readlane(rb.w, wl);
            if (rel == ~0u) {                             // too far ahead
                err = 4u;
                run = false;
                break;
            }
            const int64_t f64 = base + f;
            if (!gone) ms = f64 > ms ? f64 : ms;
            // results go out 64 at a time, one per lane
            if (lane == (done & 63)) {
                bu = id;
                bf = f64;
                bs = base + T0;
            }
            done++;
            if ((done & 63) == 0) {
                a.finish[(int64_t)bu * V + v] = bf;
                if (START) a.start[(int64_t)bu * V + v] = bs;
            }
            P = lane == (int)((wkey & kWordTh) >> 4) ? rel : P;
            const int out = lane == wl ? wk : -1;
#pragma unroll
            for (int k = 0; k < kRegK; k++) {             // (free places keep ~0)
                const uint32_t up = t[k] > rel ? t[k] : rel;
                t[k] = ((key[k] ^ wkey) & kWordTh) == 0u ? up : t[k];
                t[k] = out == k ? ~0u : t[k];
                key[k] = out == k ? ~0u : key[k];
            }
            // ---- children: the first ready one takes its parent's place ----
            if (ecnt > 0u) {
                const uint32_t e0 = __builtin_amdgcn_readlane(rb.x, wl);
                const uint32_t e1 = __builtin_amdgcn_readlane(rb.y, wl);
                const uint32_t ebeg = __builtin_amdgcn_readlane(rb.z, wl);
                if (child(e0, rel, wl, wk)) wl = -1;
                if (ecnt > 1u) {
                    if (child(e1, rel, wl, wk)) wl = -1;
                    uint32_t more = 0;
                    for (uint32_t j = 2u; j < ecnt && !err; j++) {
                        const uint32_t l = (j - 2u) & 63u;
                        if (l == 0u) {                    // 64 more out-edges, one per lane
                            const uint32_t i = j + (uint32_t)lane;
                            more = a.words[(int64_t)ebeg + (i < ecnt ? i : j)];
                        }
                        if (child(__builtin_amdgcn_readlane(more, l), rel, wl, wk)) wl = -1;
                    }
                }
            }
            if (T0 >= 1u << 31) {                         // the base moves up
                base += T0;
#pragma unroll
                for (int k = 0; k < kRegK; k++) t[k] -= key[k] == ~0u ? 0u : T0;
#pragma unroll
                for (int m = 0; m < kPendM; m++) pst[m] = pst[m] > T0 ? pst[m] - T0 : 0u;
                P = P > T0 ? P - T0 : 0u;
            }
            if (err) run = false;
        }
        if (err && lane == 0) atomicOr(a.err, err);
    }
    if (!mine) return;
    if (lane < (done & 63)) {
        a.finish[(int64_t)bu * V + v] = bf;
        if (START) a.start[(int64_t)bu * V + v] = bs;
    }
    if (done != a.n && !err) err = 1u;
    if (lane == 0) {
        a.makespan[v] = ms;
        if (err) atomicOr(a.err, err);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
hipError_t build_event_lists(const dd_graph *g, EventLists *ev, hipStream_t s) {
    const int32_t n = g->n;
    hipError_t e = hipSuccess;
    unsigned long long *cnt = nullptr;
    int64_t *beg = nullptr;
    unsigned long long *mask = nullptr;
    int64_t m = 0;
    const int blocks = grid_for(n, kBS);
#define EV_TRY(x)                  \
    do {                           \
        e = (x);                   \
        if (e != hipSuccess) goto out; \
    } while (0)
    EV_TRY(dalloc_n(&cnt, (size_t)n + 1, s));
    EV_TRY(dalloc_n(&beg, (size_t)n + 1, s));
    EV_TRY(dalloc_n(&mask, 1, s));
    EV_TRY(hipMemsetAsync(mask, 0, sizeof(unsigned long long), s));
    EV_TRY(hipMemsetAsync(cnt, 0, sizeof(unsigned long long) * ((size_t)n + 1), s));
    if (n > 0) {
        k_ev_count<<<blocks, kBS, 0, s>>>(n, g->xin_ptr, g->xin_src, g->thread_prev, cnt);
        EV_TRY(hipGetLastError());
    }
    EV_TRY(scan_exclusive((const int64_t *)cnt, beg, n, s));
    EV_TRY(hipMemcpyAsync(&m, beg + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    EV_TRY(hipStreamSynchronize(s));
    EV_TRY(dalloc_n(&ev->edges, (size_t)m + 1, s));
    EV_TRY(dalloc_n(&ev->rec, (size_t)n + 1, s));
    EV_TRY(dalloc_n(&ev->e4, (size_t)n + 1, s));
    EV_TRY(hipMemsetAsync(cnt, 0, sizeof(unsigned long long) * ((size_t)n + 1), s));
    if (n > 0) {
        k_ev_fill<<<blocks, kBS, 0, s>>>(n, g->xin_ptr, g->xin_src, g->xin_cls, g->thread_prev,
                                         beg, cnt, ev->edges, mask);
        EV_TRY(hipGetLastError());
        k_ev_rec<<<blocks, kBS, 0, s>>>(n, beg, g->thread_id, g->cls, ev->edges, ev->rec, ev->e4);
        EV_TRY(hipGetLastError());
    }
    ev->n_edges = m;
    {   // (also waits: the lists are complete before any stream uses them)
        ReadBack rb(s, sizeof(uint64_t));
        EV_TRY(rb.add(&ev->cls_mask, mask, sizeof(uint64_t)));
        EV_TRY(rb.finish());
    }
out:
#undef EV_TRY
    dfree(cnt, s);
    dfree(beg, s);
    dfree(mask, s);
    return e;
}

void free_event_lists(EventLists *ev, hipStream_t s) {
    dfree(ev->rec, s);
    dfree(ev->e4, s);
    dfree(ev->edges, s);
    *ev = EventLists();
}

hipError_t launch_sim_event(const dd_graph *g, const EventLists &ev, const dd_variants *var,
                            int32_t policy, const uint8_t *pp, const int32_t *prio, int32_t *ref,
                            int64_t *est, uint32_t **keep, int64_t *finish, int64_t *start,
                            int64_t *makespan, uint32_t *err, hipStream_t s) {
    const int64_t keep_stride = kKeepEnt + 3 * (g->n < 64 * (kRegK + kPendM) ? g->n : 64 * (kRegK + kPendM));
    if (!ref) {
        // the frontier in registers: every edge class of the graph on in
        // every variant (a task's parents are then the same in all of them),
        // 32-bit durations and gaps, times that doubles hold
        if (g->n == 0 || !var->quot_ok || g->dmax >= (int64_t(1) << 32) || g->gmax >= (int64_t(1) << 32) ||
            var->n_cls > kRegCls || g->n_threads > kRegT || (ev.cls_mask & ~var->all_mask))
            return hipErrorNotSupported;
        // the window takes most of a CU's LDS, so one workgroup runs on a CU:
        // the fewest variants per workgroup with which all run at once, and
        // the largest window that fits beside their scale tables
        int waves = 1, win = 4096;
        while (waves < kRegWaves && (int64_t)waves * 256 < var->V) waves *= 2;
        while (reg_lds(win, waves, var->n_cls) > kRegLds) win /= 2;
        EvTask *task = nullptr;
        uint32_t *words = nullptr, *parents = nullptr, *roots = nullptr;
        hipError_t e = dalloc_n(&task, (size_t)g->n, s);
        if (e == hipSuccess) e = dalloc_n(&words, (size_t)ev.n_edges + 1, s);
        if (e == hipSuccess) e = dalloc_n(&parents, (size_t)g->n, s);
        if (e == hipSuccess) e = dalloc_n(&roots, (size_t)g->n + 1, s);
        if (e == hipSuccess) e = dalloc_n(keep, (size_t)var->V * (size_t)keep_stride, s);
        if (e == hipSuccess) e = hipMemsetAsync(roots, 0, sizeof(uint32_t), s);
        if (e == hipSuccess) {
            const int64_t most = ev.n_edges > g->n ? ev.n_edges : g->n;
            k_ev_task<<<grid_for(most, kBS), kBS, 0, s>>>(g->n, ev.n_edges, ev.rec, ev.edges, g->dur, g->gap,
                                                          g->xin_ptr, g->thread_prev, pp, prio, task, words, parents,
                                                          roots);
            const EvRegArgs r{g->n, var->V, var->W, var->n_cls, win, task, words, parents, roots,
                              var->table, var->rm_bits, finish, start, makespan, err, *keep, keep_stride};
            auto go = [&](auto st, auto pr) {
                k_sim_event_reg<decltype(st)::value, decltype(pr)::value>
                    <<<(var->V + waves - 1) / waves, 64 * waves, reg_lds(win, waves, var->n_cls), s>>>(r);
            };
            const std::true_type yes{};
            const std::false_type no{};
            auto by_pr = [&](auto st) { if (policy == DD_POLICY_PRIORITY) go(st, yes); else go(st, no); };
            if (start) by_pr(yes);
            else by_pr(no);
            e = hipGetLastError();
        }
        dfree(task, s);
        dfree(words, s);
        dfree(parents, s);
        dfree(roots, s);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();             // k_sim_event alone may need less
            e = hipErrorNotSupported;
        }
        return e;
    }
    EvArgs a;
    a.keep = *keep;
    a.keep_stride = keep_stride;
    a.n = g->n;
    a.V = var->V;
    a.W = var->W;
    a.T = g->n_threads;
    a.n_cls = var->n_cls;
    a.policy = policy;
    a.rec = ev.rec;
    a.e4 = ev.e4;
    a.edges = ev.edges;
    a.in_ptr = g->xin_ptr;
    a.in_cls = g->xin_cls;
    a.tprev = g->thread_prev;
    a.tid = g->thread_id;
    a.dur = g->dur;
    a.gap = g->gap;
    a.table = var->table;
    a.rm = var->rm_bits;
    a.edge_on = var->edge_on;
    a.pp = pp;
    a.prio = prio;
    a.ref = ref;
    a.est = reinterpret_cast<unsigned long long *>(est);
    a.finish = finish;
    a.start = start;
    a.makespan = makespan;
    a.err = err;
    const size_t lds = sizeof(int64_t) * (size_t)(g->n_threads > 0 ? g->n_threads : 1);
    if (var->n_cls <= kLdsCls)
        k_sim_event<true><<<var->V, 64, lds, s>>>(a);
    else
        k_sim_event<false><<<var->V, 64, lds, s>>>(a);
    return hipGetLastError();
}

}  // namespace dd
