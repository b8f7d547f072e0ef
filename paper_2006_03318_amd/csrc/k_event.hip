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
// Two kernels.  k_sim_event_reg, below, serves what fits it; k_sim_event
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
};

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

    for (int t = lane; t < a.T; t += 64) sP[t] = 0;
    if (TLDS)
        for (int c = lane; c < a.n_cls; c += 64) sTab[c] = a.table[(int64_t)c * V + v];
    uint32_t err = 0;

    // reference counts over the active parents; tasks with none are ready
    int32_t qn = 0;
    for (int64_t base = 0; base < n; base += 64) {
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
            root = r == 0;
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
    if (done != n) err |= 1u;
    for (int o = 32; o > 0; o >>= 1) err |= (uint32_t)__shfl_xor((int)err, o, 64);
    if (lane == 0) {
        a.makespan[v] = ms;
        if (err) atomicOr(a.err, err);
    }
}

// ---------------------------------------------------------------------------
// The same simulation with the frontier in registers: a lane holds up to
// kRegK ready tasks, each with everything that dispatching it needs, so a
// step reads global memory once, for its children's records.  What a step
// costs is the chain of latencies when few variants run, and the
// instructions of its wave when 2,048 do (two waves per SIMD), so both are
// kept short:
//   * every ready task carries its time max(P[thread], start) as a double
//     (dd_time.h); dispatching raises the times of its thread's other ready
//     tasks, and schedule(Q) is one DPP minimum over the lanes, resolved by
//     a ballot (ties: by id, or by the priority rule);
//   * the lane that loads a child's record is a lane with a free place, so a
//     child that becomes ready is where it belongs; the records of its own
//     first two children are touched at once, so that they are in the CU's
//     cache when it is dispatched;
//   * a child with one parent is ready at once; the others wait in a small
//     LDS table (id -> parents done, start so far), buckets of four ids, so
//     no per-variant array of counts and starts exists and none has to be
//     cleared.
// Capacity (ready tasks, table buckets) is not known beforehand: a wave that
// runs out sets error bit 2 and stops, as do the others when they see it,
// and the caller runs k_sim_event.
// VGG-19 with P3's slices, P3 rule: 14,688 tasks x 2,048 variants 25.8 ms a
// call (33.7 with k_sim_event), x 30 variants 22.7; 918 tasks x 30 variants,
// default rule: 1.13 ms (1.43).
constexpr int kRegK = 4;              // ready tasks per lane
constexpr int kPendB = 256;           // buckets of four waiting tasks
constexpr int kRegCls = 512;          // scale entries in LDS at most
constexpr int kRegT = 1024;           // thread progress words in LDS at most
constexpr int kRegN = 32768;          // tasks whose removal bits go to LDS at most

struct alignas(64) EvTask {
    uint32_t dur, gap, ebeg, ecnt;    // duration and gap (below 2^32), out-edges
    uint32_t meta;                    // thread, push/pull << 12, class << 16
    int32_t prio;
    uint32_t parents, pad;            // all parents (every edge class on)
    uint4 e4;                         // its first four out-edges (child << 8 | class)
};

__global__ __launch_bounds__(kBS) void k_ev_task(int32_t n, const int4 *__restrict__ rec,
                                                 const uint4 *__restrict__ e4,
                                                 const int64_t *__restrict__ dur,
                                                 const int64_t *__restrict__ gap,
                                                 const int64_t *__restrict__ in_ptr,
                                                 const int32_t *__restrict__ prev,
                                                 const uint8_t *__restrict__ pp,
                                                 const int32_t *__restrict__ prio,
                                                 EvTask *__restrict__ out) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u >= n) return;
    const int4 r = rec[u];
    EvTask t;
    t.dur = (uint32_t)dur[u];
    t.gap = (uint32_t)gap[u];
    t.ebeg = (uint32_t)r.x;
    t.ecnt = (uint32_t)r.y;
    t.meta = (uint32_t)r.z | ((pp && pp[u]) ? 1u << 12 : 0u) | ((uint32_t)r.w << 16);
    t.prio = prio ? prio[u] : 0;
    t.parents = (uint32_t)(in_ptr[u + 1] - in_ptr[u]) + (prev[u] >= 0 ? 1u : 0u);
    t.pad = 0;
    t.e4 = e4[u];
    out[u] = t;
}

struct EvRegArgs {
    int32_t n, V, W, T, n_cls;
    const EvTask *__restrict__ task;
    const uint32_t *__restrict__ edges;
    const ScaleEntry *__restrict__ table;  // [n_cls][V]
    const uint32_t *__restrict__ rm;       // [n][W]
    const uint32_t *__restrict__ rmb;      // [V][rmb_stride] removal bits by task, or null
    int64_t rmb_stride;
    int64_t *finish, *start, *makespan;
    uint32_t *err;
};

// minimum over the wave (every lane active), in lane 63
template <int CTRL, int RMASK>
__device__ __forceinline__ double dpp_min_step(double x) {
    const int64_t b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)b, (int)(uint32_t)b, CTRL, RMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)((uint64_t)b >> 32), (int)((uint64_t)b >> 32), CTRL,
                                               RMASK, 0xf, false);
    return __builtin_fmin(x, __longlong_as_double(join64(lo, hi)));
}
__device__ __forceinline__ double wave_min_f64(double x) {
    x = dpp_min_step<0x111, 0xf>(x);
    x = dpp_min_step<0x112, 0xf>(x);
    x = dpp_min_step<0x114, 0xf>(x);
    x = dpp_min_step<0x118, 0xf>(x);
    x = dpp_min_step<0x142, 0xa>(x);
    x = dpp_min_step<0x143, 0xc>(x);
    return __longlong_as_double(readlane64(__double_as_longlong(x), 63));
}

// one place of the frontier
struct EvSlot {
    double t, dp;          // time (infinite: free), duration as transformed
    uint32_t id, gap;      // id: task | kPPb | kRMb; gap as transformed
    uint32_t th, ebeg, ecnt;
    int32_t pr;
    uint4 e4;
};

template <bool START, bool PRIO, bool RLDS>
__global__ __launch_bounds__(64, 2) void k_sim_event_reg(EvRegArgs a) {
    __shared__ __align__(16) uint32_t pKey[kPendB * 4];   // waiting tasks: id + 1 (0: free)
    __shared__ uint32_t pCnt[kPendB * 4];     // parents done
    __shared__ unsigned long long pEst[kPendB * 4];   // start so far (times as double bits)
    extern __shared__ double sLds[];          // [T] thread progress, [n_cls] {p, 1/q}, removal bits
    double *const sP = sLds;
    double2 *const sTab = reinterpret_cast<double2 *>(sLds + ((a.T + 1) & ~1));
    uint32_t *const sRm = reinterpret_cast<uint32_t *>(sTab + a.n_cls);
    const int lane = threadIdx.x;
    const int v = blockIdx.x;
    const int64_t V = a.V;
    const uint32_t vbit = 1u << (v & 31);
    const uint32_t *const rmv = a.rm + (v >> 5);
    const double kInf = __longlong_as_double(0x7ff0000000000000ll);
    const double kZero = 4503599627370496.0;  // 2^52: time zero (dd_time.h)
    for (int t = lane; t < a.T; t += 64) sP[t] = kZero;
    for (int c = lane; c < a.n_cls; c += 64) {
        const ScaleEntry e = a.table[(int64_t)c * V + v];
        sTab[c] = make_double2((double)e.p, inv_quotient(e));
    }
    if (RLDS)
        for (int i = lane; i < (a.n + 31) / 32; i += 64) sRm[i] = a.rmb[(int64_t)v * a.rmb_stride + i];
    for (int i = lane; i < kPendB * 4; i += 64) {
        pKey[i] = 0;
        pCnt[i] = 0;
        pEst[i] = 0;
    }
    __syncthreads();

    EvSlot s[kRegK];
#pragma unroll
    for (int k = 0; k < kRegK; k++) {
        s[k].t = kInf;
        s[k].id = ~0u;
        s[k].th = ~0u;
        s[k].dp = 0;
        s[k].gap = s[k].ebeg = s[k].ecnt = 0;
        s[k].pr = 0;
        s[k].e4 = make_uint4(0u, 0u, 0u, 0u);
    }
    uint32_t err = 0;
    uint32_t touch0 = 0, touch1 = 0;
    // a lane takes task c, ready at `est`, into place k
    auto fill = [&](EvSlot &z, uint32_t c, const uint4 &w0, const uint4 &w1, const uint4 &w2,
                    uint32_t rmw, double est) {
        const bool gone = RLDS ? (sRm[c >> 5] >> (c & 31)) & 1u : (rmw & vbit) != 0u;
        const double2 sc = sTab[w1.x >> 16];
        z.th = w1.x & 0xfffu;
        const double p = sP[z.th];
        z.t = __builtin_fmax(p, est);
        z.dp = gone ? 0.0 : scale_f64((double)w0.x, sc.x, sc.y);
        z.gap = gone ? 0u : w0.y;
        z.id = c | ((w1.x & (1u << 12)) ? kPPb : 0u) | (gone ? kRMb : 0u);
        z.ebeg = w0.z;
        z.ecnt = w0.w;
        z.pr = (int32_t)w1.y;
        z.e4 = w2;
    };
    auto words = [&](uint32_t c, uint4 &w0, uint4 &w1, uint4 &w2, uint32_t &rmw) {
        const uint4 *r = reinterpret_cast<const uint4 *>(a.task + c);
        w0 = r[0];
        w1 = r[1];
        w2 = r[2];
        rmw = RLDS ? 0u : rmv[(int64_t)c * a.W];
    };

    // tasks without parents
    for (int32_t base = 0; base < a.n; base += 64) {
        const int32_t u = base + lane;
        const bool root = u < a.n && a.task[u < a.n ? u : 0].parents == 0u;
        uint64_t todo = __ballot(root);
        while (todo) {
            int kk = -1;
            uint64_t fr = 0;
#pragma unroll
            for (int k = kRegK - 1; k >= 0; k--) {
                const uint64_t f = __ballot(s[k].t == kInf);
                if (f) { kk = k; fr = f; }
            }
            if (kk < 0) { err |= 4u; break; }
            // the r-th free lane takes the r-th root of the block
            const int r = __popcll(fr & ((1ull << lane) - 1ull));
            const bool mine = ((fr >> lane) & 1ull) && r < __popcll(todo);
            uint64_t m = todo;
            int at = 0;
            for (int i = 0; i <= r && m; i++) {
                at = __ffsll((unsigned long long)m) - 1;
                m &= m - 1;
            }
            if (mine) {
                uint4 w0, w1, w2;
                uint32_t rw;
                words((uint32_t)(base + at), w0, w1, w2, rw);
#pragma unroll
                for (int k = 0; k < kRegK; k++)
                    if (k == kk) fill(s[k], (uint32_t)(base + at), w0, w1, w2, rw, kZero);
            }
            int took = __popcll(fr) < __popcll(todo) ? __popcll(fr) : __popcll(todo);
            for (; took > 0; took--) todo &= todo - 1;
        }
        if (err) break;
    }

    double ms = kZero;
    int32_t done = 0;
    uint32_t bu = 0;                // this lane's buffered result: task, finish, start
    double bf = kZero, bs = kZero;
    err = __any(err != 0u) ? 4u : 0u;
    while (!err) {
        // ---- schedule(Q) ----
        double tl = s[0].t;
#pragma unroll
        for (int k = 1; k < kRegK; k++) tl = __builtin_fmin(tl, s[k].t);
        const double T0 = wave_min_f64(tl);
        if (T0 == kInf) break;                            // the frontier is empty
        uint32_t key = ~0u;                               // least id of the lane's tasks of that time
#pragma unroll
        for (int k = 0; k < kRegK; k++) {
            const uint32_t i = s[k].t == T0 ? s[k].id & kIdMask : ~0u;
            key = i < key ? i : key;
        }
        uint32_t wid;
        {
            const uint64_t at = __ballot(key != ~0u);
            if ((at & (at - 1)) == 0) wid = __builtin_amdgcn_readlane(key, __ffsll((unsigned long long)at) - 1);
            else wid = wave_min_u32(key);
        }
        if (PRIO) {
            // when it is a push/pull task: of those of least time, the one of
            // highest priority, least id among equals
            bool ppw = false;
#pragma unroll
            for (int k = 0; k < kRegK; k++) ppw |= s[k].t == T0 && s[k].id == ((s[k].id & kRMb) | kPPb | wid);
            if (__any(ppw)) {
                uint32_t best = ~0u;                      // descending priority
#pragma unroll
                for (int k = 0; k < kRegK; k++) {
                    const uint32_t d = ~((uint32_t)s[k].pr ^ 0x80000000u);
                    if (s[k].t == T0 && (s[k].id & kPPb) && d < best) best = d;
                }
                const uint32_t b0 = wave_min_u32(best);
                key = ~0u;
#pragma unroll
                for (int k = 0; k < kRegK; k++) {
                    const uint32_t d = ~((uint32_t)s[k].pr ^ 0x80000000u);
                    const uint32_t i = s[k].t == T0 && (s[k].id & kPPb) && d == b0 ? s[k].id & kIdMask : ~0u;
                    key = i < key ? i : key;
                }
                const uint64_t at = __ballot(key != ~0u);
                if ((at & (at - 1)) == 0)
                    wid = __builtin_amdgcn_readlane(key, __ffsll((unsigned long long)at) - 1);
                else
                    wid = wave_min_u32(key);
            }
        }
        // ---- dispatch: the winner's fields, uniform ----
        uint32_t id = 0, th = 0, ebeg = 0, ecnt = 0, gp = 0, x0 = 0, x1 = 0, x2 = 0, x3 = 0;
        double dp = 0;
#pragma unroll
        for (int k = 0; k < kRegK; k++) {
            const uint64_t at = __ballot(s[k].t == T0 && (s[k].id & kIdMask) == wid);
            if (at) {
                const int l = __ffsll((unsigned long long)at) - 1;
                id = __builtin_amdgcn_readlane(s[k].id, l);
                th = __builtin_amdgcn_readlane(s[k].th, l);
                ebeg = __builtin_amdgcn_readlane(s[k].ebeg, l);
                ecnt = __builtin_amdgcn_readlane(s[k].ecnt, l);
                gp = __builtin_amdgcn_readlane(s[k].gap, l);
                x0 = __builtin_amdgcn_readlane(s[k].e4.x, l);
                x1 = __builtin_amdgcn_readlane(s[k].e4.y, l);
                x2 = __builtin_amdgcn_readlane(s[k].e4.z, l);
                x3 = __builtin_amdgcn_readlane(s[k].e4.w, l);
                dp = __longlong_as_double(readlane64(__double_as_longlong(s[k].dp), l));
                if (lane == l) s[k].t = kInf;
            }
        }
        const double f = T0 + dp;
        const double rel = f + (double)gp;
        if (!(id & kRMb)) ms = __builtin_fmax(ms, f);
        // results go out 64 at a time, one per lane
        if (lane == (done & 63)) {
            bu = wid;
            bf = f;
            bs = T0;
        }
        done++;
        if ((done & 63) == 0) {
            a.finish[(int64_t)bu * V + v] = Tm<true>::to_time(__double_as_longlong(bf));
            if (START) a.start[(int64_t)bu * V + v] = Tm<true>::to_time(__double_as_longlong(bs));
            // another wave ran out of room: this run is thrown away
            if (load_coherent(a.err) & 4u) break;
        }
        sP[th] = rel;
#pragma unroll
        for (int k = 0; k < kRegK; k++)
            s[k].t = s[k].th == th ? __builtin_fmax(s[k].t, rel) : s[k].t;   // (free places stay infinite)
        // ---- children ----
        for (uint32_t base = 0; base < ecnt;) {
            int kk = -1;
            uint64_t fr = 0;
#pragma unroll
            for (int k = kRegK - 1; k >= 0; k--) {
                const uint64_t z = __ballot(s[k].t == kInf);
                if (z) { kk = k; fr = z; }
            }
            if (kk < 0) { err = 4u; break; }
            const uint32_t r = base + (uint32_t)__popcll(fr & ((1ull << lane) - 1ull));
            const bool mine = ((fr >> lane) & 1ull) && r < ecnt;
            base += (uint32_t)__popcll(fr);
            uint32_t c = (r == 0 ? x0 : r == 1 ? x1 : r == 2 ? x2 : x3) >> 8;
            if (ecnt > 4u) {
                if (mine && r >= 4u) c = a.edges[(int64_t)ebeg + r] >> 8;
            }
            bool ready = false;
            if (mine) {
                uint4 w0, w1, w2;
                uint32_t rw;
                words(c, w0, w1, w2, rw);
                double est = rel;
                ready = w1.z == 1u;
                if (!ready) {
                    // find the child in its bucket, or take a free word there
                    const uint32_t b = (c >> 1) & (kPendB - 1);
                    uint32_t *const kb = pKey + b * 4u;
                    const uint32_t k0 = kb[0], k1 = kb[1], k2 = kb[2], k3 = kb[3];
                    int e = k0 == c + 1u ? 0 : k1 == c + 1u ? 1 : k2 == c + 1u ? 2 : k3 == c + 1u ? 3 : -1;
                    for (int i = 0; i < 4 && e < 0; i++) {
                        const uint32_t was = atomicCAS(&kb[i], 0u, c + 1u);
                        if (was == 0u || was == c + 1u) e = i;
                    }
                    if (e < 0) {
                        err = 4u;
                    } else {
                        const uint32_t p = b * 4u + (uint32_t)e;
                        // (bit patterns of nonnegative doubles order as integers)
                        const unsigned long long oe =
                            atomicMax(&pEst[p], (unsigned long long)__double_as_longlong(rel));
                        const uint32_t before = atomicAdd(&pCnt[p], 1u);
                        if (before + 1u == w1.z) {        // its last parent: out of the table
                            ready = true;
                            est = __builtin_fmax(rel, __longlong_as_double((long long)oe));
                            pCnt[p] = 0;
                            pEst[p] = 0;
                            kb[e] = 0;
                        }
                    }
                }
                if (ready) {
#pragma unroll
                    for (int k = 0; k < kRegK; k++)
                        if (k == kk) fill(s[k], c, w0, w1, w2, rw, est);
                    // bring the records of its first two children into the cache
                    asm volatile("" ::"v"(touch0), "v"(touch1));   // (of an earlier step)
                    touch0 = a.task[w2.x >> 8].dur;
                    touch1 = a.task[w2.y >> 8].dur;
                }
            }
            if (__any(err != 0u)) { err = 4u; break; }
        }
        if (__any(err != 0u)) { err = 4u; break; }
    }
    if (lane < (done & 63)) {
        a.finish[(int64_t)bu * V + v] = Tm<true>::to_time(__double_as_longlong(bf));
        if (START) a.start[(int64_t)bu * V + v] = Tm<true>::to_time(__double_as_longlong(bs));
    }
    if (done != a.n && !err) err = 1u;
    if (lane == 0) {
        a.makespan[v] = Tm<true>::to_time(__double_as_longlong(ms));
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
                            int64_t *est, int64_t *finish, int64_t *start, int64_t *makespan,
                            uint32_t *err, hipStream_t s) {
    if (!ref) {
        // the frontier in registers: every edge class of the graph on in
        // every variant (a task's parents are then the same in all of them),
        // 32-bit durations and gaps, times that doubles hold
        if (g->n == 0 || !var->quot_ok || g->dmax >= (int64_t(1) << 32) || g->gmax >= (int64_t(1) << 32) ||
            var->n_cls > kRegCls || g->n_threads > kRegT || (ev.cls_mask & ~var->all_mask))
            return hipErrorNotSupported;
        EvTask *task = nullptr;
        hipError_t e = dalloc_n(&task, (size_t)g->n, s);
        if (e != hipSuccess) return e;
        k_ev_task<<<grid_for(g->n, kBS), kBS, 0, s>>>(g->n, ev.rec, ev.e4, g->dur, g->gap, g->xin_ptr,
                                                     g->thread_prev, pp, prio, task);
        const bool rlds = g->n <= kRegN;
        const int64_t stride = (g->n + 63) / 64 * 2;
        uint32_t *rmb = nullptr;
        if (rlds) {
            e = dalloc_n(&rmb, (size_t)var->V * (size_t)stride, s);
            if (e == hipSuccess)
                e = launch_rm_bits(g->n, var->V, var->W, stride, nullptr, var->rm_bits, rmb, s);
            if (e != hipSuccess) {
                dfree(task, s);
                dfree(rmb, s);
                return e;
            }
        }
        EvRegArgs r{g->n, var->V, var->W, g->n_threads, var->n_cls, task, ev.edges, var->table,
                    var->rm_bits, rmb, stride, finish, start, makespan, err};
        const size_t lds = sizeof(double) * (size_t)((g->n_threads + 1) & ~1) +
                           sizeof(double2) * (size_t)var->n_cls + (rlds ? sizeof(uint32_t) * (size_t)stride : 0);
        auto go = [&](auto st, auto pr, auto rl) {
            k_sim_event_reg<decltype(st)::value, decltype(pr)::value, decltype(rl)::value>
                <<<var->V, 64, lds, s>>>(r);
        };
        const std::true_type yes{};
        const std::false_type no{};
        auto by_rl = [&](auto st, auto pr) { if (rlds) go(st, pr, yes); else go(st, pr, no); };
        auto by_pr = [&](auto st) { if (policy == DD_POLICY_PRIORITY) by_rl(st, yes); else by_rl(st, no); };
        if (start) by_pr(yes);
        else by_pr(no);
        e = hipGetLastError();
        dfree(task, s);
        dfree(rmb, s);
        return e;
    }
    EvArgs a;
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
