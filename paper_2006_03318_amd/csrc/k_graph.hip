// Graph load: validation, thread-chain ranking, cross-thread edge lists,
// plus the prefix-sum utility used across the library.
//
// The task graph is the one of Sec. 4.2: tasks with an execution thread,
// duration and gap (Sec. 4.2.1) and the dependency types of Sec. 4.2.2.
// Consecutive tasks on one thread are ordered (a dependency type itself);
// the chain of each thread is ranked here by pointer jumping so that every
// later kernel can address "position p on thread t".  A dependency between
// two tasks of the same thread is implied by the thread order (release
// times never decrease along a thread) and is dropped after checking that
// it points forward.

#include "dd_common.h"
#include "dd_internal.h"

namespace dd {

// ---------------------------------------------------------------------------
// exclusive scan (three passes: chunk sums, scan of sums, apply)
namespace {
constexpr int kScanBS = 256;
constexpr int kScanIPT = 16;
constexpr int64_t kScanChunk = kScanBS * kScanIPT;

__global__ __launch_bounds__(kScanBS) void k_scan_chunk_sums(const int64_t *in, int64_t n,
                                                             int64_t *csum) {
    const int64_t lo = (int64_t)blockIdx.x * kScanChunk;
    const int64_t hi = lo + kScanChunk < n ? lo + kScanChunk : n;
    int64_t s = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kScanBS) s += in[i];
    int64_t tot;
    (void)block_excl_scan<kScanBS>(s, &tot);
    if (threadIdx.x == 0) csum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_chunk_offsets(int64_t *csum, int64_t nc,
                                                             int64_t *out_total) {
    int64_t carry = 0;
    for (int64_t base = 0; base < nc; base += 1024) {
        int64_t i = base + threadIdx.x;
        int64_t v = i < nc ? csum[i] : 0;
        int64_t tot;
        int64_t ex = block_excl_scan<1024>(v, &tot);
        if (i < nc) csum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) *out_total = carry;
}

__global__ __launch_bounds__(kScanBS) void k_scan_apply(const int64_t *in, int64_t n,
                                                        const int64_t *coff, int64_t *out) {
    const int64_t lo = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanIPT;
    int64_t v[kScanIPT];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanIPT; k++) {
        v[k] = (lo + k < n) ? in[lo + k] : 0;
        s += v[k];
    }
    int64_t tot;
    int64_t ex = block_excl_scan<kScanBS>(s, &tot) + coff[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanIPT; k++) {
        if (lo + k < n) out[lo + k] = ex;
        ex += v[k];
    }
}
}  // namespace

int64_t scan_temp_count(int64_t n) {
    const int64_t nc = (n + kScanChunk - 1) / kScanChunk;
    return nc < 1 ? 1 : nc;
}

hipError_t scan_exclusive_ws(const int64_t *in, int64_t *out, int64_t n, int64_t *csum,
                             hipStream_t s) {
    const int64_t nc = scan_temp_count(n);
    if (n > 0) k_scan_chunk_sums<<<(unsigned)nc, kScanBS, 0, s>>>(in, n, csum);
    // (with n == 0 the single chunk sum is never read: the offsets pass
    // scans one chunk of zero tasks)
    k_scan_chunk_offsets<<<1, 1024, 0, s>>>(csum, n > 0 ? nc : 0, out + n);
    if (n > 0) k_scan_apply<<<(unsigned)nc, kScanBS, 0, s>>>(in, n, csum, out);
    return hipGetLastError();
}

hipError_t scan_exclusive(const int64_t *in, int64_t *out, int64_t n, hipStream_t s) {
    int64_t *csum = nullptr;
    hipError_t e = dalloc_n(&csum, (size_t)scan_temp_count(n), s);
    if (e != hipSuccess) return e;
    e = scan_exclusive_ws(in, out, n, csum, s);
    dfree(csum, s);
    return e;
}

// ---------------------------------------------------------------------------
// The passes of dd_graph_load, in the order they run (load_device below):
//   k_load_nodes   per task: copy the fields into the graph, check them, sum
//                  the statistics, claim the thread predecessor;
//   k_load_tiles   per tile of 1,024 tasks: check the in-edges, rank the
//                  chains inside the tile;
//   k_load_exits   one workgroup: rank the tile exits, lay out the threads;
//   k_cross_count  ranks and order of all tasks, cross-thread edges per chunk;
//   k_cross_fill   the cross-thread in-edge lists.
// Small graphs are bound by the launches and host waits (a load was some 27
// launches, 10 copies, 6 fills and 5 waits, 0.2 ms for 1,612 tasks; five
// launches, a fill and two waits now), so every pass does all that its inputs
// allow, nothing comes back to the host before the end but the edge count,
// and results are written straight into the pinned read-back buffer.  Large graphs: each pass is bound by HBM.
namespace {
constexpr int kBS = 256;

constexpr int kValBlocks = 512;    // grid-stride blocks: one set of atomics per block

// what the passes share besides the graph
struct LoadWork {
    int64_t *in_ptr;               // [n+1] dependency in-edges: the call's own copies
    int32_t *in_src;
    uint8_t *ecls;                 // null: all class 0
    int32_t *succ;                 // [n] successor on the thread + 1 (zeroed)
    int32_t *heads;                // [T] first tasks (zeroed)
    int32_t *last;                 // [T] last task + 1 (zeroed)
    int32_t *xslot;                // [n] number of a tile exit + 1 (zeroed)
    uint32_t *err;                 // [2] error bits; more exits than one workgroup ranks (zeroed)
    int32_t *xcount;               // [1] tile exits (zeroed)
    LoadStats *st;                 // (zeroed)
    int32_t *dloc, *ext;           // [n] distance to, and id of, the task the tile leaves by
    int32_t *xlist, *xrank;        // [kRankXMax] the exits and their ranks
    int64_t *csum;                 // [kChunks] cross-thread edges per chunk of tasks
    LoadOut *out;                  // host memory
};

// An element of the caller's arrays is read once: what is checked is what is
// kept, and the later passes index by the copies alone, whatever the caller
// writes to the arrays meanwhile.
template <class T>
__device__ __forceinline__ void keep_own(const T *src, T *dst, int64_t u, T x) {
    if (dst != src) dst[u] = x;
}

// use(k, load(k)) for a task's edges, eight loads in flight where there are as
// many: one task may wait for all others (150,000 in-edges of one task, a
// load's walks over them: 101 ms with one edge at a time, 66 in eights)
template <class Load, class Use>
__device__ __forceinline__ void each_edge(int64_t k, int64_t k1, Load load, Use use) {
    for (; k + 8 <= k1; k += 8) {
        decltype(load(k)) x[8];
#pragma unroll
        for (int z = 0; z < 8; z++) x[z] = load(k + z);
#pragma unroll
        for (int z = 0; z < 8; z++) use(k + z, x[z]);
    }
    for (; k < k1; k++) use(k, load(k));
}
struct EdgeIn {
    int32_t src, tid;
    uint32_t cls;
};

__global__ __launch_bounds__(kBS) void k_load_nodes(
    int32_t n, int32_t T, const int32_t *s_prev, const int32_t *s_tid, const int64_t *s_dur,
    const int64_t *s_gap, const uint16_t *s_cls, const int64_t *s_ptr, int32_t *prev, int32_t *tid,
    int64_t *dur, int64_t *gap, uint16_t *cls, LoadWork w, bool one_head) {
    uint32_t e = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const int64_t end = s_ptr[n];
        keep_own(s_ptr, w.in_ptr, n, end);
        w.out->ends[1] = end;
    }
    // sums split at bit 32 so that no partial sum can overflow
    int64_t dhi = 0, dlo = 0, ghi = 0, glo = 0, dm = 0, gm = 0, cm = 0;
    for (int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x; u < n;
         u += (int64_t)gridDim.x * kBS) {
        // (all loads before the stores, which might alias them: one trip to
        // memory, not one per field)
        const int32_t t = s_tid[u], p = s_prev[u];
        int64_t d = s_dur[u], g = s_gap[u];
        const int64_t k0 = s_ptr[u], k1 = s_ptr[u + 1];
        const uint16_t c16 = s_cls ? s_cls[u] : (uint16_t)0;
        keep_own(s_tid, tid, u, t);
        keep_own(s_prev, prev, u, p);
        keep_own(s_dur, dur, u, d);
        keep_own(s_gap, gap, u, g);
        keep_own(s_ptr, w.in_ptr, u, k0);
        keep_own(s_cls, cls, u, c16);
        const bool t_ok = t >= 0 && t < T;
        if (!t_ok) e |= ERR_THREAD_RANGE;
        if (p < -1 || p >= n || p == u) {
            e |= ERR_PREV_RANGE;
        } else if (p >= 0) {
            w.succ[p] = (int32_t)u + 1;        // one claimer wins; the others are found later
        } else if (t_ok && one_head) {
            if (atomicAdd(&w.heads[t], 1) != 0) e |= ERR_HEADS;
        }
        if (d < 0 || g < 0) e |= ERR_NEG_TIME;
        if (d >= kTimeLimit || g >= kTimeLimit) e |= ERR_BIG_TIME;
        if (d < 0 || d >= kTimeLimit) d = 0;
        if (g < 0 || g >= kTimeLimit) g = 0;
        if (u == 0) w.out->ends[0] = k0;
        if (k1 < k0) e |= ERR_PTR_ORDER;
        const int64_t c = c16;
        dhi += d >> 32; dlo += d & 0xffffffffll;
        ghi += g >> 32; glo += g & 0xffffffffll;
        dm = d > dm ? d : dm;
        gm = g > gm ? g : gm;
        cm = c > cm ? c : cm;
    }
    // wave reduction, then the block's waves through LDS, one atomic set per block
    dhi = wave_sum64(dhi); dlo = wave_sum64(dlo);
    ghi = wave_sum64(ghi); glo = wave_sum64(glo);
    dm = wave_max64(dm); gm = wave_max64(gm); cm = wave_max64(cm);
    for (int o = 32; o > 0; o >>= 1) e |= (uint32_t)__shfl_xor((int)e, o, 64);
    constexpr int NW = kBS / 64;
    __shared__ int64_t red[8][NW];
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = dhi; red[1][wv] = dlo; red[2][wv] = ghi; red[3][wv] = glo;
        red[4][wv] = dm; red[5][wv] = cm; red[6][wv] = e; red[7][wv] = gm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < NW; i++) {
            dhi += red[0][i]; dlo += red[1][i]; ghi += red[2][i]; glo += red[3][i];
            dm = red[4][i] > dm ? red[4][i] : dm;
            cm = red[5][i] > cm ? red[5][i] : cm;
            e |= (uint32_t)red[6][i];
            gm = red[7][i] > gm ? red[7][i] : gm;
        }
        if (dhi) atomicAdd(&w.st->dsum_hi, (unsigned long long)dhi);
        if (dlo) atomicAdd(&w.st->dsum_lo, (unsigned long long)dlo);
        if (ghi) atomicAdd(&w.st->gsum_hi, (unsigned long long)ghi);
        if (glo) atomicAdd(&w.st->gsum_lo, (unsigned long long)glo);
        atomic_max_hot(&w.st->dmax, (unsigned long long)dm);
        atomic_max_hot(&w.st->gmax, (unsigned long long)gm);
        atomic_max_hot(&w.st->cls_max, (unsigned long long)cm);
        atomic_or_hot(w.err, e);
    }
}

// pointer jumping (Wyllie): rank = number of predecessors on the thread
__global__ __launch_bounds__(kBS) void k_rank_init(int32_t n, const int32_t *__restrict__ prev,
                                                   int32_t *__restrict__ nxt,
                                                   int32_t *__restrict__ rank) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u < n) {
        nxt[u] = prev[u];
        rank[u] = prev[u] >= 0 ? 1 : 0;
    }
}

__global__ __launch_bounds__(kBS) void k_rank_step(int32_t n, const int32_t *__restrict__ nxt_in,
                                                   const int32_t *__restrict__ rank_in,
                                                   int32_t *__restrict__ nxt_out,
                                                   int32_t *__restrict__ rank_out) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u < n) {
        const int32_t p = nxt_in[u];
        if (p >= 0) {
            // unsigned: a looping chain (reported afterwards) must not overflow
            rank_out[u] = (int32_t)((uint32_t)rank_in[u] + (uint32_t)rank_in[p]);
            nxt_out[u] = nxt_in[p];
        } else {
            rank_out[u] = rank_in[u];
            nxt_out[u] = -1;
        }
    }
}

__global__ __launch_bounds__(kBS) void k_rank_check(int32_t n, const int32_t *__restrict__ nxt,
                                                    uint32_t *__restrict__ err) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    bool bad = u < n && nxt[u] != -1;
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(err, ERR_CHAIN_CYCLE);
}

// Chain ranking in two levels.  Tasks of a thread are mostly close in id
// (traces interleave a few threads), so a tile of kRankTile consecutive ids
// resolves most of each chain with pointer jumping in LDS: every task gets
// d (predecessors up to and including the first one outside the tile) and
// e (that outside task, -1 if the chain starts in the tile), so that
// rank(u) = d + rank(e).  The outside tasks named as e (the tile exits) are
// numbered by the one task of each chain that leaves its tile and ranked by
// one workgroup, again by pointer jumping in LDS.  A thread order that loops
// inside a tile or across exits is reported like the plain pointer jumping
// does.
constexpr int kRankTile = 1024;
constexpr int kRankXMax = 8192;     // tile exits ranked in LDS at most

// (every index is clamped to its array: the errors of k_load_nodes have not
// been read; also reports a task named as previous task by two tasks, which
// left only one of them in succ)
__global__ __launch_bounds__(kRankTile) void k_load_tiles(int32_t n, int32_t T, int64_t E,
                                                          const int32_t *__restrict__ prev,
                                                          const int32_t *__restrict__ tid,
                                                          const int32_t *s_src, const uint8_t *s_ecls,
                                                          LoadWork w) {
    __shared__ int32_t sn[2][kRankTile], sd[2][kRankTile], se[2][kRankTile];
    const int64_t b0 = (int64_t)blockIdx.x * kRankTile;
    const int i = threadIdx.x;
    const int64_t u = b0 + i;
    const bool ok = u < n;
    int32_t p = ok ? prev[u] : -1;
    if (p < -1 || p >= n || p == u) p = -1;   // reported by the per-task pass
    uint32_t er = 0;
    if (ok) {
        if (p >= 0 && w.succ[p] != (int32_t)u + 1) er |= ERR_SUCC;
        const int32_t t = tid[u];
        if (p >= 0 && tid[p] != t) er |= ERR_PREV_THREAD;
        if (w.succ[u] == 0 && t >= 0 && t < T) w.last[t] = (int32_t)u + 1;
        const int64_t k0 = w.in_ptr[u] > 0 ? w.in_ptr[u] : 0;
        const int64_t k1 = w.in_ptr[u + 1] < E ? w.in_ptr[u + 1] : E;
        if (w.in_ptr[u + 1] < w.in_ptr[u]) er |= ERR_PTR_ORDER;
        // (offsets that go back and forth give every task up to all the edges:
        // refused already, and hours of work at the limits of sizes)
        const bool listed = !(load_coherent(w.err) & ERR_PTR_ORDER);
        each_edge(k0, listed ? k1 : k0,
                  [&](int64_t k) { return EdgeIn{s_src[k], 0, w.ecls ? s_ecls[k] : 0u}; },
                  [&](int64_t k, const EdgeIn &x) {
                      keep_own(s_src, w.in_src, k, x.src);
                      if (w.ecls) keep_own(s_ecls, w.ecls, k, (uint8_t)x.cls);
                      if (x.src < 0 || x.src >= n) er |= ERR_SRC_RANGE;
                      else if (x.src == u) er |= ERR_SELF_LOOP;
                      if (x.cls >= 64) er |= ERR_EDGE_CLS;
                  });
    }
    const bool in = p >= b0 && p < b0 + kRankTile && p < n;
    int nn = in ? (int)(p - b0) : -1;
    int d = p >= 0 ? 1 : 0;
    int e = in ? -1 : p;
    if (p >= 0 && !in && atomicCAS(&w.xslot[p], 0, -1) == 0) {
        const int x = atomicAdd(w.xcount, 1);
        if (x < kRankXMax) {
            w.xlist[x] = p;
            w.xslot[p] = x + 1;
        } else {
            w.err[1] = 1u;
        }
    }
    int buf = 0;
    sn[0][i] = nn; sd[0][i] = d; se[0][i] = e;
    __syncthreads();
    for (int it = 0; it < 11; it++) {        // 2^10 = kRankTile: every in-tile chain ends
        if (nn >= 0) {
            const int j = nn;
            d += sd[buf][j];
            e = se[buf][j];
            nn = sn[buf][j];
        }
        buf ^= 1;
        sn[buf][i] = nn; sd[buf][i] = d; se[buf][i] = e;
        if (!__syncthreads_or(nn >= 0)) break;
    }
    if (ok && nn >= 0) er |= ERR_CHAIN_CYCLE;
    if (ok) {
        w.dloc[u] = d;
        w.ext[u] = e;
    }
    for (int o = 32; o > 0; o >>= 1) er |= (uint32_t)__shfl_xor((int)er, o, 64);
    if ((i & 63) == 0 && er) atomicOr(w.err, er);
}

__device__ __forceinline__ void report(const LoadWork &w) {
    w.out->err[0] = load_coherent(&w.err[0]);
    w.out->err[1] = load_coherent(&w.err[1]);
    w.out->st = *w.st;
}

// one workgroup: the ranks of the tile exits, then where each thread starts
// in the order (base == null: shared threads have none; then this is the last
// pass and it reports)
__global__ __launch_bounds__(1024) void k_load_exits(int32_t T, int64_t *__restrict__ base, LoadWork w) {
    __shared__ int32_t sn[2][kRankXMax], sd[2][kRankXMax];
    const int nx = *w.xcount;
    if (w.err[0] == 0u && nx <= kRankXMax) {
        constexpr int PER = kRankXMax / 1024;
        int nn[PER], d[PER];
#pragma unroll
        for (int k = 0; k < PER; k++) {
            const int x = threadIdx.x + k * 1024;
            nn[k] = -1; d[k] = 0;
            if (x < nx) {
                const int32_t u = w.xlist[x];
                const int32_t e = w.ext[u];
                d[k] = w.dloc[u];
                nn[k] = e >= 0 ? w.xslot[e] - 1 : -1;
                sn[0][x] = nn[k]; sd[0][x] = d[k];
            }
        }
        __syncthreads();
        int buf = 0;
        bool open = false;
        for (int it = 0; it < 14; it++) {        // 2^13 = kRankXMax: every exit chain ends
            open = false;
#pragma unroll
            for (int k = 0; k < PER; k++) {
                if (nn[k] >= 0) {
                    const int j = nn[k];
                    d[k] += sd[buf][j];
                    nn[k] = sn[buf][j];
                    open |= nn[k] >= 0;
                }
            }
            buf ^= 1;
#pragma unroll
            for (int k = 0; k < PER; k++) {
                const int x = threadIdx.x + k * 1024;
                if (x < nx) { sn[buf][x] = nn[k]; sd[buf][x] = d[k]; }
            }
            if (!__syncthreads_or(open)) break;
        }
        if (__any(open) && (threadIdx.x & 63) == 0) atomicOr(w.err, ERR_CHAIN_CYCLE);
#pragma unroll
        for (int k = 0; k < PER; k++) {
            const int x = threadIdx.x + k * 1024;
            if (x < nx) w.xrank[x] = d[k];
        }
        __syncthreads();
        if (base) {
            int64_t carry = 0;
            for (int64_t t0 = 0; t0 < T; t0 += 1024) {
                const int64_t t = t0 + threadIdx.x;
                const int32_t u = t < T ? w.last[t] - 1 : -1;
                int64_t len = 0;
                if (u >= 0) len = (int64_t)w.dloc[u] + (w.ext[u] >= 0 ? w.xrank[w.xslot[w.ext[u]] - 1] : 0) + 1;
                int64_t tot;
                const int64_t ex = block_excl_scan<1024>(len, &tot);
                if (t < T) base[t] = carry + ex;
                carry += tot;
            }
            if (threadIdx.x == 0) base[T] = carry;
        }
    }
    __syncthreads();
    if (!base && threadIdx.x == 0) report(w);
}

// thread starts when the ranks are known (graphs with more tile exits)
__global__ __launch_bounds__(1024) void k_thread_base(int32_t T, const int32_t *__restrict__ last,
                                                      const int32_t *__restrict__ rank,
                                                      int64_t *__restrict__ base) {
    int64_t carry = 0;
    for (int64_t t0 = 0; t0 < T; t0 += 1024) {
        const int64_t t = t0 + threadIdx.x;
        const int32_t u = t < T ? last[t] - 1 : -1;
        const int64_t len = u >= 0 ? (int64_t)rank[u] + 1 : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan<1024>(len, &tot);
        if (t < T) base[t] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) base[T] = carry;
}

// ranks and order of the tasks; same-thread dependencies must point forward
// (dropped), cross-thread ones are counted, per chunk of tasks
template <bool RANKED>
__global__ __launch_bounds__(kBS) void k_cross_count(int32_t n, int64_t chunk,
                                                     const int32_t *__restrict__ tid,
                                                     const int64_t *__restrict__ base, int32_t *rank,
                                                     int32_t *__restrict__ order, LoadWork w) {
    // (read once: workgroups that run already add errors of their own to the
    // word, and the barrier below is for all waves of this one or none)
    __shared__ uint32_t s_failed;
    if (threadIdx.x == 0) s_failed = load_coherent(&w.err[0]) | (RANKED ? 0u : load_coherent(&w.err[1]));
    __syncthreads();
    if (s_failed) return;
    uint32_t e = 0;
    uint64_t mask = 0;
    int64_t c = 0;
    auto edge = [&](int64_t k) {
        const int32_t s = w.in_src[k];
        return EdgeIn{s, tid[s], w.ecls ? w.ecls[k] : 0u};
    };
    auto rank_of = [&](int32_t u) -> int32_t {
        if (RANKED) return rank[u];
        const int32_t x = w.ext[u];
        return w.dloc[u] + (x >= 0 ? w.xrank[w.xslot[x] - 1] : 0);
    };
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    for (int64_t u = lo + threadIdx.x; u < hi; u += kBS) {
        const int32_t tu = tid[u], ru = rank_of((int32_t)u);
        if (!RANKED) rank[u] = ru;
        order[base[tu] + ru] = (int32_t)u;
        each_edge(w.in_ptr[u], w.in_ptr[u + 1], edge, [&](int64_t, const EdgeIn &x) {
            if (x.tid == tu) {
                if (rank_of(x.src) >= ru) e |= ERR_BACK_EDGE;
            } else {
                c++;
                mask |= 1ull << x.cls;
            }
        });
    }
    c = wave_sum64(c);
    for (int o = 32; o > 0; o >>= 1) {
        e |= (uint32_t)__shfl_xor((int)e, o, 64);
        mask |= (uint64_t)shfl_xor64((int64_t)mask, o);
    }
    __shared__ int64_t part[kBS / 64];
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6] = c;
        atomic_or_hot(w.err, e);
        atomic_or_hot(&w.st->cross_mask, (unsigned long long)mask);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBS / 64; i++) c += part[i];
        w.csum[blockIdx.x] = c;
    }
}

// each chunk starts after the edges of the chunks before it, whose counts
// (at most kChunks) every workgroup sums itself
__global__ __launch_bounds__(kBS) void k_cross_fill(int32_t n, int64_t chunk,
                                                    const int32_t *__restrict__ tid,
                                                    int64_t *__restrict__ xptr, int32_t *__restrict__ xsrc,
                                                    uint8_t *__restrict__ xcls, LoadWork w) {
    if (blockIdx.x == 0 && threadIdx.x == 0) report(w);
    if (w.err[0] | w.err[1]) return;
    int64_t before = 0, tot;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kBS) before += w.csum[i];
    (void)block_excl_scan<kBS>(before, &tot);
    int64_t at = tot;
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    for (int64_t b = lo; b < hi; b += kBS) {
        const int64_t u = b + threadIdx.x;
        int64_t c = 0, k0 = 0, k1 = 0;
        int32_t tu = 0;
        if (u < hi) {
            tu = tid[u];
            k0 = w.in_ptr[u];
            k1 = w.in_ptr[u + 1];
            each_edge(k0, k1, [&](int64_t k) { return tid[w.in_src[k]]; },
                      [&](int64_t, int32_t t) { c += t != tu; });
        }
        int64_t o = at + block_excl_scan<kBS>(c, &tot);
        at += tot;
        if (u < hi) {
            xptr[u] = o;
            each_edge(k0, k1,
                      [&](int64_t k) {
                          const int32_t s = w.in_src[k];
                          return EdgeIn{s, tid[s], w.ecls ? w.ecls[k] : 0u};
                      },
                      [&](int64_t, const EdgeIn &x) {
                          if (x.tid == tu) return;
                          xsrc[o] = x.src;
                          xcls[o] = (uint8_t)x.cls;
                          o++;
                      });
        }
    }
    if (hi == n && threadIdx.x == 0) {
        xptr[n] = at;
        w.out->n_cross = at;
    }
}

void rank_chains(const dd_graph *g, int32_t *nxt, int32_t *nxt2, int32_t *rank2, uint32_t *err,
                 hipStream_t s) {
    const int32_t n = g->n;
    int gr = grid_for(n, kBS);
    k_rank_init<<<gr, kBS, 0, s>>>(n, g->thread_prev, nxt, g->rank);
    int steps = 1;
    while ((int64_t(1) << steps) <= (int64_t)n + 1) steps++;
    int32_t *a_n = nxt, *a_r = g->rank, *b_n = nxt2, *b_r = rank2;
    for (int i = 0; i < steps; i++) {
        k_rank_step<<<gr, kBS, 0, s>>>(n, a_n, a_r, b_n, b_r);
        int32_t *t;
        t = a_n; a_n = b_n; b_n = t;
        t = a_r; a_r = b_r; b_r = t;
    }
    if (a_r != g->rank) (void)hipMemcpyAsync(g->rank, a_r, sizeof(int32_t) * (size_t)n,
                                       hipMemcpyDeviceToDevice, s);
    k_rank_check<<<gr, kBS, 0, s>>>(n, a_n, err);
}
}  // namespace

hipError_t load_device(dd_graph *g, const LoadIn &in, LoadOut *out, LoadOut *out_dev, hipStream_t s,
                       const std::function<hipError_t(int64_t)> &edges) {
    const int32_t n = g->n, T = g->n_threads;
    // one block of working memory, the part that starts at zero first
    size_t off = 0;
    auto put = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t N4 = sizeof(int32_t) * (size_t)n, T4 = sizeof(int32_t) * (size_t)T;
    const size_t o_succ = put(N4), o_heads = put(T4), o_last = put(T4), o_xslot = put(N4),
                 o_err = put(8), o_xcount = put(4), o_st = put(sizeof(LoadStats));
    const size_t zero = off;
    const size_t o_dloc = put(N4), o_ext = put(N4), o_xlist = put(4 * kRankXMax),
                 o_xrank = put(4 * kRankXMax), o_csum = put(8 * kChunks);
    char *m = nullptr;
    hipError_t e = dalloc(reinterpret_cast<void **>(&m), off, s);
    if (e != hipSuccess) return e;
    LoadWork w{in.own_ptr, nullptr, nullptr, (int32_t *)(m + o_succ), (int32_t *)(m + o_heads),
               (int32_t *)(m + o_last), (int32_t *)(m + o_xslot), (uint32_t *)(m + o_err),
               (int32_t *)(m + o_xcount), (LoadStats *)(m + o_st), (int32_t *)(m + o_dloc),
               (int32_t *)(m + o_ext), (int32_t *)(m + o_xlist), (int32_t *)(m + o_xrank),
               (int64_t *)(m + o_csum), out_dev};
    *out = LoadOut{};
    int32_t *nxt = nullptr, *nxt2 = nullptr, *rank2 = nullptr;
    const int64_t chunk = chunk_len(n, kBS);
    const unsigned nc = (unsigned)((n + chunk - 1) / chunk);
    const unsigned nv = (unsigned)(grid_for(n, kBS) < kValBlocks ? grid_for(n, kBS) : kValBlocks);
#define LD(x) do { if (e == hipSuccess) e = (x); } while (0)
    LD(hipMemsetAsync(m, 0, zero, s));
    if (e == hipSuccess)
        k_load_nodes<<<nv, kBS, 0, s>>>(n, T, in.prev, in.tid, in.dur, in.gap, in.cls, in.in_ptr,
                                        g->thread_prev, g->thread_id, g->dur, g->gap, g->cls, w, !g->shared);
    LD(hipGetLastError());
    // the edge count sizes the edge arrays: in_ptr's ends come back first
    LD(hipStreamSynchronize(s));
    const int64_t E = out->ends[0] != 0 ? -1 : out->ends[1];
    if (e == hipSuccess && edges(E) == hipSuccess) {
        w.in_src = in.own_src;
        w.ecls = in.own_ecls;
        k_load_tiles<<<grid_for(n, kRankTile), kRankTile, 0, s>>>(
            n, T, E, g->thread_prev, g->thread_id, in.in_src, in.ecls, w);
        k_load_exits<<<1, 1024, 0, s>>>(T, g->shared ? nullptr : g->thread_base, w);
        if (!g->shared) {
            k_cross_count<false><<<nc, kBS, 0, s>>>(n, chunk, g->thread_id, g->thread_base, g->rank, g->order, w);
            k_cross_fill<<<nc, kBS, 0, s>>>(n, chunk, g->thread_id, g->xin_ptr, g->xin_src, g->xin_cls, w);
        }
        LD(hipGetLastError());
        LD(hipStreamSynchronize(s));
        if (e == hipSuccess && out->err[1] && !out->err[0]) {
            // more tile exits than one workgroup ranks: plain pointer jumping
            LD(dalloc_n(&nxt, (size_t)n, s));
            LD(dalloc_n(&nxt2, (size_t)n, s));
            LD(dalloc_n(&rank2, (size_t)n, s));
            LD(hipMemsetAsync(w.err, 0, 8, s));
            if (e == hipSuccess) {
                rank_chains(g, nxt, nxt2, rank2, w.err, s);
                if (g->shared) {
                    ReadBack rb(s, sizeof(uint32_t));
                    LD(rb.add(&out->err[0], w.err, sizeof(uint32_t)));
                    LD(rb.finish());
                } else {
                    k_thread_base<<<1, 1024, 0, s>>>(T, w.last, g->rank, g->thread_base);
                    k_cross_count<true><<<nc, kBS, 0, s>>>(n, chunk, g->thread_id, g->thread_base, g->rank, g->order, w);
                    k_cross_fill<<<nc, kBS, 0, s>>>(n, chunk, g->thread_id, g->xin_ptr, g->xin_src, g->xin_cls, w);
                    LD(hipGetLastError());
                    LD(hipStreamSynchronize(s));
                }
            }
        }
    }
#undef LD
    if (e != hipSuccess) (void)hipStreamSynchronize(s);
    dfree(m, s);
    dfree(nxt, s);
    dfree(nxt2, s);
    dfree(rank2, s);
    return e;
}

}  // namespace dd
