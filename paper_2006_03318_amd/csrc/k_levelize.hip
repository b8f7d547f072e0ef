// Levelization on the GPU: Kahn's algorithm over the task graph (the
// reference counts and ready frontier of Sec. 4.1, Algorithm 1), taken one
// whole frontier per round.
//
// Phases.  Because tasks on one thread run in their recorded order
// (Sec. 4.2.2), the graph is a set of thread chains plus cross-thread
// dependencies.  A round advances the front of every thread past all tasks
// whose cross-thread parents lie behind the fronts of their own threads at
// the start of the round; the tasks passed in round r form phase r, one
// contiguous run ("segment") per thread.  This is Kahn's algorithm where
// "parent done" is read off the parent thread's front instead of a
// decremented counter.  Phase = longest path counting 1 per cross-thread
// edge and 0 per thread-order edge.  A round that advances no thread while
// tasks remain means a cycle.
//
// Levels.  Kahn level = longest path counting 1 per edge.  Inside a
// segment, level_i = max(level_{i-1} + 1, X_i) with X_i = 1 + the largest
// level of a cross-thread parent; with the phases known, every segment is a
// segmented prefix maximum of X_j - j.
//
// The schedule handed to the simulation lists tasks by step (phase or
// level); within a phase step, thread runs are contiguous and in thread
// order.  Each position carries its "gathers": the cross-thread parents,
// plus the previous task on the thread for the first task of a run.

#include "dd_common.h"
#include "dd_internal.h"
#include "dd_batches.h"

#include <stddef.h>
#include <stdio.h>
#include <string.h>

namespace dd {
namespace {

constexpr int kBS = 256;
constexpr int kWG = 1024;   // the single workgroup running the rounds

struct Req {
    const int64_t *base;      // [T+1] thread start in order space
    const int32_t *order;
    const int32_t *rank;
    const int32_t *tid;
    const int64_t *xin_ptr;
    const int32_t *xin_src;
    const uint8_t *xin_cls;
};

__device__ __forceinline__ bool on(uint64_t mask, uint8_t c) { return (mask >> c) & 1ull; }

// small results of the passes (device memory, cleared by the first of them)
struct LevWork {
    int64_t result[2];             // steps, segments
    int64_t reqs;                  // active cross-thread dependencies
    unsigned long long gctr;       // gather entries handed out
    uint32_t err, pad;
};

// per chunk of order positions: candidates (positions with an active
// cross-thread parent) << 32 | active cross-thread parents
__global__ __launch_bounds__(kBS) void k_req_count(int32_t n, int64_t chunk, Req r, uint64_t mask,
                                                   int64_t *__restrict__ csum, LevWork *__restrict__ lw) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *lw = LevWork{};
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    int64_t sum = 0;
    for (int64_t p = lo + threadIdx.x; p < hi; p += kBS) {
        const int32_t u = r.order[p];
        int64_t c = 0;
        for (int64_t k = r.xin_ptr[u]; k < r.xin_ptr[u + 1]; k++) c += on(mask, r.xin_cls[k]);
        sum += c ? ((int64_t)1 << 32) | c : 0;
    }
    sum = wave_sum64(sum);
    __shared__ int64_t part[kBS / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBS / 64; i++) sum += part[i];
        csum[blockIdx.x] = sum;
    }
}

constexpr int kWinT = 16;               // graph threads of the windowed rounds at most

// A candidate packed for the windowed rounds: its order position and, for
// the first two parent threads (by id) among its requirements, the largest
// requirement position on each (order space); meta = first thread | second
// thread << 8 | number of distinct parent threads << 16.  It is blocked when
// one of those maxima lies at or past its thread's front; only a candidate
// with parents on three or more threads needs its full requirement list.
struct alignas(16) CandEnt {
    int32_t pos, g0, g1;
    uint32_t meta;
};

// candidates (positions with a cross-thread parent) and their requirements;
// with pent, the packed entries too (T <= kWinT: the first two parent
// threads by id; T <= kEntT: the first two met in the list, which serves
// the same test)
constexpr int kEntT = 255;              // graph threads a packed entry can name (8 bits)
// (each chunk starts after the chunks before it, whose counts every workgroup
// sums itself; also closes the lists: cidx[n] = C, req_ptr[C] = R)
__global__ __launch_bounds__(kBS) void k_req_fill(int32_t n, int32_t T, int64_t chunk, Req r, uint64_t mask,
                                                  const int64_t *__restrict__ csum,
                                                  int32_t *__restrict__ cidx,
                                                  int64_t *__restrict__ cand_pos,
                                                  int64_t *__restrict__ req_ptr,
                                                  int32_t *__restrict__ req_chain,
                                                  int64_t *__restrict__ req_gpos,
                                                  CandEnt *__restrict__ pent, LevWork *__restrict__ lw) {
    int64_t before = 0, tot;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kBS) before += csum[i];
    (void)block_excl_scan<kBS>(before, &tot);
    int64_t at = tot;
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    for (int64_t b = lo; b < hi; b += kBS) {
        const int64_t p = b + threadIdx.x;
        int32_t u = 0;
        int64_t c = 0, k0 = 0, k1 = 0;
        if (p < hi) {
            u = r.order[p];
            k0 = r.xin_ptr[u];
            k1 = r.xin_ptr[u + 1];
            for (int64_t k = k0; k < k1; k++) c += on(mask, r.xin_cls[k]);
        }
        const int64_t mine = at + block_excl_scan<kBS>(c ? ((int64_t)1 << 32) | c : 0, &tot);
        at += tot;
        if (p >= hi) continue;
        const int64_t i = mine >> 32;
        cidx[p] = (int32_t)i;
        if (!c) continue;
        cand_pos[i] = p;
        int64_t o = mine & 0xffffffffll;
        req_ptr[i] = o;
        int32_t mx[kWinT];                  // largest requirement per parent thread (-1: none)
#pragma unroll
        for (int z = 0; z < kWinT; z++) mx[z] = -1;
        int32_t t0 = -1, t1 = -1, m0 = -1, m1 = -1;   // T > kWinT: the first two threads met
        bool many = false;                            // a third parent thread
        for (int64_t k = k0; k < k1; k++) {
            if (!on(mask, r.xin_cls[k])) continue;
            const int32_t s = r.xin_src[k];
            const int32_t ts = r.tid[s];
            const int64_t gp = r.base[ts] + r.rank[s];
            req_chain[o] = ts;
            req_gpos[o] = gp;
#pragma unroll
            for (int z = 0; z < kWinT; z++)
                if (z == ts && (int32_t)gp > mx[z]) mx[z] = (int32_t)gp;
            if (ts == t0) m0 = (int32_t)gp > m0 ? (int32_t)gp : m0;
            else if (ts == t1) m1 = (int32_t)gp > m1 ? (int32_t)gp : m1;
            else if (t0 < 0) { t0 = ts; m0 = (int32_t)gp; }
            else if (t1 < 0) { t1 = ts; m1 = (int32_t)gp; }
            else many = true;
            o++;
        }
        if (!pent) continue;                // (more than kEntT threads: no packed entries)
        if (T > kWinT) {
            const uint32_t nd = (t0 >= 0 ? 1u : 0u) + (t1 >= 0 ? 1u : 0u) + (many ? 1u : 0u);
            pent[i] = CandEnt{(int32_t)p, m0 < 0 ? 0 : m0, m1 < 0 ? 0 : m1,
                              (uint32_t)(t0 < 0 ? 0 : t0) | ((uint32_t)(t1 < 0 ? 0 : t1) << 8) | (nd << 16)};
            continue;
        }
        CandEnt ce{(int32_t)p, 0, 0, 0u};
        uint32_t nd = 0;
#pragma unroll
        for (int z = 0; z < kWinT; z++) {
            if (mx[z] < 0) continue;
            if (nd == 0) { ce.g0 = mx[z]; ce.meta |= (uint32_t)z; }
            if (nd == 1) { ce.g1 = mx[z]; ce.meta |= (uint32_t)z << 8; }
            nd++;
        }
        ce.meta |= nd << 16;
        pent[i] = ce;
    }
    if (hi == n && threadIdx.x == 0) {
        cidx[n] = (int32_t)(at >> 32);
        req_ptr[at >> 32] = at & 0xffffffffll;
        lw->reqs = at & 0xffffffffll;
    }
}

// What both kinds of rounds leave, and what follows from the steps: the
// widest, the batches of k_solo.hip, and the results the host reads.
struct StepArgs {
    int32_t T, with_prev;
    int64_t n;
    const int64_t *base;           // [T+1]
    int32_t *step_ptr;             // [n+1]
    int32_t *segoff;               // windowed rounds: [n x T] position of each thread's run in each step
    int4 *bat;
    int32_t *nbat;
    LevWork *lw;
    LevelizeOut *out;              // host memory
};

// (the whole workgroup; step_ptr[0..R] is written)
__device__ void finish_steps(int64_t R, int64_t nseg, const StepArgs &a) {
    __shared__ int s_wmax, s_threads;
    if (threadIdx.x == 0) { s_wmax = 0; s_threads = 0; }
    __syncthreads();
    int wmax = 0, live = 0;
    for (int64_t t = threadIdx.x; t < a.T; t += kWG) live += a.base[t + 1] > a.base[t];
    for (int64_t r = threadIdx.x; r < R; r += kWG) {
        const int w = a.step_ptr[r + 1] - a.step_ptr[r];
        wmax = w > wmax ? w : wmax;
    }
    if (R <= kSplitMaxSteps)
        for (int64_t r = threadIdx.x; r <= R; r += kWG) a.out->steps[r] = a.step_ptr[r];
    if (wmax) atomicMax(&s_wmax, wmax);
    if (live) atomicAdd(&s_threads, live);
    solo_batches(R, a.step_ptr, a.bat, a.nbat);
    __syncthreads();
    if (threadIdx.x == 0) {
        a.lw->result[0] = R;
        a.lw->result[1] = nseg;
        a.out->n_steps = R;
        a.out->n_segments = nseg;
        a.out->max_width = s_wmax;
        a.out->n_gathers = a.lw->reqs + (a.with_prev ? nseg - s_threads : 0);
        a.out->err = 0;
    }
}

struct KahnArgs {
    const CandEnt *pent;      // [C] packed entries (T <= kEntT), else null
    int32_t T;
    int64_t n;
    const int64_t *base;      // [T+1]
    const int32_t *cidx;      // [n+1] candidates before each order position
    const int64_t *cand_pos;  // [C]
    const int64_t *req_ptr;   // [C+1]
    const int32_t *req_chain;
    const int64_t *req_gpos;
    int64_t *front, *ccur, *nfront, *nccur;   // [T] (more than kLdsT threads)
    int64_t *cend;            // [T+1] the same: first candidate of each thread
    int32_t *long_list;       // [T]
    int64_t *seg_start;       // [n] order position of each segment's first task
    int64_t *seg_off;         // [n+1] schedule position of it
    int32_t *seg_step;        // [n]
    int32_t *step_ptr;        // [n+1]
    LevWork *lw;              // steps, segments, error
};

// Round state of the generic rounds: with at most kLdsT graph threads the
// fronts, candidate cursors and thread bounds live in LDS (a requirement
// check then reads its parent thread's front from LDS, not from global
// memory); beyond that they stay in the global arrays.
constexpr int kLdsT = 2048;
constexpr int kProbe = 128;     // candidates a round probes per thread before the long-run scan
constexpr int kSegBuf = 2048;   // segments and rounds kept in LDS before they go out
constexpr int kAhead = 3;       // probes whose entries are loaded a round ahead
constexpr int kLong = 4;        // candidates per lane and step of that scan

// sums over the lanes up to and including this one (every lane active)
__device__ __forceinline__ int wave_scan_add(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// One round is a chain of latencies in one workgroup, 2.1 us with 51 threads
// (100 rounds of the 32,815-task data-parallel trace, two of them runs of
// 15,000 candidates together): the probes 1.4, barriers 0.3, numbering the
// segments 0.4.  2.5 us a round when each began with a load of its
// candidates, looked through long requirement lists from their start, and
// stored its segments before its last barrier.
template <bool L>
__global__ __launch_bounds__(kWG) void k_kahn_rounds(KahnArgs a) {
    __shared__ int s_nlong[2];      // long runs of the round, by its parity
    __shared__ int64_t s_unfinished;   // round + 1 when a thread is not at its end
    __shared__ unsigned long long s_first;
    __shared__ int64_t s_carry_cnt;
    __shared__ int64_t s_st[L ? 6 * (kLdsT + 1) : 1];
    const int lane = threadIdx.x & 63;
    __shared__ int64_t s_carry_len;
    __shared__ int32_t s_seg[3][L ? kSegBuf : 1], s_step[L ? kSegBuf : 1];   // (T <= 64 only)
    int64_t *const front = L ? s_st : a.front;
    int64_t *const cidx = L ? s_st + (kLdsT + 1) : a.ccur;
    int64_t *const nfront = L ? s_st + 2 * (kLdsT + 1) : a.nfront;
    int64_t *const ncidx = L ? s_st + 3 * (kLdsT + 1) : a.nccur;
    const int64_t *const base = L ? s_st + 4 * (kLdsT + 1) : a.base;
    // candidates of thread t: cbase(t) .. cbase(t + 1)
    auto cbase = [&](int t) -> int64_t { return L ? s_st[5 * (kLdsT + 1) + t] : a.cend[t]; };
    for (int t = threadIdx.x; t <= a.T; t += kWG) {
        const int64_t b = a.base[t], c = a.cidx[b];
        if (t < a.T) {
            front[t] = b;
            cidx[t] = c;
        }
        if (L) {
            s_st[4 * (kLdsT + 1) + t] = b;
            s_st[5 * (kLdsT + 1) + t] = c;
        } else {
            a.cend[t] = c;
        }
    }
    __syncthreads();
    // lanes per graph thread in step A: all threads in one pass when they fit
    int gsh = 6;
    while (gsh > 0 && ((int64_t)a.T << gsh) > kWG) gsh--;
    const int G = 1 << gsh;
    const unsigned long long gmask = G == 64 ? ~0ull : ((1ull << G) - 1ull);
    // a candidate is blocked while a requirement lies at or past the front of
    // its thread; fronts never fall, so a lane that meets the same candidate
    // again goes on at the requirement that blocked it (a task with 53 parents
    // is met every round), four loads in flight together
    int64_t lj = -1, lk = 0, lend = 0;
    auto blocked_list = [&](int64_t j) {
        if (lj != j) {
            lj = j;
            lk = a.req_ptr[j];
            lend = a.req_ptr[j + 1];
        }
        while (lk < lend) {
            int64_t gp[4];
            int32_t ch[4];
#pragma unroll
            for (int z = 0; z < 4; z++) {
                const int64_t k = lk + z < lend ? lk + z : lend - 1;
                gp[z] = a.req_gpos[k];
                ch[z] = a.req_chain[k];
            }
            bool b = false;
#pragma unroll
            for (int z = 0; z < 4; z++) {
                b = b || gp[z] >= front[ch[z]];
                lk += b ? 0 : 1;
            }
            if (b) return true;
        }
        return false;
    };
    // without packed entries every candidate's list is read, and most hold one
    // requirement: one at a time, from its start (60,000 tasks on 300 threads
    // 885 us a levelization, on 3,000 threads 1,950; 1,058 and 2,605 with
    // blocked_list)
    auto blocked_walk = [&](int64_t j) {
        for (int64_t k = a.req_ptr[j]; k < a.req_ptr[j + 1]; k++)
            if (a.req_gpos[k] >= front[a.req_chain[k]]) return true;
        return false;
    };
    // with packed entries: one 16-byte load; only a candidate with parents
    // on three or more threads reads its requirement list
    auto blocked_ent = [&](const CandEnt &e, int64_t j) {
        const uint32_t nd = e.meta >> 16;
        if (e.g0 >= front[e.meta & 0xff]) return true;
        if (nd > 1 && e.g1 >= front[(e.meta >> 8) & 0xff]) return true;
        if (nd > 2) return blocked_list(j);
        return false;
    };
    // with one group per thread throughout, the entries of its first probes
    // stay in registers from round to round
    const bool ahead = a.pent && ((int64_t)a.T << gsh) <= kWG && (kProbe >> gsh) >= kAhead;
    CandEnt e0{}, e1{}, e2{};
    int64_t eat = -1;                             // first candidate they hold
    int64_t nseg = 0, npos = 0;                   // segments and positions so far
    int64_t round = 0;
    // At most 64 threads: segments and steps wait in LDS (a store each round
    // makes the round wait for it at its next barrier), from seg0 and round0 on
    int64_t seg0 = 0, round0 = 0;
    auto flush = [&]() {
        for (int64_t i = threadIdx.x; i < nseg - seg0; i += kWG) {
            a.seg_start[seg0 + i] = s_seg[0][i];
            a.seg_off[seg0 + i] = s_seg[1][i];
            a.seg_step[seg0 + i] = s_seg[2][i];
        }
        for (int64_t i = threadIdx.x; i < round - round0; i += kWG) a.step_ptr[round0 + i] = s_step[i];
        seg0 = nseg;
        round0 = round;
        __syncthreads();
    };
    bool stalled = false;
    if (threadIdx.x == 0) {
        s_nlong[0] = s_nlong[1] = 0;
        s_unfinished = 0;
    }
    __syncthreads();
    for (;;) {
        // A: a group of G lanes per graph thread (G = 64 when few threads,
        // fewer when there are more, so that every thread is probed in one
        // pass) scans up to kProbe candidates of its thread, G at a time
        for (int t0 = 0; t0 < a.T; t0 += kWG >> gsh) {
            const int t = t0 + (int)(threadIdx.x >> gsh);        // uniform within a group
            const int gl = (int)threadIdx.x & (G - 1);
            const bool act = t < a.T;
            const int64_t f = act ? front[t] : 0, end = act ? base[t + 1] : 0;
            int64_t ci = act ? cidx[t] : 0;
            const int64_t ce = act ? cbase(t + 1) : 0;
            const int64_t c0 = ci;
            const bool fin = !act || f >= end;
            if (act && fin && gl == 0) { nfront[t] = f; ncidx[t] = ci; }
            if (!fin && gl == 0) s_unfinished = round + 1;   // (every writer the same)
            bool done = fin;
            int64_t cnew = ce;
            int32_t npos = 0;                 // order position of candidate cnew (packed entries)
            const bool kept = ahead && eat == c0;
            CandEnt x0 = e0, x1 = e1, x2 = e2;
            for (int w = 0; w < (kProbe >> gsh); w++) {
                if (__all(done)) break;                           // wave-uniform
                const int64_t j = ci + gl;
                bool b = false;
                int32_t pj = 0;
                if (!done && j < ce) {
                    if (a.pent) {
                        CandEnt e = x0;
                        if (!kept || w >= kAhead) e = a.pent[j];
                        pj = e.pos;
                        b = blocked_ent(e, j);
                    } else {
                        b = blocked_walk(j);
                    }
                }
                x0 = x1;
                x1 = x2;
                const unsigned long long bal = __ballot(b);
                const unsigned long long gb = (bal >> (lane & ~(G - 1))) & gmask;
                const int fl = gb ? __ffsll((long long)gb) - 1 : 0;
                const int32_t pf = __shfl(pj, (lane & ~(G - 1)) + fl, 64);   // the finder's position
                if (!done) {
                    if (gb) {
                        cnew = ci + fl;
                        npos = pf;
                        done = true;
                    } else if (ci + G >= ce) {
                        cnew = ce;
                        done = true;
                    } else {
                        ci += G;
                    }
                }
            }
            // the entries of the next round's first probes, while the others
            // finish and the segments are numbered
            const int64_t cn = done ? cnew : ci;
            if (ahead && !fin && cn != eat && cn < ce) {
                eat = cn;
                e0 = a.pent[cn + gl < ce ? cn + gl : cn];
                e1 = a.pent[cn + G + gl < ce ? cn + G + gl : cn];
                e2 = a.pent[cn + 2 * G + gl < ce ? cn + 2 * G + gl : cn];
            }
            if (!fin && gl == 0) {
                if (done) {
                    ncidx[t] = cnew;
                    nfront[t] = cnew < ce ? (a.pent ? (int64_t)npos : a.cand_pos[cnew]) : end;
                } else {
                    ncidx[t] = ci;
                    a.long_list[atomicAdd(&s_nlong[round & 1], 1)] = t;
                }
            }
        }
        __syncthreads();
        // B: threads with long ready runs, scanned by the whole workgroup
        const int nlong = s_nlong[round & 1];
        const int pass = a.pent ? kLong * kWG : kWG;          // candidates looked at together
        for (int i = 0; i < nlong; i++) {
            const int t = a.long_list[i];
            int64_t ci = ncidx[t];
            const int64_t ce = cbase(t + 1);
            int64_t cnew = ce;
            for (;;) {
                if (threadIdx.x == 0) s_first = ~0ull;
                __syncthreads();
                // (kLong per lane, whose loads are in flight together)
                if (a.pent) {
                    CandEnt e[kLong];
#pragma unroll
                    for (int z = 0; z < kLong; z++) {
                        const int64_t j = ci + z * kWG + threadIdx.x;
                        e[z] = a.pent[j < ce ? j : ci];
                    }
#pragma unroll
                    for (int z = 0; z < kLong; z++) {
                        const int64_t j = ci + z * kWG + threadIdx.x;
                        if (j < ce && blocked_ent(e[z], j)) atomicMin(&s_first, (unsigned long long)j);
                    }
                } else {
                    const int64_t j = ci + threadIdx.x;
                    if (j < ce && blocked_walk(j)) atomicMin(&s_first, (unsigned long long)j);
                }
                __syncthreads();
                const unsigned long long fb = s_first;
                __syncthreads();
                if (fb != ~0ull) { cnew = (int64_t)fb; break; }
                if (ci + pass >= ce) { cnew = ce; break; }
                ci += pass;
            }
            if (threadIdx.x == 0) {
                ncidx[t] = cnew;
                nfront[t] = cnew < ce ? a.cand_pos[cnew] : base[t + 1];
            }
        }
        if (nlong) __syncthreads();
        if (s_unfinished != round + 1) break;                 // every thread at its end
        // C: emit one segment per advanced thread.  Up to 64 threads: one
        // wave ranks them with a ballot; else a workgroup scan of packed
        // count<<32 | length per block of kWG threads.
        if (a.T <= 64) {
            if (threadIdx.x < 64) {
                const int t = (int)threadIdx.x;
                const int len = t < a.T ? (int)(nfront[t] - front[t]) : 0;
                const unsigned long long bal = __ballot(len > 0);
                const int sum = wave_scan_add(len);       // lengths up to and including t
                if (len > 0) {
                    const int i = (int)(nseg - seg0) + __popcll(bal & ((1ull << t) - 1ull));
                    s_seg[0][i] = (int32_t)front[t];
                    s_seg[1][i] = (int32_t)npos + sum - len;
                    s_seg[2][i] = (int32_t)round;
                }
                if (t == 0) {
                    s_step[round - round0] = (int32_t)npos;
                    s_carry_cnt = __popcll(bal);
                    s_nlong[(round + 1) & 1] = 0;
                }
                if (t == 63) s_carry_len = sum;
                if (t < a.T) {                            // the fronts advance
                    front[t] = nfront[t];
                    cidx[t] = ncidx[t];
                }
            }
            __syncthreads();
        } else {
            if (threadIdx.x == 0) { s_carry_cnt = 0; s_carry_len = 0; }
            __syncthreads();
            for (int b0 = 0; b0 < a.T; b0 += kWG) {
                const int t = b0 + threadIdx.x;
                int64_t len = 0;
                if (t < a.T) len = nfront[t] - front[t];
                const int64_t packed = len > 0 ? ((int64_t(1) << 32) | len) : 0;
                int64_t tot;
                const int64_t ex = block_excl_scan<kWG>(packed, &tot);
                if (len > 0) {
                    const int64_t sg = nseg + s_carry_cnt + (ex >> 32);
                    a.seg_start[sg] = front[t];
                    a.seg_off[sg] = npos + s_carry_len + (ex & 0xffffffffll);
                    a.seg_step[sg] = (int32_t)round;
                }
                __syncthreads();
                if (threadIdx.x == 0) {
                    s_carry_cnt += tot >> 32;
                    s_carry_len += tot & 0xffffffffll;
                }
                __syncthreads();
            }
        }
        const int64_t adv = s_carry_cnt, advlen = s_carry_len;
        if (adv == 0) {                               // stalled: cycle
            stalled = true;
            break;
        }
        if (a.T > 64 && threadIdx.x == 0) a.step_ptr[round] = (int32_t)npos;
        nseg += adv;
        npos += advlen;
        round++;
        if (a.T <= 64) {
            if (nseg - seg0 > kSegBuf - 64 || round - round0 == kSegBuf) flush();
        } else {
            // D: advance the fronts
            for (int t = threadIdx.x; t < a.T; t += kWG) {
                front[t] = nfront[t];
                cidx[t] = ncidx[t];
            }
            if (threadIdx.x == 0) s_nlong[round & 1] = 0;
            __syncthreads();
        }
    }
    if (a.T <= 64) flush();
    if (threadIdx.x == 0) {
        a.step_ptr[round] = (int32_t)npos;
        a.seg_off[nseg] = npos;
        a.lw->result[0] = round;
        a.lw->result[1] = nseg;
        if (stalled) a.lw->err = ERR_KAHN_CYCLE;
    }
}

// Windowed rounds for graphs with at most kWinT threads: the same rounds as
// above, with each thread's next candidates staged in LDS (a wave per thread,
// waves taking threads w, w + waves, ...) so that a round reads no global
// memory except to refill a window that is less than half full, to cross a
// ready run longer than the window, or for a requirement past the first two
// of a candidate.
//
// A long ready run is crossed with tile maxima: for tiles of 64 and of 4096
// consecutive candidates (global candidate order), the largest requirement
// position on each parent thread.  A tile whose maxima all lie behind the
// round's fronts holds no blocked candidate.  Candidates before the search
// start are ready already, so only a tile that also holds another thread's
// candidates can look blocked without being so; the search then simply goes
// on after it.
constexpr int kWinBytes = 6144 * 16;    // LDS window of candidate entries, shared by all threads
constexpr int kRefill = 16;             // window entries loaded per lane at once

// tile maxima over candidates: tm1[k * T + s] = largest requirement position
// on thread s among candidates [64k, 64k + 64) (-1 if none), tm2 the same for
// [4096m, 4096m + 4096); a wave per tile of 64, a workgroup per tile of 4,096
__global__ __launch_bounds__(kWG) void k_tile_max(const int32_t *__restrict__ pC, int32_t T,
                                                  const CandEnt *__restrict__ pent,
                                                  const int64_t *__restrict__ req_ptr,
                                                  const int32_t *__restrict__ req_chain,
                                                  const int64_t *__restrict__ req_gpos,
                                                  int32_t *__restrict__ tm1, int32_t *__restrict__ tm2) {
    const int64_t C = *pC;                // candidates (the grid covers every position)
    const int64_t b0 = (int64_t)blockIdx.x << 12;
    if (b0 >= C) return;
    __shared__ int32_t s_mx[kWG / 64][kWinT];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int32_t best[kWinT];
#pragma unroll
    for (int z = 0; z < kWinT; z++) best[z] = -1;
    for (int i = wv; i < 64; i += kWG / 64) {
        const int64_t j = b0 + i * 64 + lane, k = j >> 6;
        if ((k << 6) >= C) break;         // whole waves past the last tile
        const bool ok = j < C;
        const CandEnt e = pent[ok ? j : 0];
        const uint32_t nd = ok ? e.meta >> 16 : 0u;
        const bool list = nd > 2;         // parents on three or more threads
        const int64_t q0 = list ? req_ptr[j] : 0, q1 = list ? req_ptr[j + 1] : 0;
#pragma unroll
        for (int ts = 0; ts < kWinT; ts++) {
            if (ts < T) {
                int32_t r = -1;
                if (nd > 0 && (int)(e.meta & 0xff) == ts) r = e.g0;
                if (nd > 1 && (int)((e.meta >> 8) & 0xff) == ts) r = e.g1;
                for (int64_t q = q0; q < q1; q++)
                    if (req_chain[q] == ts && (int32_t)req_gpos[q] > r) r = (int32_t)req_gpos[q];
                for (int o = 32; o > 0; o >>= 1) {
                    const int32_t y = __shfl_xor(r, o, 64);
                    r = y > r ? y : r;
                }
                if (lane == 0) tm1[k * T + ts] = r;
                best[ts] = r > best[ts] ? r : best[ts];
            }
        }
    }
    if (lane == 0)
#pragma unroll
        for (int z = 0; z < kWinT; z++) s_mx[wv][z] = best[z];
    __syncthreads();
    if ((int)threadIdx.x < T) {
        int32_t r = -1;
        for (int w = 0; w < kWG / 64; w++) r = s_mx[w][threadIdx.x] > r ? s_mx[w][threadIdx.x] : r;
        tm2[(b0 >> 12) * T + threadIdx.x] = r;
    }
}

struct WinArgs {
    int32_t T, wlog;                    // window of 2^wlog entries per thread
    const int64_t *base;                // [T+1]
    const int32_t *cidx;                // [n+1] candidates before each order position
    const CandEnt *pent;                // [C]
    const int64_t *req_ptr;             // [C+1]
    const int32_t *req_chain;
    const int64_t *req_gpos;
    const int32_t *tm1, *tm2;           // tile maxima (tiles of 64 and 4096 candidates)
    int32_t *ftab;                      // [(n+1) x T] fronts at the start of each round
    LevWork *lw;                        // steps, error
};

__device__ __forceinline__ bool win_blocked(const WinArgs &a, const CandEnt &e, int64_t j,
                                            const int32_t *front) {
    const uint32_t nd = e.meta >> 16;
    if (e.g0 >= front[e.meta & 0xff]) return true;
    if (nd > 1 && e.g1 >= front[(e.meta >> 8) & 0xff]) return true;
    if (nd > 2) {                        // parents on three or more threads
        for (int64_t k = a.req_ptr[j]; k < a.req_ptr[j + 1]; k++)
            if (a.req_gpos[k] >= front[a.req_chain[k]]) return true;
    }
    return false;
}

// One barrier per round: round r reads the fronts of buffer r & 1 and writes
// the advanced fronts, plus one flag per thread (advanced, unfinished), into
// buffer (r + 1) & 1 and r & 1; a buffer is rewritten only two rounds later,
// after the next barrier.  The fronts of every round go to a table from which
// the segments are cut afterwards (k_steps, k_place_win).
__global__ __launch_bounds__(kWG) void k_kahn_win(WinArgs a) {
    static_assert(kWG / 64 >= kWinT, "a wave per graph thread");
    constexpr int kWinE = kWinBytes / (int)sizeof(CandEnt);
    __shared__ CandEnt s_win[kWinE + 64];
    __shared__ __align__(16) int32_t s_front[2][kWinT];
    __shared__ __align__(16) uint8_t s_adv[2][16], s_unf[2][16];   // flags of graph threads
    const int lane = threadIdx.x & 63;
    // wave t walks graph thread t (uniform: the wave's state stays scalar)
    const int t = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int W = 1 << a.wlog;
    const int T = a.T;
    const bool mine = t < T;
    CandEnt *const win = s_win + (mine ? t : 0) * W;
    // the wave's own thread: front end, candidate range and window in registers
    const int end = mine ? (int)a.base[t + 1] : 0;
    const int ce = mine ? a.cidx[a.base[t + 1]] : 0;
    int ci = mine ? a.cidx[a.base[t]] : 0;
    int wend = ci;
    int f = mine ? (int)a.base[t] : 0;             // the wave's own front (also in LDS for the others)
    if (threadIdx.x < 32) reinterpret_cast<uint8_t *>(s_adv)[threadIdx.x] = 0;
    if (threadIdx.x < 32) reinterpret_cast<uint8_t *>(s_unf)[threadIdx.x] = 0;
    if (threadIdx.x < 2 * kWinT) s_front[0][threadIdx.x] = 0;   // fronts past T stay 0
    __syncthreads();
    if (threadIdx.x < T) {
        s_front[0][threadIdx.x] = (int32_t)a.base[threadIdx.x];
        a.ftab[threadIdx.x] = (int32_t)a.base[threadIdx.x];
    }
    __syncthreads();
    int64_t round = 0;
    int32_t frow = 0;                             // front table rows of the current batch
    for (;;) {
        const int cur = (int)(round & 1);
        // refill this thread's window when less than half of it lies ahead
        if (mine && wend < ce && wend - ci < (W >> 1)) {
            // all loads of a refill are in flight together (one memory latency)
            const int nend = ci + W < ce ? ci + W : ce;
            const int from = wend > ci ? wend : ci;     // entries behind ci are spent
            for (int j0 = from; j0 < nend; j0 += kRefill * 64) {
                CandEnt v[kRefill];
#pragma unroll
                for (int r = 0; r < kRefill; r++) {
                    const int j = j0 + r * 64 + lane;
                    v[r] = a.pent[j < nend ? j : from];
                }
#pragma unroll
                for (int r = 0; r < kRefill; r++) {   // past the end: a spare slot
                    const int j = j0 + r * 64 + lane;
                    CandEnt *dst = j < nend ? &win[j & (W - 1)] : &s_win[kWinE + lane];
                    *dst = v[r];
                }
            }
            wend = nend;
        }
        // advance this thread's front past its ready candidates
        if (mine) {
            int cnew = ce;
            int npos = end;                        // order position of candidate cnew (end if none)
            const int32_t *front = s_front[cur];
            if (f < end) {
                for (;;) {
                    if (ci >= ce) { cnew = ce; break; }
                    if (ci < wend) {
                        const int lim = wend < ce ? wend : ce;
                        const int j = ci + lane;
                        const CandEnt e = win[j & (W - 1)];
                        const bool bl = j < lim && win_blocked(a, e, j, front);
                        const unsigned long long bal = __ballot(bl);
                        if (bal) {
                            const int L = __ffsll((long long)bal) - 1;
                            cnew = ci + L;
                            npos = __builtin_amdgcn_readlane(e.pos, L);   // the finder's entry
                            break;
                        }
                        ci = ci + 64 < lim ? ci + 64 : lim;
                    } else {
                        // past the window (a long ready run): tiles of 4096,
                        // then of 64, then single candidates, 64 per probe
                        int32_t fr[kWinT];         // the round's fronts (wave-uniform)
#pragma unroll
                        for (int q = 0; q < kWinT / 4; q++) {
                            const int4 v = reinterpret_cast<const int4 *>(front)[q];
                            fr[4 * q] = v.x; fr[4 * q + 1] = v.y; fr[4 * q + 2] = v.z; fr[4 * q + 3] = v.w;
                        }
                        auto tile_blocked = [&](const int32_t *row) {
                            bool b = false;
#pragma unroll
                            for (int ts = 0; ts < kWinT; ts++)
                                if (ts < T && row[ts] >= fr[ts]) b = true;
                            return b;
                        };
                        int64_t pos = ci;          // every candidate before pos is ready
                        cnew = ce;
                        while (pos < ce) {
                            const int64_t k2 = pos >> 12, t2 = k2 + lane;
                            const bool b2 = (t2 << 12) < ce && tile_blocked(a.tm2 + t2 * T);
                            const unsigned long long bal2 = __ballot(b2);
                            if (!bal2) { pos = (k2 + 64) << 12; continue; }
                            const int64_t L2 = k2 + __ffsll((long long)bal2) - 1;
                            pos = pos > (L2 << 12) ? pos : (L2 << 12);
                            const int64_t end2 = ce < ((L2 + 1) << 12) ? ce : ((L2 + 1) << 12);
                            const int64_t k1 = pos >> 6, t1 = k1 + lane;
                            const bool b1 = (t1 << 6) < end2 && tile_blocked(a.tm1 + t1 * T);
                            const unsigned long long bal1 = __ballot(b1);
                            if (!bal1) { pos = end2; continue; }
                            const int64_t L1 = k1 + __ffsll((long long)bal1) - 1;
                            pos = pos > (L1 << 6) ? pos : (L1 << 6);
                            const int64_t end1 = ce < ((L1 + 1) << 6) ? ce : ((L1 + 1) << 6);
                            const int64_t j = pos + lane;
                            const CandEnt e1 = a.pent[j < end1 ? j : pos];
                            const bool b0 = j < end1 && win_blocked(a, e1, j, front);
                            const unsigned long long bal0 = __ballot(b0);
                            if (bal0) {
                                const int L = __ffsll((long long)bal0) - 1;
                                cnew = (int)(pos + L);
                                npos = __builtin_amdgcn_readlane(e1.pos, L);
                                break;
                            }
                            pos = end1;
                        }
                        break;
                    }
                }
            } else {
                cnew = ci;
            }
            const int nf = f >= end ? f : (cnew < ce ? npos : end);
            if (lane == 0) {
                s_front[cur ^ 1][t] = nf;
                s_adv[cur][t] = nf > f;
                s_unf[cur][t] = f < end;
            }
            // front table row round + 1: lane (round & 63) keeps it until a
            // batch of 64 rows goes out in one store (a store each round would
            // make the next round wait for it)
            const int slotr = (int)(round & 63);
            frow = lane == slotr ? nf : frow;
            if (slotr == 63) a.ftab[(round - 63 + lane + 1) * T + t] = frow;
            ci = cnew;
            f = nf;
        }
        __syncthreads();
        // every wave reads the same flags: all threads done, or a stall (cycle)
        const uint4 uf = *reinterpret_cast<const uint4 *>(s_unf[cur]);
        const uint4 av = *reinterpret_cast<const uint4 *>(s_adv[cur]);
        const bool unf = (uf.x | uf.y | uf.z | uf.w) != 0;
        const bool adv = (av.x | av.y | av.z | av.w) != 0;
        if (!unf || !adv) {
            if (!unf) {
                // rows of the last, partial batch
                const int slotr = (int)(round & 63);
                if (mine && slotr != 63 && lane <= slotr)
                    a.ftab[(round - slotr + lane + 1) * T + t] = frow;
            } else if (threadIdx.x == 0) {
                a.lw->err = ERR_KAHN_CYCLE;
            }
            break;
        }
        round++;
    }
    if (threadIdx.x == 0) a.lw->result[0] = round;
}

// What follows from the rounds, by one workgroup (a launch of its own: as the
// end of k_kahn_win it cost that kernel's refills their registers, 1.2 ->
// 1.5 ms for 1,633 rounds).  Windowed rounds: where every thread's run of
// every step lies -- the positions of a step start at the sum of the fronts'
// advances before it, its runs follow in thread order.
__global__ __launch_bounds__(kWG) void k_steps(bool windowed, const int32_t *__restrict__ ftab, StepArgs a) {
    __shared__ int s_seg;
    const int64_t R = a.lw->result[0];
    if (a.lw->err) {
        if (threadIdx.x == 0) {
            a.out->err = a.lw->err;
            a.out->n_steps = R;
        }
        return;
    }
    if (threadIdx.x == 0) s_seg = 0;
    __syncthreads();
    const int T = a.T;
    if (windowed) {
        int segs = 0;
        for (int64_t r = threadIdx.x; r <= R; r += kWG) {
            int o = 0;
            for (int z = 0; z < T; z++) o += ftab[r * T + z] - (int)a.base[z];
            a.step_ptr[r] = o;
            if (r < R)
                for (int z = 0; z < T; z++) {
                    const int len = ftab[(r + 1) * T + z] - ftab[r * T + z];
                    a.segoff[r * T + z] = o;
                    o += len;
                    segs += len > 0;
                }
        }
        if (segs) atomicAdd(&s_seg, segs);
    }
    __syncthreads();
    finish_steps(R, windowed ? (int64_t)s_seg : a.lw->result[1], a);
}

// schedule position of every task from the fronts of the windowed rounds: the
// last round whose front on the task's thread lies at or before it
__global__ __launch_bounds__(kBS) void k_place_win(int64_t n, int32_t T, const LevWork *__restrict__ lw,
                                                   const int32_t *__restrict__ ftab,
                                                   const int32_t *__restrict__ segoff,
                                                   const int32_t *__restrict__ order,
                                                   const int32_t *__restrict__ tid,
                                                   int32_t *__restrict__ pos_node, int32_t *__restrict__ pos_of,
                                                   uint8_t *__restrict__ pos_flags,
                                                   int32_t *__restrict__ node_step) {
    const int64_t p = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (p >= n || lw->err) return;
    const int32_t u = order[p], t = tid[u];
    int64_t lo = 0, hi = lw->result[0] - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (ftab[mid * T + t] <= p) lo = mid; else hi = mid - 1;
    }
    const int32_t f = ftab[lo * T + t];
    const int64_t q = segoff[lo * T + t] + (p - f);
    pos_node[q] = u;
    pos_of[u] = (int32_t)q;
    pos_flags[q] = p == f ? 1 : 0;
    node_step[u] = (int32_t)lo;
}

// the same from the segments of the generic rounds
__global__ __launch_bounds__(kBS) void k_place_seg(int64_t n, const LevWork *__restrict__ lw,
                                                   const int64_t *__restrict__ seg_off,
                                                   const int64_t *__restrict__ seg_start,
                                                   const int32_t *__restrict__ seg_step,
                                                   const int32_t *__restrict__ order,
                                                   int32_t *__restrict__ pos_node, int32_t *__restrict__ pos_of,
                                                   uint8_t *__restrict__ pos_flags,
                                                   int32_t *__restrict__ node_step) {
    const int64_t q = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (q >= n || lw->err) return;
    int64_t lo = 0, hi = lw->result[1] - 1;          // last segment with seg_off <= q
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (seg_off[mid] <= q) lo = mid; else hi = mid - 1;
    }
    const int32_t u = order[seg_start[lo] + (q - seg_off[lo])];
    pos_node[q] = u;
    pos_of[u] = (int32_t)q;
    pos_flags[q] = q == seg_off[lo] ? 1 : 0;
    node_step[u] = seg_step[lo];
}

// The gathers of each position (thread predecessor of a run's first task
// without thread carries, then the active cross-thread parents) and the
// records the simulation reads.  A workgroup takes its gather entries with
// one atomic, so the lists of different workgroups lie in any order;
// gat_rng[q] = first entry | entries << 32.
struct RecArgs {
    int64_t n;
    uint64_t mask;
    int32_t with_prev;
    const int32_t *pos_node, *pos_of;
    const uint8_t *pos_flags;
    const int32_t *tid, *prev;
    const int64_t *dur, *gap;
    const uint16_t *cls;
    const int64_t *xin_ptr;
    const int32_t *xin_src;
    const uint8_t *xin_cls;
    LevWork *lw;
    uint64_t *gat_rng;
    int32_t *gat_src, *gat_spos;
    uint8_t *gat_cls;
    int64_t *gat_gap;
    Rec *rec;
    SoloRec *so_rec;
};

__global__ __launch_bounds__(kBS) void k_records(RecArgs a) {
    __shared__ int64_t s_base;
    if (a.lw->err) return;
    const int64_t q = (int64_t)blockIdx.x * kBS + threadIdx.x;
    const bool ok = q < a.n;
    int32_t u = 0, pv = -1;
    int64_t k0 = 0, k1 = 0, ng = 0;
    uint32_t head = 0;
    if (ok) {
        u = a.pos_node[q];
        head = a.pos_flags[q] & 1u;
        pv = a.with_prev && head ? a.prev[u] : -1;
        k0 = a.xin_ptr[u];
        k1 = a.xin_ptr[u + 1];
        ng = pv >= 0 ? 1 : 0;
        for (int64_t k = k0; k < k1; k++) ng += on(a.mask, a.xin_cls[k]);
    }
    int64_t tot;
    const int64_t ex = block_excl_scan<kBS>(ng, &tot);
    if (threadIdx.x == 0) s_base = tot ? (int64_t)atomicAdd(&a.lw->gctr, (unsigned long long)tot) : 0;
    __syncthreads();
    if (!ok) return;
    int64_t o = s_base + ex;
    a.gat_rng[q] = (uint64_t)o | ((uint64_t)ng << 32);
    Rec r;
    r.dur = a.dur[u];
    r.gap = a.gap[u];
    r.node = u;
    r.g0_src = -1; r.g1_src = -1; r.g0_spos = 0; r.g1_spos = 0;
    r.g0_gap32 = 0;
    uint32_t c0 = 0, c1 = 0;
    int i = 0;
    auto add = [&](int32_t s, uint32_t c) {
        const int32_t sp = a.pos_of[s];
        const int64_t g = a.gap[s];
        a.gat_src[o] = s; a.gat_spos[o] = sp; a.gat_cls[o] = (uint8_t)c; a.gat_gap[o] = g;
        o++;
        if (i == 0) { r.g0_src = s; r.g0_spos = sp; r.g0_gap32 = (uint32_t)g; c0 = c; }
        if (i == 1) { r.g1_src = s; r.g1_spos = sp; c1 = c; }
        i++;
    };
    if (pv >= 0) add(pv, 255u);
    for (int64_t k = k0; k < k1; k++)
        if (on(a.mask, a.xin_cls[k])) add(a.xin_src[k], a.xin_cls[k]);
    const int32_t t = a.tid[u];
    r.cls = (uint32_t)a.cls[u] | (c0 << 16) | (c1 << 24);
    int64_t extra = ng > 2 ? ng - 2 : 0;   // count saturates; the gather ranges are exact
    if (extra > 0xFFFFFF) extra = 0xFFFFFF;
    // last task of a run: the next position starts a run (or the schedule ends)
    const bool last = (q + 1 == a.n) || (a.pos_flags[q + 1] & 1);
    r.flags = head | (last ? 2u : 0u) |
              ((uint32_t)(t < kMaxCarryThreads ? t : 0) << 2) | ((uint32_t)extra << 8);
    a.rec[q] = r;
    if (!a.so_rec) return;                   // durations or gaps past 32 bits
    if (extra > 0xFFFF) extra = 0xFFFF;
    a.so_rec[q] = SoloRec{(uint32_t)r.dur, (uint32_t)r.gap, r.node, r.g0_src >= 0 ? r.g0_spos : -1, r.cls,
                          (r.flags & 0xffu) | (r.g1_src >= 0 ? kSoG1 : 0u) | ((uint32_t)extra << 16),
                          r.g1_spos, 0};
}

// Kahn levels from the phase schedule (one workgroup, phases in order)
struct LevelArgs {
    int64_t nsteps;
    const int32_t *step_ptr;
    const int32_t *pos_node;
    const uint8_t *pos_flags;
    const int32_t *prev;
    const int64_t *xin_ptr;
    const int32_t *xin_src;
    const uint8_t *xin_cls;
    uint64_t mask;
    int32_t *level;          // [n] by task
    unsigned long long *max_level;
};

__global__ __launch_bounds__(kWG) void k_levels(LevelArgs a) {
    __shared__ int64_t s_val[kWG];
    __shared__ uint8_t s_head[kWG];
    __shared__ int64_t s_tmp[kWG];
    __shared__ uint8_t s_htmp[kWG];
    __shared__ int64_t s_carry;
    int64_t lmax = 0;
    for (int64_t r = 0; r < a.nsteps; r++) {
        const int64_t p0 = a.step_ptr[r], p1 = a.step_ptr[r + 1];
        if (threadIdx.x == 0) s_carry = INT64_MIN / 4;
        __syncthreads();
        for (int64_t w0 = p0; w0 < p1; w0 += kWG) {
            const int64_t q = w0 + threadIdx.x;
            int64_t x = INT64_MIN / 4;
            uint8_t h = 1;
            int32_t u = -1;
            if (q < p1) {
                u = a.pos_node[q];
                h = a.pos_flags[q] & 1;
                int64_t best = 0;
                if (h && a.prev[u] >= 0) best = (int64_t)a.level[a.prev[u]] + 1;
                for (int64_t k = a.xin_ptr[u]; k < a.xin_ptr[u + 1]; k++)
                    if (on(a.mask, a.xin_cls[k])) {
                        const int64_t l = (int64_t)a.level[a.xin_src[k]] + 1;
                        best = l > best ? l : best;
                    }
                x = best - q;          // level_q - q is a running max inside a run
            }
            if (threadIdx.x == 0 && !h) {   // run continues from the previous window
                x = x > s_carry ? x : s_carry;
            }
            s_val[threadIdx.x] = x;
            s_head[threadIdx.x] = h;
            __syncthreads();
            // segmented inclusive max-scan (Hillis-Steele with head flags)
            for (int d = 1; d < kWG; d <<= 1) {
                int64_t v = s_val[threadIdx.x];
                uint8_t hh = s_head[threadIdx.x];
                if ((int)threadIdx.x >= d && !hh) {
                    const int64_t o = s_val[threadIdx.x - d];
                    v = o > v ? o : v;
                    hh = s_head[threadIdx.x - d];
                }
                s_tmp[threadIdx.x] = v;
                s_htmp[threadIdx.x] = hh;
                __syncthreads();
                s_val[threadIdx.x] = s_tmp[threadIdx.x];
                s_head[threadIdx.x] = s_htmp[threadIdx.x];
                __syncthreads();
            }
            if (q < p1) {
                const int64_t lv = s_val[threadIdx.x] + q;
                a.level[u] = (int32_t)lv;
                lmax = lv > lmax ? lv : lmax;
            }
            __syncthreads();
            if (threadIdx.x == kWG - 1) s_carry = s_val[kWG - 1];
            __syncthreads();
        }
    }
    lmax = wave_max64(lmax);
    if ((threadIdx.x & 63) == 0) atomic_max_hot(a.max_level, (unsigned long long)lmax);
}

__global__ __launch_bounds__(kBS) void k_level_count(int32_t n, const int32_t *__restrict__ level,
                                                     int64_t *__restrict__ cnt) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u < n) atomicAdd((unsigned long long *)&cnt[level[u]], 1ull);
}

__global__ __launch_bounds__(kBS) void k_level_scatter(int32_t n, const int32_t *__restrict__ level,
                                                       int64_t *__restrict__ fill,
                                                       int32_t *__restrict__ pos_node,
                                                       int32_t *__restrict__ pos_of,
                                                       uint8_t *__restrict__ pos_flags,
                                                       int32_t *__restrict__ node_step) {
    const int64_t u = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (u >= n) return;
    const int32_t l = level[u];
    const int64_t q = (int64_t)atomicAdd((unsigned long long *)&fill[l], 1ull);
    pos_node[q] = (int32_t)u;
    pos_of[u] = (int32_t)q;
    pos_flags[q] = 1;            // every task is its own run: thread predecessor gathered
    node_step[u] = l;
}

// (levels) the widest step, the batches and the steps for the host
__global__ __launch_bounds__(kWG) void k_level_finish(int64_t R, StepArgs a) {
    finish_steps(R, a.n, a);
}

__global__ __launch_bounds__(kBS) void k_i64_to_i32(int64_t n, const int64_t *__restrict__ in,
                                                    int32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x;
    if (i < n) out[i] = (int32_t)in[i];
}

}  // namespace

#define CK(x)                                                              \
    do {                                                                   \
        hipError_t e_ = (x);                                               \
        if (e_ != hipSuccess) {                                            \
            snprintf(msg, msg_len, "%s: %s", #x, hipGetErrorString(e_));   \
            st = e_ == hipErrorOutOfMemory ? DD_ENOMEM : DD_EHIP;          \
            goto done;                                                     \
        }                                                                  \
    } while (0)

dd_status levelize_device(const dd_graph *g, uint64_t mask, int32_t mode, dd_sched *sch,
                          hipStream_t s, char *msg, size_t msg_len) {
    dd_status st = DD_OK;
    const int64_t n = g->n;
    const int32_t T = g->n_threads;
    const size_t N1 = (size_t)n + 1;
    const size_t Cmax = (size_t)n;                       // candidates <= tasks
    const size_t Rmax = (size_t)g->n_cross;              // requirements <= cross edges
    const bool windowed = T <= kWinT;
    const bool with_prev = T > kMaxCarryThreads;
    const size_t Gmax = Rmax + (with_prev ? (size_t)n : 0);
    char *m = nullptr;                                   // working memory of the call
    int64_t *lvl_cnt = nullptr;
    int32_t *level = nullptr, *tmp_ptr = nullptr;
    unsigned long long *lmax = nullptr;
    LevelizeOut *out = nullptr, *out_dev = nullptr;
    const int gN = grid_for(n, kBS);
    const int64_t chunk = chunk_len(n, kBS);
    Req rq{g->thread_base, g->order, g->rank, g->thread_id, g->xin_ptr, g->xin_src, g->xin_cls};
    size_t off = 0;
    auto put = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t C1 = (Cmax + 63) / 64, C2 = (C1 + 63) / 64;   // tiles at most
    const size_t o_lw = put(sizeof(LevWork)), o_csum = put(8 * kChunks), o_cidx = put(4 * N1),
                 o_cpos = put(8 * (Cmax + 1)), o_rptr = put(8 * (Cmax + 1)), o_rch = put(4 * (Rmax + 1)),
                 o_rgp = put(8 * (Rmax + 1)), o_pent = put(T <= kEntT ? sizeof(CandEnt) * (Cmax + 1) : 0),
                 o_ftab = put(windowed ? 4 * (size_t)(n + 2) * T : 0),
                 o_segoff = put(windowed ? 4 * (size_t)(n + 1) * T : 0),
                 o_tm1 = put(windowed ? 4 * (C1 + 1) * T : 0), o_tm2 = put(windowed ? 4 * (C2 + 1) * T : 0),
                 o_gen = put(windowed ? 0 : 8 * (5 * (size_t)T + 1)), o_long = put(windowed ? 0 : 4 * (size_t)T),
                 o_sst = put(windowed ? 0 : 8 * N1), o_sof = put(windowed ? 0 : 8 * (N1 + 1)),
                 o_sstep = put(windowed ? 0 : 4 * N1), o_posof = put(4 * N1), o_flags = put(N1);
    LevWork *lw;
    int64_t *csum, *cand_pos, *req_ptr, *req_gpos, *gen, *seg_start, *seg_off;
    int32_t *cidx, *req_chain, *ftab, *segoff, *tm1, *tm2, *long_list, *seg_step, *pos_of;
    uint8_t *pos_flags;
    CandEnt *pent;
    StepArgs sa{};

    sch->n = (int32_t)n;
    sch->mode = mode;
    sch->mask = mask;
    sch->thread_carry = !with_prev;
    {
        void *h = nullptr, *d = nullptr;
        CK(direct_buf(&h, &d));
        out = static_cast<LevelizeOut *>(h);
        out_dev = static_cast<LevelizeOut *>(d);
        static_assert(sizeof(LevelizeOut) <= kDirectBytes, "results fit the buffer");
    }
    memset(static_cast<void *>(out), 0, offsetof(LevelizeOut, steps));
    CK(dalloc(reinterpret_cast<void **>(&m), off, s));
    lw = (LevWork *)(m + o_lw);
    csum = (int64_t *)(m + o_csum); cidx = (int32_t *)(m + o_cidx); cand_pos = (int64_t *)(m + o_cpos);
    req_ptr = (int64_t *)(m + o_rptr); req_chain = (int32_t *)(m + o_rch); req_gpos = (int64_t *)(m + o_rgp);
    pent = T <= kEntT ? (CandEnt *)(m + o_pent) : nullptr;
    ftab = (int32_t *)(m + o_ftab); segoff = (int32_t *)(m + o_segoff);
    tm1 = (int32_t *)(m + o_tm1); tm2 = (int32_t *)(m + o_tm2);
    gen = (int64_t *)(m + o_gen); long_list = (int32_t *)(m + o_long);
    seg_start = (int64_t *)(m + o_sst); seg_off = (int64_t *)(m + o_sof); seg_step = (int32_t *)(m + o_sstep);
    pos_of = (int32_t *)(m + o_posof); pos_flags = (uint8_t *)(m + o_flags);
    // the schedule, sized by bounds (at most n steps), so nothing has to come
    // back to the host before the end
    CK(dalloc_n(&sch->step_ptr, N1, s));
    CK(dalloc_n(&sch->pos_node, N1, s));
    CK(dalloc_n(&sch->node_step, N1, s));
    CK(dalloc_n(&sch->gat_rng, N1, s));
    CK(dalloc_n(&sch->gat_src, Gmax + 1, s));
    CK(dalloc_n(&sch->gat_spos, Gmax + 1, s));
    CK(dalloc_n(&sch->gat_cls, Gmax + 1, s));
    CK(dalloc_n(&sch->gat_gap, Gmax + 1, s));
    CK(dalloc_n(&sch->rec, N1, s));
    CK(dalloc_n(&sch->bat, (size_t)solo_batch_max(n), s));
    CK(dalloc_n(&sch->nbat, 1, s));
    // Records of the one-variant-per-workgroup kernel (one more than n: idle
    // lanes read it); where there is no memory for them, the schedule goes
    // without, and the kernels that need less serve it.
    if (g->dmax < (int64_t(1) << 32) && g->gmax < (int64_t(1) << 32)) {
        const hipError_t e = dalloc_n(&sch->so_rec, N1, s);
        if (e == hipErrorOutOfMemory) (void)hipGetLastError();
        else CK(e);
    }
    if (n == 0) {
        CK(hipMemsetAsync(sch->step_ptr, 0, sizeof(int32_t), s));
        sch->h_step_ptr.assign(1, 0);
        CK(hipStreamSynchronize(s));
        goto done;
    }
    sa = StepArgs{T, with_prev ? 1 : 0, n, g->thread_base, sch->step_ptr, segoff, sch->bat, sch->nbat, lw, out_dev};
    k_req_count<<<(unsigned)((n + chunk - 1) / chunk), kBS, 0, s>>>((int32_t)n, chunk, rq, mask, csum, lw);
    k_req_fill<<<(unsigned)((n + chunk - 1) / chunk), kBS, 0, s>>>((int32_t)n, T, chunk, rq, mask, csum, cidx,
                                                                  cand_pos, req_ptr, req_chain, req_gpos,
                                                                  pent, lw);
    if (windowed) {
        int wlog = 6;                                  // 2^wlog entries per thread
        while ((int64_t)T << (wlog + 1) <= kWinBytes / (int64_t)sizeof(CandEnt)) wlog++;
        k_tile_max<<<(unsigned)C2, kWG, 0, s>>>(cidx + n, T, pent, req_ptr, req_chain, req_gpos, tm1, tm2);
        WinArgs wa{T, wlog, g->thread_base, cidx, pent, req_ptr, req_chain, req_gpos, tm1, tm2, ftab, lw};
        k_kahn_win<<<1, kWG, 0, s>>>(wa);
        k_steps<<<1, kWG, 0, s>>>(true, ftab, sa);
        k_place_win<<<gN, kBS, 0, s>>>(n, T, lw, ftab, segoff, g->order, g->thread_id, sch->pos_node, pos_of,
                                       pos_flags, sch->node_step);
    } else {
        KahnArgs ka{pent, T, n, g->thread_base, cidx, cand_pos, req_ptr, req_chain, req_gpos,
                    gen, gen + T, gen + 2 * (size_t)T, gen + 3 * (size_t)T,
                    gen + 4 * (size_t)T, long_list, seg_start,
                    seg_off, seg_step, sch->step_ptr, lw};
        if (T <= kLdsT) k_kahn_rounds<true><<<1, kWG, 0, s>>>(ka);
        else k_kahn_rounds<false><<<1, kWG, 0, s>>>(ka);
        k_steps<<<1, kWG, 0, s>>>(false, nullptr, sa);
        k_place_seg<<<gN, kBS, 0, s>>>(n, lw, seg_off, seg_start, seg_step, g->order, sch->pos_node, pos_of,
                                       pos_flags, sch->node_step);
    }
    CK(hipGetLastError());
    if (mode == DD_LEVELS) {
        // levels from phases, then tasks sorted by level
        CK(hipStreamSynchronize(s));
        if (out->err) goto cycle;
        const int64_t nph = out->n_steps;
        unsigned long long h_lmax = 0;
        CK(dalloc_n(&level, N1, s));
        CK(dalloc_n(&tmp_ptr, (size_t)nph + 1, s));
        CK(dalloc_n(&lmax, 1, s));
        CK(hipMemsetAsync(lmax, 0, sizeof(unsigned long long), s));
        CK(hipMemcpyAsync(tmp_ptr, sch->step_ptr, sizeof(int32_t) * ((size_t)nph + 1), hipMemcpyDeviceToDevice, s));
        LevelArgs la{nph, tmp_ptr, sch->pos_node, pos_flags, g->thread_prev, g->xin_ptr,
                     g->xin_src, g->xin_cls, mask, level, lmax};
        k_levels<<<1, kWG, 0, s>>>(la);
        CK(hipGetLastError());
        {
            ReadBack rb(s, sizeof(h_lmax));
            CK(rb.add(&h_lmax, lmax, sizeof(h_lmax)));
            CK(rb.finish());
        }
        const int64_t nl = (int64_t)h_lmax + 1;
        CK(dalloc_n(&lvl_cnt, (size_t)nl + 1, s));
        CK(hipMemsetAsync(lvl_cnt, 0, sizeof(int64_t) * ((size_t)nl + 1), s));
        k_level_count<<<gN, kBS, 0, s>>>((int32_t)n, level, lvl_cnt);
        CK(hipGetLastError());
        CK(scan_exclusive(lvl_cnt, lvl_cnt, nl, s));
        k_i64_to_i32<<<grid_for(nl + 1, kBS), kBS, 0, s>>>(nl + 1, lvl_cnt, sch->step_ptr);
        k_level_scatter<<<gN, kBS, 0, s>>>((int32_t)n, level, lvl_cnt, sch->pos_node, pos_of, pos_flags,
                                           sch->node_step);
        k_level_finish<<<1, kWG, 0, s>>>(nl, sa);
        CK(hipGetLastError());
    }
    {
        RecArgs ra{n, mask, with_prev ? 1 : 0, sch->pos_node, pos_of, pos_flags, g->thread_id, g->thread_prev,
                   g->dur, g->gap, g->cls, g->xin_ptr, g->xin_src, g->xin_cls, lw, sch->gat_rng,
                   sch->gat_src, sch->gat_spos, sch->gat_cls, sch->gat_gap, sch->rec, sch->so_rec};
        k_records<<<gN, kBS, 0, s>>>(ra);
        CK(hipGetLastError());
    }
    CK(hipStreamSynchronize(s));
    if (out->err) goto cycle;
    sch->n_steps = out->n_steps;
    sch->n_segments = out->n_segments;
    sch->max_width = out->max_width;
    sch->n_gathers = out->n_gathers;
    if (sch->n_steps <= kSplitMaxSteps)
        sch->h_step_ptr.assign(out->steps, out->steps + sch->n_steps + 1);
    goto done;
cycle:
    snprintf(msg, msg_len, "dependencies plus thread order contain a cycle "
                           "(Kahn rounds stalled after %lld steps)", (long long)out->n_steps);
    st = DD_ECYCLE;
done:
    if (st != DD_OK && st != DD_ECYCLE) (void)hipStreamSynchronize(s);
    dfree(m, s);
    dfree(lvl_cnt, s); dfree(level, s); dfree(tmp_ptr, s); dfree(lmax, s);
    return st;
}

}  // namespace dd
