// Batched simulation with one variant per workgroup: sweeps whose variants
// all fit on the chip at once, where a schedule's steps set the time.
//
// What is computed is what the other simulation kernels compute (Sec. 4.1,
// Algorithm 1, with the transformations of Sec. 4.4 applied per variant): for
// each task u,
//     d' = removed ? 0 : floor(d * p / q),   g' = removed ? 0 : g
//     start  = max(0, release of every parent present in v)
//     finish = start + d',   release = finish + g'
//     makespan[v] = max finish over tasks not removed in v.
//
// How.  A workgroup of 512 threads walks the whole schedule for one variant,
// a lane per position.  The schedule is cut into batches of at most 512
// positions once, when it is levelized (dd_batches.h): a batch is either a run
// of consecutive narrow steps or a part of a wider step.  Whatever a position
// needs that does not depend on the batch in progress -- its record, removal
// bit, scaled duration, and the release of a parent that finished in an
// earlier batch -- is loaded one to two batches ahead by all lanes.  Then
//   * a narrow batch is resolved by one wave, step after step, with no
//     barrier and no global memory in between: the releases of recent
//     positions sit in an LDS window (positions modulo its size), 64
//     positions are a few LDS reads, a DPP scan as deep as the step is wide,
//     and an LDS write.  The other waves meanwhile wait at the barrier;
//   * a wide batch is resolved by all waves: one DPP scan per wave, one
//     exchange of the wave totals.
// All lanes then store their positions' results.
//
// Bound: the chain of steps (the latency of each) for narrow ones, the
// instructions of the workgroup for wide ones.  With one variant per
// workgroup every finish goes to a cache line of its own, so everything else
// is laid out for contiguous access: records of 32 bytes read as two 16-byte
// loads per lane, removal bits transposed to one bit string per variant
// (k_rm_bits), and every release written a second time into a ring of recent
// positions per variant, from which the parents' releases are gathered
// (parents of neighbouring positions are neighbours themselves in a trace).
//
// Times are integers held in doubles (dd_time.h): launches whose times or
// durations do not fit that form go to the strip kernel.

#include "dd_common.h"
#include "dd_internal.h"
#include "dd_time.h"

#include <type_traits>

namespace dd {
namespace {

constexpr int kSoNT = kSoloPos;        // threads per workgroup: one per position of a batch
constexpr int kSoW = kSoNT / 64;

struct SoloArgs {
    const int32_t *step_ptr;
    const SoloRec *rec;           // [n] by position
    const uint64_t *gat_rng;      // all gathers of a position: first entry | entries << 32
    const int32_t *gat_src, *gat_spos;
    const uint8_t *gat_cls;
    const int64_t *gap;           // [n] gap of every task
    const ScaleEntry *table;      // [n_cls][V]
    const uint32_t *rm;           // [n][W] removal bits by task
    const uint32_t *rmb;          // [V][rmb_stride] removal bits by schedule position
    const uint64_t *edge_on;      // [V]
    uint64_t cls_mask;            // edge classes present in the schedule's gathers
    int32_t n_cls, V, W, thread_carry;
    int64_t rmb_stride;
    int64_t *ring;                // [V][ring_size] releases of recent positions
    int32_t ring_size;            // a power of two
    int64_t *finish, *start, *makespan;
    int64_t *dummy;               // [2 * waves] target of stores from idle lanes
};

// Removal bits by schedule position, one bit string per variant.  A wave
// takes 64 positions and one word of their rows: bit j of the 64 words is a
// ballot, kept by lane j, so 32 lanes then store 8 bytes each.
__global__ __launch_bounds__(256) void k_rm_bits(int64_t n, int32_t V, int32_t W, int64_t stride,
                                                 const int32_t *__restrict__ pos_node,
                                                 const uint32_t *__restrict__ rm,
                                                 uint32_t *__restrict__ rmb) {
    const int lane = threadIdx.x & 63;
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
    if (q0 >= n) return;
    const int64_t q = q0 + lane;
    const int64_t u = q < n ? (pos_node ? pos_node[q] : q) : 0;
    for (int w = blockIdx.y; w < W; w += gridDim.y) {
        const uint32_t x = q < n ? rm[u * W + w] : 0u;
        uint64_t mine = 0;
#pragma unroll
        for (int j = 0; j < 32; j++) {
            const uint64_t m = __ballot((x >> j) & 1u);
            mine = lane == j ? m : mine;
        }
        const int64_t v = (int64_t)w * 32 + lane;
        if (lane < 32 && v < V) *reinterpret_cast<uint64_t *>(rmb + v * stride + (q0 >> 5)) = mine;
    }
}

// one scale entry as the kernel keeps it (scale_f64)
struct alignas(16) SoScale {
    double p, iq;
};

typedef __attribute__((address_space(1))) int64_t so_gi64;

// What is known of a position before its batch is resolved, as a narrow batch
// keeps it in LDS.  Parents still to come are byte offsets into the LDS
// window; an absent one points at a word past it that holds time zero, so
// that reading it changes nothing, and so does the thread carry of a task
// that does not start a run.
struct alignas(16) SoPos {
    int64_t x;          // latest release among the parents of earlier batches
    int64_t w;          // duration + gap as transformed
    uint32_t i0, i1;    // first and second parent
    uint32_t i23;       // two more (16 bits each)
    uint32_t fl;        // bit 0 run head, 1 last of its run (with thread carries), 2..8 carry
                        // to read, 9..14 thread, 15 two more parents, 16 further parents
};
constexpr uint32_t kSoHead = 1u, kSoLast = 2u, kSoTwo = 1u << 15, kSoMore = 1u << 16;

template <bool START>
__global__ __launch_bounds__(kSoNT, 4) void k_sim_solo(const int4 *__restrict__ bat,
                                                       const int32_t *__restrict__ nbat, SoloArgs a) {
    typedef Tm<true> TM;
    constexpr int WIN = 2 * kSoNT;            // two batches
    constexpr uint32_t kNone = WIN * 8u;      // the word that holds time zero
    __shared__ int64_t sR[WIN + 1];           // releases of recent positions
    __shared__ SoPos sP[kSoNT];               // a narrow batch, as far as known
    __shared__ int32_t sPh[kSoNT + 1];        // step offsets of a narrow batch
    __shared__ int64_t sSA[2][kSoW], sSB[2][kSoW];
    __shared__ int64_t sTC[kMaxCarryThreads + 1];   // thread carries, time zero
    __shared__ unsigned long long sMs;
    extern __shared__ SoScale sT[];           // [n_cls]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups of one XCD (b % 8) own neighbouring variants, so the lines
    // of a task row are completed in one L2
    const int xcd = blockIdx.x & 7, share = gridDim.x >> 3, rest = gridDim.x & 7;
    const int v = xcd * share + (xcd < rest ? xcd : rest) + (blockIdx.x >> 3);
    const int64_t V = a.V, W = a.W;
    const int vw = v >> 5;
    const int vb = v & 31;
    const uint64_t eon = a.edge_on[v];
    const bool all_on = (eon & a.cls_mask) == a.cls_mask;
    const bool tcar = a.thread_carry != 0;
    const int nb = *nbat;
    const uint32_t rmask = (uint32_t)a.ring_size - 1u;
    so_gi64 *const ring = (so_gi64 *)(a.ring + (int64_t)v * a.ring_size);
    const uint32_t *const rmb = a.rmb + (int64_t)v * a.rmb_stride;
    so_gi64 *const dummy = (so_gi64 *)(a.dummy + wv * 2);

    for (int c = tid; c < a.n_cls; c += kSoNT) {
        const ScaleEntry e = a.table[(int64_t)c * V + v];
        sT[c] = SoScale{(double)e.p, inv_quotient(e)};
    }
    if (tid <= kMaxCarryThreads) sTC[tid] = TM::zero;
    if (tid == 0) {
        sMs = 0ull;
        sR[WIN] = TM::zero;
    }

    // batches b, b+1, b+2 (clamped to the closing entry: no positions)
    struct Bat { int p0, p1, f, np, wide; };
    auto bat_of = [&](int b, const int4 &x, const int4 &y) -> Bat {
        return Bat{x.x, b < nb ? y.x : x.x, x.y, y.y - x.y, x.z};
    };
    auto entry = [&](int b) -> int4 { return bat[b < nb ? b : nb]; };

    // stage 1: the record of the lane's position (and a step offset, if narrow)
    struct Raw { uint4 u, w; uint32_t rm; int32_t ph; };
    auto load_raw = [&](const Bat &B, Raw &r) {
        const uint32_t q = (uint32_t)(B.p0 + (tid < B.p1 - B.p0 ? tid : 0));   // (up to n: so_rec and rmb hold it)
        const uint4 *s = reinterpret_cast<const uint4 *>(a.rec + q);
        r.u = s[0];
        r.w = s[1];
        r.rm = rmb[q >> 5];
        r.ph = 0;
        if (!B.wide) r.ph = a.step_ptr[(uint32_t)(B.f + (tid < B.np ? tid : B.np))];
    };
    // stage 2: the release of the first parent when it is in the ring:
    // positions from rlo (the oldest kept) up to lo (the first of the batch
    // in progress)
    auto load_dep = [&](const Raw &r, int lo, int rlo) -> int64_t {
        const int sp = (int)r.u.w;
        return ring[(uint32_t)(sp >= rlo && sp < lo ? sp : 0) & rmask];
    };
    // release of a parent older than the ring, loaded on demand
    auto old_rel = [&](int64_t s) -> int64_t {
        const uint32_t rw = a.rm[s * W + vw];
        const int64_t f = a.finish[s * V + v];
        const uint32_t g = (uint32_t)a.gap[s];
        return TM::add(TM::from_time(f), ((rw >> vb) & 1u) ? 0 : TM::w32(g));
    };
    int64_t gp = 0;                           // the lane's position: gap, duration as transformed
    int64_t dp = 0;
    int32_t node = 0;
    bool live = false;
    // stage 3: a position as far as it is known before its batch
    auto prep = [&](const Bat &B, const Raw &r, int64_t g0, int lo, int rlo) -> SoPos {
        SoPos o;
        const int q = B.p0 + tid;
        const bool ok = q < B.p1;
        const uint32_t cl = r.w.x, flags = ok ? r.w.y : 0u;
        const SoScale sc = sT[ok ? cl & 0xffffu : 0u];
        const double t = scale_f64((double)r.u.x, sc.p, sc.iq);
        live = ok && !((r.rm >> (q & 31)) & 1u);
        dp = live ? TM::i(t) : 0;
        gp = live ? TM::w32(r.u.y) : 0;
        o.w = TM::add(dp, gp);
        node = (int)r.u.z;
        int s0 = ok ? (int)r.u.w : -1;
        if (!all_on) s0 = cls_on(eon, (cl >> 16) & 0xffu) ? s0 : -1;
        int64_t x = s0 >= rlo && s0 < lo && s0 >= 0 ? g0 : TM::zero;
        o.i0 = s0 >= lo && s0 >= 0 ? ((uint32_t)s0 & (WIN - 1)) * 8u : kNone;
        o.i1 = kNone;
        uint32_t i2 = kNone, i3 = kNone;
        const bool far0 = s0 >= 0 && s0 < rlo;
        uint32_t more = 0;
        if (__any(far0 | (flags >= kSoG1))) {
            // rarer cases: a parent older than the ring, further parents (the
            // second to fourth here, the rest when the batch is resolved)
            if (far0) x = TM::mx(x, old_rel(a.gat_src[(uint32_t)a.gat_rng[q]]));
            if ((flags & kSoG1) && cls_on(eon, cl >> 24)) {
                const int s1 = (int)r.w.z;
                if (s1 >= lo) o.i1 = ((uint32_t)s1 & (WIN - 1)) * 8u;
                else if (s1 >= rlo) x = TM::mx(x, ring[(uint32_t)s1 & rmask]);
                else x = TM::mx(x, old_rel(a.gat_src[(uint32_t)a.gat_rng[q] + 1u]));
            }
            const uint32_t extra = flags >> 16;
            if (extra > 2u) more = kSoMore;
            else if (extra != 0u) {
                more = kSoTwo;
                const int64_t e0 = (int64_t)(uint32_t)a.gat_rng[q] + 2;
                for (uint32_t z = 0; z < extra; z++) {
                    const int32_t sp = a.gat_spos[e0 + z];
                    if (!cls_on(eon, a.gat_cls[e0 + z])) continue;
                    const uint32_t at = ((uint32_t)sp & (WIN - 1)) * 8u;
                    if (sp < lo) x = TM::mx(x, sp >= rlo ? ring[(uint32_t)sp & rmask] : old_rel(a.gat_src[e0 + z]));
                    else if (z == 0) i2 = at;
                    else i3 = at;
                }
            }
        }
        o.x = x;
        o.i23 = i2 | (i3 << 16);
        const uint32_t th = (flags >> 2) & 63u, head = flags & kSoHead;
        o.fl = head | (tcar ? flags & kSoLast : 0u) | ((head && tcar ? th : (uint32_t)kMaxCarryThreads) << 2) |
               (th << 9) | more;
        return o;
    };
    static_assert(kNone < 0x10000u, "window offsets are 16 bits");
    // the window word at a byte offset
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) int64_t lds_i64;
    lds_char *const win = (lds_char *)&sR[0];
    auto wrel = [&](uint32_t off) -> int64_t { return *(lds_i64 *)(win + off); };
    // a narrow batch goes to LDS for the wave that resolves it
    auto put_prep = [&](const Bat &B, const SoPos &o, int32_t ph) {
        sP[tid] = o;
        if (tid <= B.np) sPh[tid] = ph - B.p0;
    };
    // latest release among a position's parents
    auto parents = [&](const SoPos &o) -> int64_t {
        // (read on every lane: an absent parent reads time zero)
        int64_t y0 = wrel(o.i0), y1 = wrel(o.i1), tc = sTC[(o.fl >> 2) & 127u];
        asm volatile("" : "+v"(y0), "+v"(y1), "+v"(tc));
        return TM::mx(TM::mx(o.x, tc), TM::mx(y0, y1));
    };
    // parents beyond four (beyond two, where there are more than four): the
    // wave's lanes share such a position's list; a parent before lo is read
    // from memory, a later one from the LDS window
    auto many_parents = [&](bool more, int q, int lo, int64_t &x) {
        uint64_t todo = __ballot(more);
        while (todo) {
            const int ld = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int qs = __shfl(q, ld, 64);
            const uint64_t rg = a.gat_rng[qs];
            const int64_t e0 = (int64_t)(uint32_t)rg + 2, e1 = (int64_t)(uint32_t)rg + (int64_t)(rg >> 32);
            int64_t mx = 0;
            for (int64_t e = e0 + lane; e < e1; e += 64) {
                const int32_t sp = a.gat_spos[e];
                const int64_t rel = sp < lo ? old_rel(a.gat_src[e]) : sR[sp & (WIN - 1)];
                if (cls_on(eon, a.gat_cls[e])) mx = TM::mx(mx, rel);
            }
            mx = wave_max64(mx);              // (bit patterns of nonnegative doubles order as integers)
            if (lane == ld) x = TM::mx(x, mx);
        }
    };
    auto rarer_parents = [&](const SoPos &o, int q, int lo, int64_t &x) {
        if (__any(o.fl & kSoTwo)) x = TM::mx(x, TM::mx(wrel(o.i23 & 0xffffu), wrel(o.i23 >> 16)));
        if (__any(o.fl & kSoMore)) many_parents(o.fl & kSoMore, q, lo, x);
    };
    // the oldest position in the ring until batch B is resolved
    auto ring_lo = [&](const Bat &B) { return B.p0 - (int)(rmask + 1u); };

    Bat B0, B1, B2;
    int4 e3;
    {
        const int4 x0 = entry(0), x1 = entry(1), x2 = entry(2);
        e3 = entry(3);
        B0 = bat_of(0, x0, x1);
        B1 = bat_of(1, x1, x2);
        B2 = bat_of(2, x2, e3);
    }
    SoPos P;
    Raw R1;
    {
        Raw R0;
        load_raw(B0, R0);
        load_raw(B1, R1);
        __syncthreads();                      // the scale table
        P = prep(B0, R0, 0, 0, 0);
        if (!B0.wide) put_prep(B0, P, R0.ph);
        __syncthreads();
    }

    int64_t carry = TM::zero, ms = TM::zero;
    int par = 0;
    // one batch; the ring loads of the next one and the records of the one
    // after it are issued first, so they are in flight while it is resolved
    auto batch = [&](auto wide_tag, int b) {
        constexpr bool WIDE = decltype(wide_tag)::value;
        const int lo = B0.p0;
        const int64_t D1 = load_dep(R1, lo, ring_lo(B1));
        Raw R2;
        load_raw(B2, R2);
        const int4 e4 = entry(b + 4);
        const int q0 = B0.p0 + tid;
        int64_t Rv;
        if constexpr (WIDE) {
            int64_t X = parents(P);
            if (__any(P.fl >= kSoTwo)) rarer_parents(P, q0, lo, X);
            // (idle lanes: the identity, as their time is zero)
            int64_t sa = (P.fl & kSoHead) ? TM::head : P.w;
            int64_t sb = TM::add(X, P.w);
            wave_scan<true>(sa, sb);
            if (lane == 63) {
                sSA[par][wv] = sa;
                sSB[par][wv] = sb;
            }
            __syncthreads();
            // lane w: the release after wave w (every 8 lanes alike)
            int64_t ta = sSA[par][lane & (kSoW - 1)], tb = sSB[par][lane & (kSoW - 1)];
            static_assert(kSoW == 8, "three scan steps");
            scan_step<0x111, 0xf, true>(ta, tb);
            scan_step<0x112, 0xf, true>(ta, tb);
            scan_step<0x114, 0xf, true>(ta, tb);
            const int64_t cl = TM::mx(TM::add(carry, ta), tb);
            const int64_t cw = wv > 0 ? readlane64(cl, wv - 1) : carry;
            carry = readlane64(cl, kSoW - 1);
            par ^= 1;
            Rv = TM::mx(TM::add(cw, sa), sb);
            if (q0 < B0.p1) sR[q0 & (WIN - 1)] = Rv;
            if (P.fl & kSoLast) sTC[(P.fl >> 9) & 63u] = Rv;
        } else {
            if (wv == 0) {
                // narrow steps, one after the other, 64 positions at a time;
                // what a position needs is fetched while the ones before it
                // are resolved
                int s = 0;                                // step
                int c0 = 0;                               // first position (in the batch)
                int s1 = __builtin_amdgcn_readfirstlane(sPh[1]);
                const int end = B0.p1 - B0.p0;
                SoPos nx = sP[lane];
                int64_t cr = TM::zero;                    // release before c0
                while (c0 < end) {
                    const int w = s1 - c0 < 64 ? s1 - c0 : 64;
                    const bool ok = lane < w;
                    const SoPos o = nx;
                    const int q = B0.p0 + c0 + lane;
                    int64_t X = parents(o);
                    c0 += w;
                    const bool ends = c0 == s1;
                    if (ends) {                           // the next step
                        s++;
                        s1 = __builtin_amdgcn_readfirstlane(sPh[s < B0.np ? s + 1 : s]);
                    }
                    const int j = c0 + lane;
                    nx = sP[j < kSoNT ? j : kSoNT - 1];
                    if (__any(ok && o.fl >= kSoTwo)) {
                        SoPos z = o;
                        if (!ok) z.fl = 0u;
                        rarer_parents(z, q, lo, X);
                    }
                    int64_t sa = (o.fl & kSoHead) ? TM::head : o.w;
                    int64_t sb = TM::add(X, o.w);
                    // the release before these positions, when they continue a step
                    if (!(o.fl & kSoHead) && lane == 0) sb = TM::mx(TM::add(cr, sa), sb);
                    if (w > 1) {
                        scan_step<0x111, 0xf, true>(sa, sb);
                        if (w > 2) {
                            scan_step<0x112, 0xf, true>(sa, sb);
                            if (w > 4) {
                                scan_step<0x114, 0xf, true>(sa, sb);
                                if (w > 8) {
                                    scan_step<0x118, 0xf, true>(sa, sb);
                                    if (w > 16) scan_step<0x142, 0xa, true>(sa, sb);
                                    if (w > 32) scan_step<0x143, 0xc, true>(sa, sb);
                                }
                            }
                        }
                    }
                    if (ok) {
                        sR[q & (WIN - 1)] = sb;
                        if (o.fl & kSoLast) sTC[(o.fl >> 9) & 63u] = sb;
                    }
                    if (!ends) cr = readlane64(sb, 63);
                }
            }
            __syncthreads();
            Rv = sR[q0 & (WIN - 1)];
        }
        // results: one store each on every path
        {
            const bool ok = q0 < B0.p1;
            const int64_t F = TM::sub(Rv, gp);
            ms = live ? TM::mx(ms, F) : ms;
            const int64_t off = (int64_t)((uint64_t)(uint32_t)node * (uint64_t)(uint32_t)a.V) + v;
            so_gi64 *o = ok ? (so_gi64 *)(a.finish + off) : dummy;
            so_gi64 *rg = ok ? ring + ((uint32_t)q0 & rmask) : dummy;
            asm volatile("" : "+v"(o));
            asm volatile("" : "+v"(rg));
            *o = TM::to_time(F);
            *rg = Rv;
            if (START) {
                so_gi64 *os = ok ? (so_gi64 *)(a.start + off) : dummy;
                asm volatile("" : "+v"(os));
                *os = TM::to_time(TM::sub(F, dp));
            }
        }
        // the next batch, as far as it is known now
        P = prep(B1, R1, D1, lo, ring_lo(B1));
        if (!B1.wide) put_prep(B1, P, R1.ph);
        // the records of the batch after it have landed (on this path: the
        // stores issued since need not have)
        asm volatile("" ::"v"(R2.u.x), "v"(R2.w.x), "v"(R2.rm));
        R1 = R2;
        B0 = B1;
        B1 = B2;
        B2 = bat_of(b + 3, e3, e4);
        e3 = e4;
        __syncthreads();
    };
    for (int b = 0; b < nb;) {
        for (; b < nb && B0.wide; b++) batch(std::true_type{}, b);
        for (; b < nb && !B0.wide; b++) batch(std::false_type{}, b);
    }
    ms = wave_max64(ms);
    if (lane == 0) atomicMax(&sMs, (unsigned long long)ms);
    __syncthreads();
    if (tid == 0) a.makespan[v] = TM::to_time((int64_t)sMs);
}

template <bool START>
hipError_t launch_k(const dd_sched *sch, const SoloArgs &args, hipStream_t s) {
    const size_t dyn = sizeof(SoScale) * (size_t)args.n_cls;
    k_sim_solo<START><<<(unsigned)args.V, kSoNT, dyn, s>>>(sch->bat, sch->nbat, args);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rm_bits(int64_t n, int32_t V, int32_t W, int64_t stride, const int32_t *order,
                          const uint32_t *rm, uint32_t *rmb, hipStream_t s) {
    const int64_t bx = (n + 255) / 256;
    // enough blocks along the words that few positions still fill the chip
    int64_t by = bx < 1024 ? 1024 / bx : 1;
    if (by > W) by = W;
    k_rm_bits<<<dim3((unsigned)bx, (unsigned)by), 256, 0, s>>>(n, V, W, stride, order, rm, rmb);
    return hipGetLastError();
}

hipError_t launch_solo(const dd_graph *g, const dd_sched *sch, const dd_variants *var,
                       int64_t *finish, int64_t *start, int64_t *makespan, hipStream_t s) {
    // scratch of the call: removal bits by position, the rings, the target
    // of idle lanes' stores
    const int64_t n = g->n;
    const int64_t stride = rm_stride(n);
    int32_t ring = kSoloPos;
    while (ring < kSoloRing && ring < n) ring <<= 1;
    uint32_t *rmb = nullptr;
    int64_t *rings = nullptr;
    hipError_t e = dalloc_n(&rmb, (size_t)var->V * (size_t)stride, s);
    if (e == hipSuccess) e = dalloc_n(&rings, (size_t)var->V * (size_t)ring + 16, s);
    if (e == hipSuccess) {
        e = launch_rm_bits(n, var->V, var->W, stride, sch->pos_node, var->rm_bits, rmb, s);
    }
    if (e == hipSuccess) {
        SoloArgs args{sch->step_ptr, sch->so_rec, sch->gat_rng, sch->gat_src, sch->gat_spos,
                      sch->gat_cls, g->gap, var->table, var->rm_bits, rmb, var->edge_on,
                      sch->mask & g->cross_mask, var->n_cls, var->V, var->W,
                      sch->thread_carry ? 1 : 0, stride, rings + 16, ring, finish, start, makespan,
                      rings};
        e = start ? launch_k<true>(sch, args, s) : launch_k<false>(sch, args, s);
    }
    dfree(rmb, s);
    dfree(rings, s);
    return e;
}

}  // namespace dd
