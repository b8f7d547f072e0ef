// Runtime breakdown of every variant (Sec. 6.2, Fig. 6: where the iteration
// time goes once the CPU and the GPU overlap), from a finished simulation:
//   total    = the iteration time (makespan);
//   CPU-only = total minus all GPU kernel runtime, i.e. minus the sum of the
//              scaled durations d' of the kernels kept in the variant;
//   GPU-only = the time the CPU is blocked on the GPU: for every call that
//              waits for GPU work (synchronization, device-to-host copy), its
//              start minus the moment its thread reached it (the release of
//              the previous task on the thread, 0 for the first);
//   CPU+GPU parallel = total - CPU-only - GPU-only.
// A call's start is its finish minus its scaled duration, and a release is
// finish + g', so the finish array alone carries the schedule.
//
// One pass (k_bd_sum) over (chunk of tasks) x (128 variants) per workgroup,
// after a small launch that writes what does not depend on the sums
// (k_bd_init).  Bound: the instructions per (kernel, variant) pair, about
// nine: the workgroup first sorts its chunk's kernels by class in LDS, so a
// lane's scale stays in registers along a run of one class; a wave takes 64
// kernels at a time, lane j loading kernel j's removal words, and then walks
// them with the duration and the removal masks in scalar registers, two
// variants per lane.  Where every duration times its p stays below 2^50 the
// scaled duration is floor((d * p + 0.5) * (1 / q)) in doubles (dd_time.h),
// three instructions for any q.  Sums join the output with one atomic per
// variant and workgroup.  32,768 tasks x 256 variants: 14 us a call (199 with
// a sort of the whole graph by class and four variants per lane), 262,144 x
// 1,000: 69 us (250).

#include "dd_common.h"
#include "dd_internal.h"
#include "dd_time.h"

namespace dd {
namespace {

constexpr int kBT = 256;          // threads per workgroup
constexpr int kBW = kBT / 64;
constexpr int kBV = 128;          // variants per workgroup, two per lane
constexpr int kMaxChunk = 512;    // tasks per workgroup at most
constexpr int kKeys = 1024;       // buckets of the sort (classes, modulo this)

__global__ __launch_bounds__(kBT) void k_bd_init(int32_t V, const int64_t *__restrict__ makespan,
                                                 int64_t *__restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (v >= V) return;
    const int64_t ms = makespan[v];
    out[v * 4 + 0] = ms;
    out[v * 4 + 1] = ms;
    out[v * 4 + 2] = 0;
    out[v * 4 + 3] = 0;
}

struct BdArgs {
    int64_t n;
    int32_t V, W, chunk, bx;      // bx: workgroups per chunk (128 variants each)
    const uint8_t *role;
    const int64_t *dur, *gap;
    const uint16_t *cls;
    const int32_t *tprev;
    const ScaleEntry *table;
    const uint32_t *rm;
    const int64_t *finish;
    unsigned long long *out;      // [V][4]
};

// a kernel of the chunk
struct alignas(16) BdEnt {
    int64_t dur;
    int32_t u;
    uint32_t cls;
};

// scaled duration and its sum, in doubles or (general form) in integers
template <bool F64> struct BdScale;
template <> struct BdScale<true> {
    double p, iq;
    typedef double T;
    __device__ __forceinline__ void set(const ScaleEntry &e) {
        p = (double)e.p;
        iq = inv_quotient(e);
    }
    __device__ __forceinline__ static T dur(int64_t d) { return (double)d; }
    __device__ __forceinline__ T of(T d) const { return scale_f64(d, p, iq); }
    __device__ __forceinline__ static int64_t whole(T x) { return (int64_t)x; }
};
template <> struct BdScale<false> {
    ScaleEntry e;
    typedef int64_t T;
    __device__ __forceinline__ void set(const ScaleEntry &x) { e = x; }
    __device__ __forceinline__ static T dur(int64_t d) { return d; }
    __device__ __forceinline__ T of(T d) const {
        const uint64_t a = (uint64_t)d * (uint64_t)e.p;
        return (int64_t)(e.magic ? (__umul64hi(a, e.magic) >> e.shift) : (a >> e.shift));
    }
    __device__ __forceinline__ static int64_t whole(T x) { return x; }
};

template <bool F64>
__global__ __launch_bounds__(kBT) void k_bd_sum(BdArgs a) {
    typedef BdScale<F64> S;
    typedef typename S::T T;
    __shared__ BdEnt sE[kMaxChunk];           // the chunk's kernels by class
    __shared__ uint32_t sKey[kKeys];          // counts, then first places, of the buckets
    __shared__ int32_t sWait[kMaxChunk];      // its waiting calls
    __shared__ int sNk, sNw;
    __shared__ int64_t sSum[kBW][kBV];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bx = (int)(blockIdx.x % (uint32_t)a.bx);
    const int64_t u0 = (int64_t)(blockIdx.x / (uint32_t)a.bx) * a.chunk;
    const int64_t u1 = u0 + a.chunk < a.n ? u0 + a.chunk : a.n;
    const int64_t V = a.V, W = a.W;
    const int64_t va = (int64_t)bx * kBV + lane, vb = va + 64;   // the lane's variants
    const int64_t vac = va < V ? va : 0, vbc = vb < V ? vb : 0;

    // sort: count, place
    for (int i = tid; i < kKeys; i += kBT) sKey[i] = 0;
    if (tid == 0) { sNk = 0; sNw = 0; }
    __syncthreads();
    constexpr int PER = kMaxChunk / kBT;
    uint32_t rank[PER], c_[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int64_t u = u0 + k * kBT + tid;
        const uint8_t r = u < u1 ? a.role[u] : 0;
        c_[k] = ~0u;
        rank[k] = 0;
        if (r == 1u) {
            c_[k] = a.cls[u];
            rank[k] = atomicAdd(&sKey[c_[k] & (kKeys - 1)], 1u);
        } else if (r == 2u) {
            sWait[atomicAdd(&sNw, 1)] = (int32_t)u;
        }
    }
    __syncthreads();
    {
        constexpr int KP = kKeys / kBT;
        uint32_t cnt[KP];
        int64_t mine = 0, tot;
#pragma unroll
        for (int k = 0; k < KP; k++) { cnt[k] = sKey[tid * KP + k]; mine += cnt[k]; }
        uint32_t at = (uint32_t)block_excl_scan<kBT>(mine, &tot);
#pragma unroll
        for (int k = 0; k < KP; k++) { sKey[tid * KP + k] = at; at += cnt[k]; }
        if (tid == 0) sNk = (int)tot;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
        if (c_[k] == ~0u) continue;
        const int64_t u = u0 + k * kBT + tid;
        sE[sKey[c_[k] & (kKeys - 1)] + rank[k]] = BdEnt{a.dur[u], (int32_t)u, c_[k]};
    }
    __syncthreads();

    // kernels: each wave a contiguous quarter of the sorted list, 64 at a time
    const int nk = sNk;
    const int quarter = (nk + kBW - 1) / kBW;
    const int e0 = wv * quarter, e1 = e0 + quarter < nk ? e0 + quarter : nk;
    const int64_t w0 = (int64_t)bx * (kBV / 32);    // first removal word of the variants
    S sa, sb;
    T ka = 0, kb = 0;
    uint32_t cur = ~0u;
    for (int eb = e0; eb < e1; eb += 64) {
        const int i = eb + lane < e1 ? eb + lane : e1 - 1;
        const BdEnt x = sE[i];
        uint32_t m[kBV / 32];
#pragma unroll
        for (int k = 0; k < kBV / 32; k++) {
            const int64_t w = w0 + k < W ? w0 + k : W - 1;  // (past the last word: variants past V)
            m[k] = a.rm[(int64_t)x.u * W + w];
        }
        const T d = S::dur(x.dur);
        const uint32_t dlo = (uint32_t)__builtin_bit_cast(uint64_t, d),
                       dhi = (uint32_t)(__builtin_bit_cast(uint64_t, d) >> 32);
        const int cnt = e1 - eb < 64 ? e1 - eb : 64;
        for (int j = 0; j < cnt; j++) {
            const uint32_t c = __builtin_amdgcn_readlane(x.cls, j);
            if (c != cur) {                                 // wave-uniform: the class changed
                cur = c;
                sa.set(a.table[(int64_t)c * V + vac]);
                sb.set(a.table[(int64_t)c * V + vbc]);
            }
            const uint64_t db = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(dlo, j) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(dhi, j) << 32);
            const T dj = __builtin_bit_cast(T, db);
            const uint64_t ma = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(m[0], j) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(m[1], j) << 32);
            const uint64_t mb = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(m[2], j) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(m[3], j) << 32);
            const T xa = sa.of(dj), xb = sb.of(dj);
            ka += __builtin_amdgcn_inverse_ballot_w64(ma) ? (T)0 : xa;
            kb += __builtin_amdgcn_inverse_ballot_w64(mb) ? (T)0 : xb;
        }
    }
    sSum[wv][lane] = S::whole(ka);
    sSum[wv][lane + 64] = S::whole(kb);
    __syncthreads();
    {
        // thread tid: variant tid % kBV, and every kBT / kBV-th waiting call
        // (start minus the moment the thread reached the call; 2,048 of them
        // in 256 variants: 135 us before this kernel, 152 with all calls on
        // the first kBV threads, 99 now)
        static_assert(kBT % kBV == 0, "the threads of a variant");
        const int64_t v = (int64_t)bx * kBV + tid % kBV;
        int64_t k = 0, b = 0;
        if (tid < kBV)
#pragma unroll
            for (int w = 0; w < kBW; w++) k += sSum[w][tid];
        const int nw = sNw;
        if (v < V) {
            const int64_t vw = v >> 5;
            const uint32_t bit = (uint32_t)(v & 31);
#pragma unroll 2
            for (int i = tid / kBV; i < nw; i += kBT / kBV) {
                const int64_t u = sWait[i];
                const bool rmu = (a.rm[u * W + vw] >> bit) & 1u;
                S s;
                s.set(a.table[(int64_t)a.cls[u] * V + v]);
                const int64_t dp = rmu ? 0 : S::whole(s.of(S::dur(a.dur[u])));
                const int64_t start = a.finish[u * V + v] - dp;
                const int32_t p = a.tprev[u];
                int64_t reached = 0;
                if (p >= 0) {
                    const bool rmp = (a.rm[(int64_t)p * W + vw] >> bit) & 1u;
                    reached = a.finish[(int64_t)p * V + v] + (rmp ? 0 : a.gap[p]);
                }
                b += start - reached;
            }
            // total - kernels, blocked, the rest (sums of integers: any order)
            if (k) atomicAdd(&a.out[v * 4 + 1], (unsigned long long)-k);
            if (b) atomicAdd(&a.out[v * 4 + 2], (unsigned long long)b);
            if (k - b) atomicAdd(&a.out[v * 4 + 3], (unsigned long long)(k - b));
        }
    }
}

}  // namespace

hipError_t launch_breakdown(const dd_graph *g, const dd_variants *var, const uint8_t *role_dev,
                            const int64_t *finish, const int64_t *makespan, int64_t *out, hipStream_t s) {
    k_bd_init<<<grid_for(var->V, kBT), kBT, 0, s>>>(var->V, makespan, out);
    if (g->n > 0) {
        // chunks as long as leaves about four workgroups per compute unit,
        // from 256 tasks (shorter ones are mostly sorting) to 512 (longer
        // ones leave fewer workgroups resident: 262,144 tasks x 1,000 variants
        // 95 us with 2,048 tasks per chunk, 77 with 1,024, 69 with 512)
        const int64_t bx = (var->V + kBV - 1) / kBV;
        int64_t chunk = kBT;
        while (chunk < kMaxChunk && (g->n + chunk - 1) / chunk * bx > 1024) chunk *= 2;
        const int64_t rows = (g->n + chunk - 1) / chunk;
        BdArgs a{g->n, var->V, var->W, (int32_t)chunk, (int32_t)bx, role_dev, g->dur, g->gap, g->cls,
                 g->thread_prev, var->table, var->rm_bits, finish,
                 reinterpret_cast<unsigned long long *>(out)};
        if (var->quot_ok) k_bd_sum<true><<<(unsigned)(rows * bx), kBT, 0, s>>>(a);
        else k_bd_sum<false><<<(unsigned)(rows * bx), kBT, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace dd
