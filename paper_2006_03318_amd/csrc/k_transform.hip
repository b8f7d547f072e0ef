// Per-(class, variant) shrink/scale table (Sec. 4.4, "shrink/scale"
// primitive; the AMP recipe of Sec. 5.1 divides durations by 3 or 2).
//
// A scaled duration is floor(d * p / q) in integer nanoseconds.  To keep the
// simulation kernel free of 64-bit division, each (p, q) becomes a
// multiply-shift:  q = 2^k  ->  (d*p) >> k;  otherwise, with l = ceil(log2 q)
// and m = ceil(2^(62+l) / q),  floor(a / q) = floor(a * m / 2^(62+l)) for
// every a < 2^62 (Granlund & Montgomery, "Division by invariant integers
// using multiplication", PLDI 1994, Thm. 4.2 with N = 62); the load-time
// range check guarantees d * p < 2^62.

#include "dd_common.h"
#include "dd_internal.h"

namespace dd {
namespace {

constexpr int kBS = 256;

__device__ uint32_t ceil_log2(uint32_t q) {
    uint32_t l = 0;
    while ((1u << l) < q) l++;
    return l;
}

constexpr int kTabBlocks = kTransformBlocks;   // grid-stride blocks of the table

// One launch per call: the first blocks build the table and leave what they
// saw (errors, bounds) in host memory, one line per block; the next copy the
// edge-class masks and fold them; the rest copy the removal bits (large ones
// are copied by the runtime).
__global__ __launch_bounds__(kBS) void k_transforms(TransformIn t, ScaleEntry *__restrict__ table,
                                                    int32_t tab_blocks, int32_t mask_blocks,
                                                    TransformOut *__restrict__ out) {
    const int b = (int)blockIdx.x;
    constexpr int NW = kBS / 64;
    __shared__ int64_t red[4][NW];
    const int w = threadIdx.x >> 6;
    const int mb = b - tab_blocks, rb0 = mb - mask_blocks;
    if (rb0 >= 0) {                                  // removal bits
        const int64_t step = (int64_t)(gridDim.x - tab_blocks - mask_blocks) * kBS;
        for (int64_t i = (int64_t)rb0 * kBS + threadIdx.x; i < t.rm_words; i += step)
            t.rm_dst[i] = t.rm_src ? t.rm_src[i] : 0u;
        return;
    }
    if (mb >= 0) {                                   // edge classes
        uint64_t any = 0, all = ~0ull;
        for (int64_t v = (int64_t)mb * kBS + threadIdx.x; v < t.V; v += (int64_t)mask_blocks * kBS) {
            const uint64_t m = t.on_src ? t.on_src[v] : ~0ull;
            if (t.on_dst != t.on_src) t.on_dst[v] = m;
            any |= m;
            all &= m;
        }
        for (int o = 32; o > 0; o >>= 1) {
            any |= (uint64_t)shfl_xor64((int64_t)any, o);
            all &= (uint64_t)shfl_xor64((int64_t)all, o);
        }
        if ((threadIdx.x & 63) == 0) { red[0][w] = (int64_t)any; red[1][w] = (int64_t)all; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < NW; k++) {
                any |= (uint64_t)red[0][k];
                all &= (uint64_t)red[1][k];
            }
            out->used[mb] = any;
            out->all[mb] = all;
        }
        return;
    }
    uint32_t e = 0, mg = 0;
    int64_t pm = 0;
    int64_t rb = 0;
    const int64_t count = (int64_t)t.n_cls * t.V;
    for (int64_t i = (int64_t)b * kBS + threadIdx.x; i < count; i += (int64_t)tab_blocks * kBS) {
        int32_t p = 1, q = 1;
        if (t.scale) { p = t.scale[i].p; q = t.scale[i].q; }
        ScaleEntry se{0ull, 0u, 0u};
        if (p < 0 || q < 1) {
            e |= ERR_SCALE;
        } else {
            se.p = (uint32_t)p;
            const uint32_t uq = (uint32_t)q;
            const uint32_t l = ceil_log2(uq);
            if ((uq & (uq - 1)) == 0) {
                se.shift = l;                       // power of two
            } else {
                // m = floor(2^(62+l) / q) + 1 by long division in base 2^32:
                // 2^(62+l) = hi * 2^64 with hi = 2^(l-2) < q (l >= 2 here)
                uint64_t r = 1ull << (l - 2);
                uint64_t x = r << 32;
                const uint64_t d1 = x / uq;
                r = x % uq;
                x = r << 32;
                const uint64_t d0 = x / uq;
                se.magic = ((d1 << 32) | d0) + 1;  // q is not a power of two: remainder != 0
                se.shift = l - 2;
                mg = 1;
            }
            pm = p > pm ? p : pm;
            const double ratio = (double)p / (double)q;
            const int64_t bits = (int64_t)__double_as_longlong(ratio);   // order-preserving for ratio >= 0
            rb = bits > rb ? bits : rb;
        }
        table[i] = se;
    }
    // wave, then the block's waves through LDS
    pm = wave_max64(pm);
    rb = wave_max64(rb);
    for (int o = 32; o > 0; o >>= 1) {
        e |= (uint32_t)__shfl_xor((int)e, o, 64);
        mg |= (uint32_t)__shfl_xor((int)mg, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][w] = pm; red[1][w] = rb; red[2][w] = e; red[3][w] = mg;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < NW; k++) {
            pm = red[0][k] > pm ? red[0][k] : pm;
            rb = red[1][k] > rb ? red[1][k] : rb;
            e |= (uint32_t)red[2][k];
            mg |= (uint32_t)red[3][k];
        }
        out->blk[b] = TransformOut::Block{e, mg, pm, rb};
    }
}

}  // namespace

hipError_t transforms_device(const TransformIn &t, ScaleEntry *table, TransformOut *out, TransformOut *out_dev,
                             hipStream_t s) {
    const int64_t nb = grid_for((int64_t)t.n_cls * t.V, kBS);
    const int tab = (int)(nb < kTabBlocks ? nb : kTabBlocks);
    int64_t rmb = (t.rm_words + 4 * kBS - 1) / (4 * kBS);
    if (rmb > 512) rmb = 512;
    // one block folds 2,048 masks in the time the launch takes anyway, more
    // share the rest (200,000 variants: 302 us a call with one block for all,
    // 222 with a copy to the host and a loop there, 25 with these)
    const int mask = (int)(t.V > 2048 * kMaskBlocks ? kMaskBlocks : (t.V + 2047) / 2048);
    k_transforms<<<(unsigned)(tab + mask + rmb), kBS, 0, s>>>(t, table, tab, mask, out_dev);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    out->used_mask = 0;
    out->all_mask = ~0ull;
    for (int b = 0; b < mask; b++) {
        out->used_mask |= out->used[b];
        out->all_mask &= out->all[b];
    }
    out->err = out->magic = 0;
    out->pmax = out->rmax_bits = 0;
    for (int b = 0; b < tab; b++) {
        out->err |= out->blk[b].err;
        out->magic |= out->blk[b].magic;
        if (out->blk[b].pmax > out->pmax) out->pmax = out->blk[b].pmax;
        if (out->blk[b].rmax_bits > out->rmax_bits) out->rmax_bits = out->blk[b].rmax_bits;
    }
    return hipSuccess;
}

}  // namespace dd
