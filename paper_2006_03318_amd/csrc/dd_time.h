// Time arithmetic and the max-plus wave scan shared by the simulation kernels.
// The files that include this are compiled with IEEE mode off and NaNs
// assumed absent (none ever occurs), so a double max is one instruction.
#pragma once

#include "dd_common.h"
#include "dd_internal.h"

namespace dd {
namespace {

__device__ __forceinline__ int64_t max64(int64_t a, int64_t b) { return a > b ? a : b; }

__device__ __forceinline__ bool cls_on(uint64_t eon, uint8_t c) {
    return c == 255 || ((eon >> c) & 1ull);
}

// 64-bit value from its two 32-bit halves, as one register pair (left
// visible as shift-or, the compiler adds the halves to a sum one at a time)
__device__ __forceinline__ int64_t join64(int lo, int hi) {
    int64_t r = (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    asm("" : "+v"(r));
    return r;
}

// Run heads without flags.  A range of positions maps the release entering
// it to c -> max(c + a, b), with b >= a.  A range that holds the first task of
// a run ignores c; it is written with a = kHead + (its weights after the
// head), so c + a < 0 <= b for every c that occurs: every simulated time is
// below 2^62 (the graph and transform checks reject anything larger), and c
// plus the weights of later positions is itself such a time.  Composing keeps
// a >= kHead, so no sum overflows.
constexpr int64_t kHead = -(int64_t(1) << 62);

// Time arithmetic.  Tm<false>: plain int64.  Tm<true>: every value is an
// integer held in a double, which the hardware adds and compares in one
// full-rate instruction each (int64 takes two to three).  Times are biased
// by 2^52: the double of time t (0 <= t < 2^52) has the bit pattern
// 0x4330000000000000 + t, so moving a time between HBM (int64) and a
// register is one operation on its high word, and the bit patterns of
// nonnegative doubles order as integers do.  Weights (durations, gaps and
// their sums) stay unbiased, and a range holding a run head carries -inf,
// which any sum keeps (c + -inf = -inf loses to every b in a max).  All of
// it is exact while every simulated time stays below 2^51 and every
// duration times the scale numerator below 2^53 (checked on the host; the
// int64 form serves every other launch).  Values travel as int64 bit
// patterns either way.
template <bool FP> struct Tm;
template <> struct Tm<false> {
    static constexpr int64_t zero = 0;          // time 0
    static constexpr int64_t head = kHead;      // weight sum of a range holding a run head
    __device__ static __forceinline__ int64_t add(int64_t x, int64_t y) { return x + y; }
    __device__ static __forceinline__ int64_t sub(int64_t x, int64_t y) { return x - y; }
    __device__ static __forceinline__ int64_t mx(int64_t x, int64_t y) { return max64(x, y); }
    __device__ static __forceinline__ int64_t from_time(int64_t t) { return t; }
    __device__ static __forceinline__ int64_t to_time(int64_t x) { return x; }
    __device__ static __forceinline__ int64_t w32(uint32_t w) { return (int64_t)w; }
    __device__ static __forceinline__ double d(int64_t x) { return __longlong_as_double(x); }
    __device__ static __forceinline__ int64_t i(double x) { return __double_as_longlong(x); }
};
template <> struct Tm<true> {
    static constexpr int64_t zero = 0x4330000000000000ll;                    // 2^52
    static constexpr int64_t head = (int64_t)0xFFF0000000000000ull;          // -inf
    __device__ static __forceinline__ double d(int64_t x) { return __longlong_as_double(x); }
    __device__ static __forceinline__ int64_t i(double x) { return __double_as_longlong(x); }
    __device__ static __forceinline__ int64_t add(int64_t x, int64_t y) { return i(d(x) + d(y)); }
    __device__ static __forceinline__ int64_t sub(int64_t x, int64_t y) { return i(d(x) - d(y)); }
    __device__ static __forceinline__ int64_t mx(int64_t x, int64_t y) {
        return i(__builtin_fmax(d(x), d(y)));
    }
    __device__ static __forceinline__ int64_t from_time(int64_t t) { return t | zero; }
    __device__ static __forceinline__ int64_t to_time(int64_t x) { return x ^ zero; }
    __device__ static __forceinline__ int64_t w32(uint32_t w) { return i((double)w); }
};

// floor(d * p / q) in doubles, for d * p < 2^50 (dd_variants::quot_ok).  With
// x = d * p + 1/2 (exact), x / q lies at least 1/(2q) from any integer; the
// rounded reciprocal and product are off by at most x / q * 2^-52 < 1/(2q),
// so the floor is the quotient.
__device__ __forceinline__ double scale_f64(double d, double p, double iq) {
    return __builtin_floor(__builtin_fma(d, p, 0.5) * iq);
}
// 1 / q of a scale entry.  magic = floor(2^(64 + shift) / q) + 1 with
// q < 2^31, so q is 2^(64 + shift) / magic to the nearest integer; without a
// magic number q = 2^shift.
__device__ __forceinline__ double inv_quotient(const ScaleEntry &e) {
    if (!e.magic) return __builtin_ldexp(1.0, -(int)e.shift);
    return 1.0 / __builtin_rint(__builtin_ldexp(1.0, 64 + (int)e.shift) / (double)e.magic);
}

// (la, lb) then (a, b)
template <bool FP = false>
__device__ __forceinline__ void compose(int64_t la, int64_t lb, int64_t &a, int64_t &b) {
    b = Tm<FP>::mx(Tm<FP>::add(lb, a), b);
    if (FP) a = Tm<FP>::add(la, a);
    else a = a < 0 ? a : la + a;
}

// one Kogge-Stone step of the max-plus scan across the wave, the left
// operand taken with a DPP lane shift (lanes without one see the identity
// (0, 0), as b >= a; in the double form the bits 0 are 0.0, below every
// biased time).  Row shifts write every lane (bound control: 0 where the
// source lies outside the row), so no lane needs its old value.
template <int CTRL, int RMASK, bool FP = false>
__device__ __forceinline__ void scan_step(int64_t &a, int64_t &b) {
    constexpr bool BC = RMASK == 0xf;
    const int alo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)a, CTRL, RMASK, 0xf, BC);
    const int ahi = __builtin_amdgcn_update_dpp(0, (int)((uint64_t)a >> 32), CTRL, RMASK, 0xf, BC);
    const int blo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, RMASK, 0xf, BC);
    const int bhi = __builtin_amdgcn_update_dpp(0, (int)((uint64_t)b >> 32), CTRL, RMASK, 0xf, BC);
    const int64_t la = join64(alo, ahi);
    const int64_t lb = join64(blo, bhi);
    compose<FP>(la, lb, a, b);
}

__device__ __forceinline__ int64_t readlane64(int64_t x, int l) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)x, l);
    const int hi = __builtin_amdgcn_readlane((int)((uint64_t)x >> 32), l);
    return join64(lo, hi);
}

// inclusive scan over the 64 lanes of a wave
template <bool FP = false>
__device__ __forceinline__ void wave_scan(int64_t &a, int64_t &b) {
    scan_step<0x111, 0xf, FP>(a, b);   // row_shr:1
    scan_step<0x112, 0xf, FP>(a, b);   // row_shr:2
    scan_step<0x114, 0xf, FP>(a, b);   // row_shr:4
    scan_step<0x118, 0xf, FP>(a, b);   // row_shr:8
    scan_step<0x142, 0xa, FP>(a, b);   // row_bcast:15 into rows 1 and 3
    scan_step<0x143, 0xc, FP>(a, b);   // row_bcast:31 into rows 2 and 3
}

}  // namespace
}  // namespace dd
