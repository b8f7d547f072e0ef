// The batch list of the one-variant-per-workgroup kernel (k_solo.hip), built
// by one workgroup when a schedule is made.
#pragma once

#include "dd_common.h"
#include "dd_internal.h"

namespace dd {
namespace {

// Entry b: first position, first step, wide flag; the batch ends where the
// next one begins (the list is closed by an entry {n, steps}).  Narrow steps
// are grouped by the kSoloGroup-aligned span of positions in which they
// start, so a group holds fewer than kSoloGroup + kSoloNarrow positions.
// Every thread of a workgroup of 1,024 calls it.
__device__ void solo_batches(int64_t nsteps, const int32_t *step_ptr, int4 *bat, int32_t *nbat) {
    int64_t carry = 0;
    for (int64_t base = 0; base < nsteps; base += 1024) {
        const int64_t r = base + threadIdx.x;
        int32_t p0 = 0, p1 = 0, pm = 0;
        if (r < nsteps) {
            p0 = step_ptr[r];
            p1 = step_ptr[r + 1];
            pm = r > 0 ? step_ptr[r - 1] : 0;
        }
        const bool wide = p1 - p0 > kSoloNarrow;
        const bool first = r == 0 || p0 - pm > kSoloNarrow || p0 / kSoloGroup != pm / kSoloGroup;
        int64_t cnt = 0;
        if (r < nsteps) cnt = wide ? (p1 - p0 + kSoloPos - 1) / kSoloPos : (first ? 1 : 0);
        int64_t tot;
        const int64_t ex = block_excl_scan<1024>(cnt, &tot);
        for (int64_t i = 0; i < cnt; i++)
            bat[carry + ex + i] = make_int4(p0 + (int32_t)i * kSoloPos, (int32_t)r, wide ? 1 : 0, 0);
        carry += tot;
    }
    if (threadIdx.x == 0) {
        bat[carry] = make_int4(step_ptr[nsteps], (int32_t)nsteps, 1, 0);
        nbat[0] = (int32_t)carry;
    }
}

}  // namespace
}  // namespace dd
