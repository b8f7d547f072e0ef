// The sizes that host code gives its launches and arrays, at the edges of
// what the kernels index.  Exit status 0 = every check held.
#include <stdio.h>

#include "dd_internal.h"

static int bad = 0;
#define EXPECT(cond, n)                                                            \
    do {                                                                           \
        if (!(cond)) {                                                             \
            fprintf(stderr, "FAILED: %s at n = %lld\n", #cond, (long long)(n));    \
            bad++;                                                                 \
        }                                                                          \
    } while (0)

int main() {
    const int64_t top = (int64_t(1) << 31) - 1;      // most tasks
    const int64_t sizes[] = {1, 31, 32, 63, 64, 65, 127, 128, 129, 256, 1024, 32768, 163840,
                             top - 1024, top - 1023, top - 1, top};
    for (const int64_t n : sizes) {
        // chunks of tasks: whole workgroups, at most kChunks, all of the tasks
        const int64_t c = dd::chunk_len(n, 256), k = (n + c - 1) / c;
        EXPECT(c > 0 && c % 256 == 0 && k >= 1 && k <= dd::kChunks, n);
        EXPECT(k * c >= n && (k - 1) * c < n, n);
        EXPECT((int64_t)dd::grid_for(n, 1024) * 1024 >= n, n);
        // removal strings: 8-byte stores for 64 positions at a time, and the
        // word that holds bit n inside the string of its own variant
        const int64_t s = dd::rm_stride(n);
        EXPECT(s % 2 == 0 && (n + 63) / 64 * 2 <= s && (n >> 5) < s, n);
    }
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}
