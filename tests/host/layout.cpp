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
        // removal strings: 8-byte stores for 64 positions at a time, and the
        // word that holds bit n inside the string of its own variant
        const int64_t s = dd::rm_stride(n);
        EXPECT(s % 2 == 0 && (n + 63) / 64 * 2 <= s && (n >> 5) < s, n);
    }
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}
