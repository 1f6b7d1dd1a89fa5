// The fill's grid (rmx_blur.h) over the whole range of unit counts: at least one block, no more
// than the units need, and fewer than 2^32 threads, the most that a launch takes.  Test
// infrastructure only.
#include "hip/hip_runtime.h"
#include "rmx_blur.h"
#include <cstdio>
int main() {
    long bad = 0, n = 0;
    for (int cus : {0, 1, 64, 256, 304}) {
        for (int p = 0; p < 62; ++p) {
            for (int64_t d = -1; d <= 1; ++d) {
                const int64_t units = ((int64_t)1 << p) + d;
                if (units < 1) continue;
                const int64_t g = rmx::fill_blocks(units, cus);
                ++n;
                if (g < 1 || g > (units + 3) / 4 || g * 256 >= ((int64_t)1 << 32)) {
                    printf("%lld units, %d CUs: %lld blocks\n", (long long)units, cus, (long long)g);
                    ++bad;
                }
            }
        }
    }
    printf("fill_blocks_check: %ld counts, %ld bad\n", n, bad);
    return bad != 0;
}
