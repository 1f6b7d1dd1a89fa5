// How a grid's blocks share a list (xcd_range, built for the host over the HIP emulation): every
// entry is taken once, and no block takes more entries than an even deal gives.  Test
// infrastructure only.
#include "hip/hip_runtime.h"
#include "rmx_device.h"
#include <cstdio>
#include <vector>
namespace rmx_emu {
thread_local dim3 threadIdx_, blockIdx_;
dim3 blockDim_, gridDim_;
}  // namespace rmx_emu
int main() {
    long bad = 0, n = 0;
    std::vector<int> grids, taken;
    for (int G = 1; G <= 64; ++G) grids.push_back(G);
    for (int G : {100, 767, 1023, 1024, 1025, 70000}) grids.push_back(G);
    for (int G : grids) {
        std::vector<int> counts;
        for (int c = 0; c <= 3 * G + 5 && c <= 4000; ++c) counts.push_back(c);
        for (int c : {G - 1, G, G + 1, 5 * G + 3, 100000}) counts.push_back(c);
        for (int count : counts) {
            gridDim = dim3(G);
            taken.assign(count, 0);
            int most = 0;
            for (int b = 0; b < G; ++b) {
                blockIdx = dim3(b);
                const rmx::dev::XcdRange r = rmx::dev::xcd_range(count);
                int mine = 0;
                for (int e = r.begin; e < r.end; e += r.stride, ++mine)
                    if (e < 0 || e >= count || taken[e]++) ++bad;
                most = std::max(most, mine);
            }
            long left = 0;
            for (int t : taken) left += t == 0;
            ++n;
            if (left || most > (count + G - 1) / G) {
                if (++bad <= 5)
                    printf("%d entries, %d blocks: %ld left, a block takes %d\n", count, G, left, most);
            }
        }
    }
    // the ends of the range: two billion entries, one block and many
    for (int G : {1, 8, 1024, 100003}) {
        gridDim = dim3(G);
        long long all = 0;
        for (int b = 0; b < G; ++b) {
            blockIdx = dim3(b);
            const rmx::dev::XcdRange r = rmx::dev::xcd_range(2000000000);
            if (r.end > r.begin) all += ((long long)r.end - r.begin + r.stride - 1) / r.stride;
        }
        if (all != 2000000000LL) ++bad;
    }
    printf("xcd_range_check: %ld cases, %ld bad\n", n, bad);
    return bad != 0;
}
