// Host check of the choice between the weight gradient's two kernels
// (csrc/nn_plan.h) against times of both, in us on an MI355X: the chosen one
// takes at most 1.2 times the faster one's.  Exit status 0: it does.
#include <cstdio>

#include "nn_plan.h"

struct Row {
    int n, d, h, w, cin, cout;
    double tap, march;
};
static const Row rows[] = {
    // many small maps, flat maps, few voxels
    {256, 2, 2, 2, 64, 64, 24.3, 278.2},
    {256, 4, 4, 4, 64, 64, 40.9, 265.9},
    {64, 4, 4, 4, 128, 128, 55.6, 189.3},
    {64, 8, 8, 8, 64, 64, 58.7, 84.9},
    {256, 8, 8, 8, 128, 128, 701.6, 1026.8},
    {512, 1, 8, 8, 64, 64, 54.0, 484.7},
    {512, 1, 16, 16, 128, 128, 716.8, 1303.8},
    {512, 1, 1, 64, 192, 64, 158.4, 4052.4},
    {4, 64, 1, 64, 16, 16, 10.7, 23.3},
    {1, 20, 20, 20, 16, 16, 7.8, 12.3},
    // ragged and narrow maps of many channels
    {32, 18, 5, 21, 96, 48, 146.8, 112.1},
    {1, 9, 4, 19, 96, 64, 14.4, 10.9},
    {2, 11, 3, 16, 32, 128, 20.5, 10.4},
    {1, 4, 7, 19, 192, 32, 15.2, 9.1},
    {4, 10, 10, 10, 16, 256, 19.8, 12.4},
    {4, 17, 24, 3, 48, 192, 28.8, 44.2},
    {4, 20, 14, 17, 48, 48, 29.6, 14.0},    // the network's maps and larger ones
    {8, 64, 64, 64, 16, 16, 1105.8, 47.1},
    {1, 64, 64, 64, 16, 16, 141.5, 24.3},
    {16, 16, 16, 16, 192, 64, 331.6, 70.8},
    {16, 12, 12, 12, 128, 128, 164.8, 73.4},
    {256, 12, 12, 12, 16, 16, 227.7, 30.4},
    {1, 48, 48, 48, 16, 64, 80.1, 25.8},
    {512, 1, 32, 32, 16, 16, 289.9, 134.5},
    {1, 96, 96, 96, 64, 64, 1304.2, 264.9},
    {2, 37, 41, 50, 96, 32, 325.0, 77.8},
    {1, 256, 24, 24, 16, 64, 105.9, 29.2},
};

int main() {
    using namespace mg::nn;
    int bad = 0;
    for (const Row &r : rows) {
        const MarchPlan m = march_plan(r.n, r.d, r.h, r.w, r.cin, r.cout);
        const long long V = (long long)r.n * r.d * r.h * r.w;
        const double t = per_tap(m, r.cin, r.cout, V, r.h, r.w) ? r.tap : r.march;
        if (t > 1.2 * std::min(r.tap, r.march)) {
            std::printf("FAILED %d x %d x %d x %d, %d -> %d: %.1f us\n", r.n, r.d, r.h, r.w, r.cin, r.cout, t);
            bad++;
        }
        // the split covers every plane
        if ((long long)m.nzc * m.zc < r.d || (long long)(m.nzc - 1) * m.zc >= r.d) bad++;
    }
    // what the march's grid (channel tiles, work-items) and offsets cannot hold goes to the kernel per tap
    const auto tap = [](int n, int d, int h, int w, int cin, int cout) {
        return per_tap(march_plan(n, d, h, w, cin, cout), cin, cout, (long long)n * d * h * w, h, w);
    };
    if (!tap(1, 64, 256, 256, 192, 16 * 5462)) bad++;   // 65544 channel tiles
    if (tap(1, 64, 256, 256, 192, 16 * 64)) bad++;
    if (!tap(1 << 23, 1, 1, 1, 16, 16)) bad++;           // 2^23 columns of 512 threads
    if (!tap(1, 2, 9472, 9472, 192, 16)) bad++;          // 2^31 pieces of 8 channels in a plane
    if (tap(1, 64, 4096, 4096, 64, 64)) bad++;
    std::printf("conv plan: %d failed\n", bad);
    return bad != 0;
}
