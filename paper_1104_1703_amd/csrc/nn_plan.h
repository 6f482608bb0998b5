// Host side of the weight gradient's split: the z march's plan and the choice
// between the march and the kernel per tap (nn.hip).  No device code.
#pragma once

#include <algorithm>
#include <cmath>

namespace mg {
namespace nn {

constexpr int BW_T = 16;    // edge of a march's column of voxels
constexpr int BW_NT = 512;  // threads of a march's block
constexpr int BW_KV = 32;   // voxels the kernel per tap stages at a time

// Voxel chunk of a block of k_conv_bwd_w_tap: about 2048 blocks over the 27
// taps x channel groups.
inline long long tap_chunk(long long V, int groups) {
    const long long nchunks = std::max(1, 2048 / (27 * groups));
    const long long chunk = (V + nchunks - 1) / nchunks;
    return std::max<long long>(BW_KV, (chunk + BW_KV - 1) / BW_KV * BW_KV);
}

// The march's split: z chunks per column, planes per chunk, columns and channel tiles.
struct MarchPlan {
    int ntx, nty, nzc, zc;
    long long cols, tiles;
};

// The split with the shortest march over the rounds it takes (one block per CU
// at once, two planes more staged than multiplied, and about six steps' worth of
// reduction at the end of a block); splits beyond the bound only add rounds.
inline MarchPlan march_plan(int n, int D, int H, int W, int cin, int cout) {
    MarchPlan m;
    m.ntx = (W + BW_T - 1) / BW_T;
    m.nty = (H + BW_T - 1) / BW_T;
    m.tiles = (long long)(cin / 16) * (cout / 16);
    m.cols = (long long)m.ntx * m.nty * n;
    const long long all = m.cols * m.tiles;
    const int kmax = (int)std::min<long long>(D, std::max<long long>(64, 256 / all + 1));
    int best_k = 1;
    long long best = 0;
    for (int k = 1; k <= kmax; k++) {
        const int zc = (D + k - 1) / k;
        const long long t = (all * ((D + zc - 1) / zc) + 255) / 256 * (zc + 8);
        if (k == 1 || t < best) {
            best = t;
            best_k = k;
        }
    }
    m.zc = (D + best_k - 1) / best_k;
    m.nzc = (D + m.zc - 1) / m.zc;
    return m;
}

// Whether the kernel per tap takes the layer.  Estimated times in us, fitted to
// both kernels at 1487 shapes (1 to 512 samples of 1 to 64 voxels an edge, flat
// and ragged ones among them, 16 to 256 channels; median errors 8 and 5%): the
// kernel per tap takes a block's steps of 32 voxels one after the other, then
// pays per voxel and channel tile and 2.6 ps per atomic of its blocks; the march
// takes 41 ns for each block that adds to the same weights, and per plane 0.61 us
// for a round of 256 blocks and 0.9 ns for each block.
// The line at 1.05 times: over these shapes the choice takes 1.005 times the
// faster kernel's time (geometric mean; 26 shapes more than 1.1 times, 9 more
// than 1.2).  The march also leaves to the other kernel what its grid and its
// 32-bit offsets cannot hold.
inline bool per_tap(const MarchPlan &m, int cin, int cout, long long V, int H, int W) {
    const long long blocks = m.cols * m.nzc * m.tiles;
    if (m.tiles > 65535 || m.cols * m.nzc * BW_NT >= (1LL << 32)) return true;
    if ((long long)H * W * (std::max(cin, cout) / 8) >= (1LL << 31)) return true;
    const int groups = (cout + 63) / 64;
    const double chunk = (double)tap_chunk(V, groups), chunks = std::ceil((double)V / chunk);
    const double tap = 2.1 + chunk / BW_KV * (0.72 + 0.148 * (cin / 16)) + 1.83e-4 * (double)V * groups * (cin / 16) +
                       2.6e-6 * chunks * 27 * groups * std::min(cout, 64) * cin;
    const double march = 0.1 + 0.041 * (double)(m.cols * m.nzc) +
                         (m.zc + 11) * (0.61 * (double)((blocks + 255) / 256) + 0.0009 * (double)blocks);
    return tap < 1.05 * march;
}

}  // namespace nn
}  // namespace mg
