// Kernels of the learned initial guess: a 3D U-Net whose convolutions are
// implicit GEMMs on the gfx950 BF16 matrix cores (v_mfma_f32_16x16x32_bf16),
// BF16 storage and FP32 accumulation.  Tensors are channels-last (NDHWC):
// element (n, z, y, x, c) at ((((n*D + z)*H + y)*W + x)*C + c).
//
// Convolution (3x3x3, zero padding, stride 1) as a GEMM: M = voxels,
// N = output channels, K = 27 taps x input channels.  A wave owns 4 x 16
// voxels by NTC x 16 output channels.  At each K step of 32, lane l supplies
// row (l mod 16) of A and column (l mod 16) of B as 8 consecutive K entries
// starting at 8*(l div 16); with channels-last tensors and [tap][co][ci]
// weights both are single 16-byte reads (A from a halo tile in LDS, B from
// global memory).  The input may be the channel concatenation of a tensor
// read at half resolution (nearest up-sampling, resolved while the tile is
// staged) and a full-resolution tensor.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "mg.h"
#include "mg_core.h"
#include "nn_core.h"
#include "nn_plan.h"

namespace mg {
namespace nn {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NTH = 256;

__device__ __forceinline__ bf16x8 zero8() {
    bf16x8 z;
#pragma unroll
    for (int j = 0; j < 8; j++) z[j] = (bf16)0.0f;
    return z;
}

__device__ __forceinline__ f32x4 mfma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------ conv fwd, LDS tiles
// out = [ReLU](conv3x3x3(concat(up2?(ina), inb)) + bias) as an implicit GEMM
// (M = voxels, N = output channels, K = 27 taps x input channels), organised
// around LDS: a block owns a 16 x 4 x 4 tile of output voxels of one sample
// and, for each chunk of CK input channels, stages the 18 x 6 x 6 halo of its
// input in LDS (zeros outside the box, nearest up-sampling and the skip
// concatenation resolved while staging).  The tap loop then reads every A
// fragment from LDS at a uniform tap offset, with no bounds tests.  Wave w
// computes z-plane w of the tile; its fragment mt is row y = mt, lane row r
// the voxel x = r.  With CK = 32 a voxel's LDS row is 40 channels long (an odd
// number of 16-byte bank groups), so the 16 x-consecutive rows of a fragment
// fall in 16 distinct bank groups.  Rows of 16 channels are not padded: the
// eight lanes a 16-byte read serves at a time fall in distinct groups anyhow,
// and a tile of 21 KB lets seven blocks share a CU instead of five (16 -> 16
// channels on 8 x 64^3 57 -> 50 us).  A chunk holding only 16 input channels (CK = 16,
// or with HALF the last chunk when C_in = 32 q + 16) takes two taps per K step
// of 32 (lane groups 0, 1: tap 2p; 2, 3: tap 2p + 1) instead of padding K
// with zeros.
//
// The products take the weights as A and the voxels as B, so that a lane ends
// with four channels of one voxel: one 8-byte store instead of four of two
// bytes.  All pieces of a tile are in flight together while it is staged, the
// weights run a tap row ahead of the products, and every LDS address is a
// constant beyond a base per lane.  8 x 64^3 voxels, before and after: 16 -> 16
// channels 95 -> 50 us (134 MB: 2.7 TB/s, bound by its LDS reads and the
// staging's latency), 16 -> 48 278 -> 137 us (three channel groups share a
// tile: 268 MB at 2.0 TB/s), 48 -> 16 (32 up-sampled) 212 -> 152 us; 8 x 32^3:
// 96 -> 32 72 -> 58 us (750 TFLOP/s); 8 x 8^3: 128 -> 128 24 -> 20 us (bound by
// latency: 64 blocks, a chain of four chunks).
constexpr int TX = 16, TY = 4, TZ = 4;
constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2, HV = HX * HY * HZ;

// What becomes of a convolution's output besides bias and ReLU.
struct ConvOut {
    const bf16 *gate = nullptr;  // output zeroed where not gate > 0 (the ReLU below a gradient)
    // split (up non-null): the output is the gradient of a concatenated input
    // whose first cup channels were up-sampled; those are summed over the 8
    // children of each coarse voxel into up (gated there by gate), the others
    // go to out, cout - cup channels wide
    bf16 *up = nullptr;
    int cup = 0;
};

// Place of weight (co, ci) within a tap in fragment order: the 16 x 32 weights
// of one B fragment as its lanes hold them, 8 channels a lane.  A fragment is
// then 1024 consecutive bytes; in [co][ci] order it is 16 pieces of 64 bytes,
// and fetching those held the layers of 32 and more channels back: 192 -> 64
// channels on 8 x 16^3 voxels 48 -> 30 us, 96 -> 32 on 8 x 32^3 58 -> 47, 128 ->
// 128 on 8 x 8^3 20 -> 14.
__device__ __forceinline__ size_t frag_place(int co, int ci, int cin) {
    return ((size_t)((co >> 4) * (cin >> 5) + (ci >> 5)) * 64 + (ci >> 3 & 3) * 16 + (co & 15)) * 8 + (ci & 7);
}

__device__ __forceinline__ bf16x8 gated(bf16x8 v, const bf16x8 &g) {
#pragma unroll
    for (int j = 0; j < 8; j++)
        if (!((float)g[j] > 0.f)) v[j] = (bf16)0.0f;
    return v;
}

// Blocks per CU that the tilings' registers have to leave room for.  A lane
// holds 16 NTC sums, 72 registers of voxels and 12 NTC of weights; with the
// weights a tap row ahead of the products and the staged pieces the compiler
// took 276 to 314 registers at NTC = 3 (HALF) and 4 and 201 at NTC = 2, which
// left one block on a CU, and two, where LDS allows three.  So the wide tilings
// of 32-channel chunks fetch a row's weights when its products come (NTC = 3 of
// whole chunks alone has room for both), and the bound keeps the rest of the
// schedule within 256 and 168 registers.  8 x 64^3 voxels: 32 -> 64 channels
// 467 -> 334 us, 48 -> 64 602 -> 411, 64 -> 64 1037 -> 870, 48 -> 48 489 -> 354;
// 64 maps of 64 x 1 x 64, 48 -> 64, 269 -> 170.
constexpr int conv_blocks(int ck, int ntc) { return ntc >= 3 ? 2 : ck == 32 && ntc == 2 ? 3 : 1; }

template <int CK, int NTC, bool HALF = false>
__global__ __launch_bounds__(NTH, conv_blocks(CK, NTC)) void k_conv_tile(const bf16 *__restrict__ ina, int ca, int upa,
                                                   const bf16 *__restrict__ inb, int cb, const bf16 *__restrict__ wt,
                                                   const float *__restrict__ bias, bf16 *__restrict__ out, int cout,
                                                   int relu, int D, int H, int W, int ntx, int nty, int ntz,
                                                   int nblk, ConvOut eo, int frag) {
    constexpr int CKP = CK == 16 ? CK : CK + 8;
    constexpr int MT = 4;
    constexpr bool AHEAD = NTC == 1 || (NTC == 3 && !HALF);
    static_assert(MT == TY && NTH / 64 == TZ && TX == 16, "a wave owns the 16 x 4 voxels of one tile plane");
    constexpr int UP = TX * TY * TZ * NTC * 16;  // up-sampled part of a split output, on its way to the sums
    __shared__ __attribute__((aligned(16))) bf16 tile[HV * CKP > UP ? HV * CKP : UP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    // the 8 XCDs take contiguous runs of tiles, so neighbouring halos share an L2
    int b = blockIdx.x;
    if ((nblk & 7) == 0) b = (b & 7) * (nblk >> 3) + (b >> 3);
    const int tx = b % ntx;
    int t = b / ntx;
    const int ty = t % nty;
    t /= nty;
    const int tz = t % ntz;
    const int n = t / ntz;
    const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
    const int co_base = blockIdx.y * NTC * 16;
    const int cin = ca + cb;
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1;
    f32x4 acc[MT][NTC];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int nt = 0; nt < NTC; nt++) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Staging: thread t copies the 16-byte piece `sub` of voxels t / SUB,
    // t / SUB + VPT, ... of the halo tile, its (row, x) stepped by VPT voxels
    // in mixed radix (no divisions in the loop).
    constexpr int SUB = CK / 8, VPT = NTH / SUB;
    const int sub = threadIdx.x % SUB, hv0 = threadIdx.x / SUB;
    // base pointers of the halo's 36 (z, y) source rows at x = 0, per input
    // (null outside the box), built once per block: an element's address is
    // then its row base plus x times the voxel stride
    __shared__ const bf16 *rowb[2][HZ * HY];
    if (threadIdx.x < 2 * HZ * HY) {
        const int src = threadIdx.x / (HZ * HY), r = threadIdx.x % (HZ * HY);
        const int gz = z0 - 1 + r / HY, gy = y0 - 1 + r % HY;
        const bf16 *bp = nullptr;
        if ((unsigned)gz < (unsigned)D && (unsigned)gy < (unsigned)H) {
            if (src == 0)
                bp = upa ? ina + ((((size_t)n * Dc + (gz >> 1)) * Hc + (gy >> 1)) * Wc) * ca
                         : ina + ((((size_t)n * D + gz) * H + gy) * W) * ca;
            else if (inb)
                bp = inb + ((((size_t)n * D + gz) * H + gy) * W) * cb;
        }
        rowb[src][r] = bp;
    }
    // this lane's voxel of its wave's fragment 0, displaced by tap (0, 0, 0):
    // fragment mt at tap (dz, dy, dx) lies ((dz HY + dy + mt) HX + dx) voxels on
    const bf16 *tb = tile + (wave * HY * HX + row) * CKP;
    // weights [tap][co][ci]: a uniform per-tap base and this lane's offset
    const size_t wtap = (size_t)cout * cin;
    for (int c0 = 0; c0 < cin; c0 += CK) {
        // Whole chunks of 32 channels: B fragments of a (dz, dy) row of taps are
        // fetched a row ahead, the first before the staging (AHEAD)
        const bool full = CK == 32 && (!HALF || cin - c0 >= 32);
        // byte offsets within a tap's weights (K entries c0 + 8 grp .. + 7; past the
        // last channel, where the voxels are zeros, the last ones again: what
        // follows them may be no number, or not be there at all)
        unsigned wl[NTC];
        const int cl = min(c0 + grp * 8, cin - 8);
#pragma unroll
        for (int nt = 0; nt < NTC; nt++)
            wl[nt] = frag ? (unsigned)((((co_base >> 4) + nt) * (cin >> 5) + (c0 >> 5)) * 1024 + lane * 16)
                          : (unsigned)(((co_base + nt * 16 + row) * cin + cl) * 2);
        bf16x8 bfr[AHEAD ? 2 : 1][3][NTC];
        const auto fetch = [&](int r) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const char *wb = (const char *)(wt + (r * 3 + dx) * wtap);  // uniform
#pragma unroll
                for (int nt = 0; nt < NTC; nt++) bfr[AHEAD ? r & 1 : 0][dx][nt] = *(const bf16x8 *)(wb + wl[nt]);
            }
        };
        if (AHEAD && full) fetch(0);
        __syncthreads();
        {
            const int c = c0 + sub * 8;  // this thread's 8 channels: all of a or all of b (8 | ca)
            const bool cok = c < cin, isa = c < ca;
            const int coff = isa ? c : c - ca, cs = isa ? ca : cb, sh = (isa && upa) ? 1 : 0;
            const bf16 *const *rb = rowb[isa ? 0 : 1];
            // voxel hv = row hr (z-major over (z, y)) x HX + hx, stepped by VPT.
            // Pieces outside the box load the tensor's first one and are zeroed,
            // so that no branch keeps the loads from being in flight together;
            // in the wide tilings of 32-channel chunks they are left out, which
            // costs nothing there and saves a flat map most of its loads (512
            // maps of 1 x 64, 96 -> 32: 90 -> 81 us).
            constexpr bool SKIP = CK == 32 && NTC > 1;
            constexpr int SDR = VPT / HX, SDX2 = VPT % HX, NK = (HV + VPT - 1) / VPT;
            int hx = hv0 % HX, hr = hv0 / HX;
            bf16x8 v[NK];
            bool ok[NK];
#pragma unroll
            for (int k = 0; k < NK; k++) {
                const int gx = x0 - 1 + hx;
                const bf16 *bp = rb[min(hr, HZ * HY - 1)];
                ok[k] = cok && bp && (unsigned)gx < (unsigned)W;
                // x < 2^24, channels < 2^24
                if constexpr (SKIP) {
                    v[k] = zero8();
                    if (ok[k]) v[k] = *(const bf16x8 *)(bp + (__umul24((unsigned)(gx >> sh), (unsigned)cs) + coff));
                } else {
                    v[k] = *(const bf16x8 *)(ok[k] ? bp + (__umul24((unsigned)(gx >> sh), (unsigned)cs) + coff) : ina);
                }
                hx += SDX2;
                hr += SDR;
                if (hx >= HX) {
                    hx -= HX;
                    hr++;
                }
            }
#pragma unroll
            for (int k = 0; k < NK; k++)
                if (hv0 + k * VPT < HV)
                    *(bf16x8 *)(tile + (hv0 + k * VPT) * CKP + sub * 8) = ok[k] ? v[k] : zero8();
        }
        __syncthreads();
        if (full) {
            // the A fragments of a tap plane's MT + 2 rows are read once for its
            // three dy (row mt + 1 of dy is row mt of dy + 1)
#pragma unroll
            for (int dz = 0; dz < 3; dz++) {
                bf16x8 afr[MT + 2][3];
#pragma unroll
                for (int r = 0; r < MT + 2; r++)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        afr[r][dx] = *(const bf16x8 *)(tb + ((dz * HY + r) * HX + dx) * CKP + grp * 8);
#pragma unroll
                for (int dy = 0; dy < 3; dy++) {
                    const int r = dz * 3 + dy;
                    if constexpr (!AHEAD) fetch(r);
                    else if (r < 8) fetch(r + 1);
                    // keep the loads ahead of the products (with HALF the registers
                    // that takes cost more: 153 against 171 us)
                    if constexpr (!HALF) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                        for (int mt = 0; mt < MT; mt++)
#pragma unroll
                            for (int nt = 0; nt < NTC; nt++)
                                acc[mt][nt] = mfma(bfr[AHEAD ? r & 1 : 0][dx][nt], afr[mt + dy][dx], acc[mt][nt]);
                }
            }
        } else if constexpr (CK == 16 || HALF) {
            // 16 channels per tap: one K step of 32 covers taps 2p (lane groups 0, 1) and 2p + 1 (2, 3)
            const int half = grp >> 1, cl = (grp & 1) * 8, cw = c0 + cl;
            const bool cok = cw < cin;
            unsigned wp[NTC];  // byte offsets within tap 2p's weights (this lane's tap is 2p + half)
#pragma unroll
            for (int nt = 0; nt < NTC; nt++)
                wp[nt] = (unsigned)((half * (int)wtap + (co_base + nt * 16 + row) * cin + cw) * 2);
            // tap 2p + 1 lies one voxel, one row less two or one plane less two
            // rows and two voxels beyond tap 2p: one base for each, so that all
            // fragment addresses are constants beyond it
            const bf16 *t1 = tb + cl + half * CKP, *t2 = tb + cl + half * (HX - 2) * CKP,
                       *t3 = tb + cl + half * ((HY - 2) * HX - 2) * CKP;
#pragma unroll
            for (int p = 0; p < 14; ++p) {
                const int ta = 2 * p;  // its second tap, 27, does not exist for p = 13: zeros
                const bf16 *base = ta % 3 < 2 ? t1 : ta % 9 < 8 ? t2 : t3;
                const int off = ((ta / 9 * HY + ta / 3 % 3) * HX + ta % 3) * CKP;
                const bool tok = cok && (p < 13 || !half);
                const char *wb = (const char *)(wt + ta * wtap);  // uniform
                bf16x8 bp[NTC];
#pragma unroll
                for (int nt = 0; nt < NTC; nt++) bp[nt] = tok ? *(const bf16x8 *)(wb + wp[nt]) : zero8();
#pragma unroll
                for (int mt = 0; mt < MT; mt++) {
                    bf16x8 afr = *(const bf16x8 *)((p < 13 ? base : tb + cl) + off + mt * HX * CKP);
                    if (p == 13 && half) afr = zero8();
#pragma unroll
                    for (int nt = 0; nt < NTC; nt++) acc[mt][nt] = mfma(bp[nt], afr, acc[mt][nt]);
                }
            }
        }
    }
    // lane l holds D[4 (l div 16) + r][l mod 16]: channel 4 grp + r of voxel x = row of row y = mt
    const int x = x0 + row, z = z0 + wave;
    const bool zx = z < D && x < W;
    const int cskip = cout - eo.cup;  // channels of out (eo.cup = 0 without a split)
    const bool vec = ((uintptr_t)out & 7) == 0;
    typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));
    if (eo.up) __syncthreads();  // the input tile becomes the up-sampled part
#pragma unroll
    for (int nt = 0; nt < NTC; nt++) {
        const int co = co_base + nt * 16 + grp * 4;
        float bv[4];
#pragma unroll
        for (int r = 0; r < 4; r++) bv[r] = bias ? bias[co + r] : 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const int y = y0 + mt;
            bf16x4v v;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                float val = acc[mt][nt][r] + bv[r];
                if (relu) val = fmaxf(val, 0.f);
                v[r] = (bf16)val;
            }
            if (co < eo.cup) {  // uniform: cup is a multiple of 16
                *(bf16x4v *)(tile + ((wave * TY + mt) * TX + row) * (NTC * 16) + nt * 16 + grp * 4) = v;
                continue;
            }
            if (!(zx && y < H)) continue;
            const size_t o = ((((size_t)n * D + z) * H + y) * W + x) * cskip + (co - eo.cup);
            if (eo.gate && !eo.up) {
                const bf16x4v g = *(const bf16x4v *)(eo.gate + o);
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (!((float)g[r] > 0.f)) v[r] = (bf16)0.0f;
            }
            if (vec) {
                *(bf16x4v *)(out + o) = v;
            } else {
#pragma unroll
                for (int r = 0; r < 4; r++) out[o + r] = v[r];
            }
        }
    }
    if (!eo.up || co_base >= eo.cup) return;
    __syncthreads();
    // coarse voxels of the tile (8 x 2 x 2), 8 channels a thread; children summed z, y, x-major
    const int nc8 = min(NTC * 16, eo.cup - co_base) >> 3;
    for (int e = threadIdx.x; e < (TX / 2) * (TY / 2) * (TZ / 2) * nc8; e += NTH) {
        const int c8 = e % nc8, q = e / nc8;
        const int cx = q % (TX / 2), cy = q / (TX / 2) % (TY / 2), cz = q / (TX / 2 * (TY / 2));
        const int X = (x0 >> 1) + cx, Y = (y0 >> 1) + cy, Z = (z0 >> 1) + cz;
        if (X >= Wc || Y >= Hc || Z >= Dc) continue;
        float sum[8];
#pragma unroll
        for (int j = 0; j < 8; j++) sum[j] = 0.f;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int vox = ((2 * cz + (k >> 2)) * TY + 2 * cy + ((k >> 1) & 1)) * TX + 2 * cx + (k & 1);
            const bf16x8 v = *(const bf16x8 *)(tile + vox * (NTC * 16) + c8 * 8);
#pragma unroll
            for (int j = 0; j < 8; j++) sum[j] += (float)v[j];
        }
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = (bf16)sum[j];
        const size_t o = ((((size_t)n * Dc + Z) * Hc + Y) * Wc + X) * eo.cup + co_base + c8 * 8;
        if (eo.gate) v = gated(v, *(const bf16x8 *)(eo.gate + o));
        *(bf16x8 *)(eo.up + o) = v;
    }
}

// -------------------------------------------------------------- conv bwd W
// dW[tap][co][ci] += sum_v dout[v][co] * X[v shifted by tap][ci] (X the
// possibly concatenated, possibly upsampled input), dbias[co] += sum_v dout:
// per tap a GEMM with M = co, N = ci, K = voxels.
//
// A block owns one 16 x 16 channel tile for all 27 taps and marches up z over
// a 16 x 16 column of voxels, two rows a wave.  Each plane of X (1-cell xy
// halo) and of dout is staged once in LDS, channels-last as it comes, with the
// global loads of the next two planes in flight.  The matrix operands need
// eight voxels of one channel per lane: LDS transpose reads
// (ds_read_b64_tr_b16) deliver four voxels of a row each, so one half-fragment
// covers the 16 voxels of a row (lane group g: voxels 4g .. 4g + 3) and a K
// step of 32 is the row pair (y, y + 1) of the wave.  A tap's x shift is an
// address, its y shift picks neighbouring half-fragments (row y + 1 of dy is
// row y of dy + 1), and its z shift one of the dout fragments of the last three
// planes, kept in registers: 12 transpose reads of X and two of dout feed 27
// matrix products.  The waves' sums meet in LDS and go to global FP32 with one
// atomic per weight and block; one address takes about 50 ns per atomic, so
// the sums of single waves (8 times as many) took most of a launch.
//
// Against the kernel per tap (below), which re-stages its input for every tap
// and transposes it element by element (8 x 64^3 voxels unless stated): 16 -> 16
// channels 1190 -> 46 us (134 MB read: 2.9 TB/s; 34 us of it the march, the
// rest the sums), 48 -> 16 2360 -> 114 us, 96 -> 32 on 8 x 32^3 600 -> 72 us
// (650 TFLOP/s), 64 -> 64 on 8 x 16^3 50 -> 18 us.  The fine resolutions are
// bound by the bytes staged, the coarse ones by the march's latency and the
// sums at the end.
// BW_T (nn_plan.h): voxels of a row, and rows of the column
constexpr int BW_H = BW_T + 2;           // ... with halo
constexpr int BW_G = 4;                  // taps reduced at a time (28 with the bias)
constexpr int BW_XN = 2 * BW_H * BW_H;   // 16-byte pieces (8 channels of a voxel) of an X plane
constexpr int BW_DN = 2 * BW_T * BW_T;   // ... of a dout plane: one per thread
static_assert(BW_NT == BW_DN && BW_XN <= 2 * BW_NT, "two X pieces and one dout piece per thread");
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Half-fragment of 16 consecutive voxels x 16 channels at p (LDS, 32 bytes a
// voxel): lane (g, i) receives channel i of voxels 4g .. 4g + 3.
__device__ __forceinline__ bf16x4 read_tr(const bf16 *p, int lane_off) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (__attribute__((address_space(3))) bf16x4 *)(const_cast<bf16 *>(p) + lane_off));
}

__device__ __forceinline__ bf16x8 join(const bf16x4 &a, const bf16x4 &b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct BwLds {
    union {
        struct {
            bf16 x[2][BW_XN * 8];
            bf16 d[2][BW_DN * 8];
        };
        float red[BW_NT / 64][BW_G * 256];
    };
};

// EDGE: the column may leave the box (W or H no multiple of 16; the masking costs a tenth)
template <bool EDGE>
__global__ __launch_bounds__(BW_NT, 2) void k_conv_bwd_w(const bf16 *__restrict__ dout, int cout,
                                                         const bf16 *__restrict__ ina, int ca, int upa,
                                                         const bf16 *__restrict__ inb, int cb, float *__restrict__ dw,
                                                         float *__restrict__ dbias, int D, int H, int W, int ntx,
                                                         int nty, int nzc, int zc) {
    __shared__ __attribute__((aligned(16))) BwLds lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = lane & 15, grp = lane >> 4;
    int b = blockIdx.x;
    const int tx = b % ntx;
    b /= ntx;
    const int ty = b % nty;
    b /= nty;
    const int zk = b % nzc, n = b / nzc;
    const int x0 = tx * BW_T, y0 = ty * BW_T, z0 = zk * zc, z1 = min(D, z0 + zc);
    const int cin = ca + cb, nci = cin >> 4;
    const int ci0 = ((int)blockIdx.y % nci) * 16, co0 = ((int)blockIdx.y / nci) * 16;
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1;

    // staging: a piece's place in its plane is fixed, only z moves.  Offsets in
    // a z plane of the piece's source (in pieces, -1: outside the box, read as
    // zero); the 8 channels of a piece come all from a or all from b (8 | ca)
    const bool fromb = ci0 + (tid & 1) * 8 >= ca;
    int xoff[2];
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const int p = tid + q * BW_NT;
        const int vx = (p >> 1) % BW_H, vy = (p >> 1) / BW_H;
        const int gx = x0 - 1 + vx, gy = y0 - 1 + vy, c = ci0 + (p & 1) * 8;
        xoff[q] = -1;
        if (p < BW_XN && (unsigned)gx < (unsigned)W && (unsigned)gy < (unsigned)H)
            xoff[q] = fromb ? (gy * W + gx) * (cb >> 3) + ((c - ca) >> 3)
                    : upa   ? ((gy >> 1) * Wc + (gx >> 1)) * (ca >> 3) + (c >> 3)
                            : (gy * W + gx) * (ca >> 3) + (c >> 3);
    }
    const int dx_ = x0 + (tid >> 1) % BW_T, dy_ = y0 + (tid >> 1) / BW_T;
    const int doff = dx_ < W && dy_ < H ? (dy_ * W + dx_) * (cout >> 3) + (co0 >> 3) + (tid & 1) : -1;
    const int xsh = !fromb && upa ? 1 : 0;
    const size_t xplane = fromb ? (size_t)H * W * cb : upa ? (size_t)Hc * Wc * ca : (size_t)H * W * ca;
    const bf16 *xbase = (fromb ? inb : ina) + (size_t)n * (xsh ? Dc : D) * xplane;
    const size_t dplane = (size_t)H * W * cout;
    const bf16 *dbase = dout + (size_t)n * D * dplane;
    struct Regs {
        bf16x8 x[2], d;
    };
    // X plane z and dout plane z + 1: every lane loads (pieces outside the box
    // from a clamped place) and keeps zero instead where it is outside, so the
    // loads of two steps stay in flight under exact wait counts
    auto fetch = [&](Regs &r, int z) {
        const bf16x8 *px = (const bf16x8 *)(xbase + (size_t)(min(max(z, 0), D - 1) >> xsh) * xplane);
        const bf16x8 *pd = (const bf16x8 *)(dbase + (size_t)min(z + 1, D - 1) * dplane);
#pragma unroll
        for (int q = 0; q < 2; q++) r.x[q] = px[max(xoff[q], 0)];
        r.d = pd[max(doff, 0)];
    };
    // the registers of X plane z -> LDS
    auto commit = [&](const Regs &r, int z, int buf) {
        const bool zin = z >= 0 && z < D, din = z + 1 < z1;  // uniform (z + 1 >= z0 always)
        *(bf16x8 *)(lds.x[buf] + tid * 8) = zin && xoff[0] >= 0 ? r.x[0] : zero8();
        if (tid + BW_NT < BW_XN) *(bf16x8 *)(lds.x[buf] + (tid + BW_NT) * 8) = zin && xoff[1] >= 0 ? r.x[1] : zero8();
        *(bf16x8 *)(lds.d[buf] + tid * 8) = din && doff >= 0 ? r.d : zero8();
    };
    f32x4 acc[27], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 27; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; j++) ones[j] = (bf16)1.0f;
    const bool bias = dbias && ci0 == 0;  // uniform
    // this lane's element of a half-fragment: voxel 4 grp + row / 4, channels 4 (row mod 4) ..
    const int loff = (grp * 4 + (row >> 2)) * 16 + (row & 3) * 4;
    // an X value takes part only where the dout voxel of its slot is in the box
    // (the zero staged there would turn an infinity into a NaN): 16 bits a
    // voxel, applied with EDGE
    u32x4 keep;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int x = x0 + grp * 4 + (j & 1) * 2, y = y0 + 2 * wave + (j >> 1);
        keep[j] = y < H ? (x < W ? 0xffffu : 0u) | (x + 1 < W ? 0xffff0000u : 0u) : 0u;
    }
    bf16x8 a[3];  // dout fragments of planes z - 1, z, z + 1 (slot: plane - z0 + 3 mod 3)
    a[0] = a[1] = a[2] = zero8();
    // step st: X plane z = z0 - 1 + st against dout planes z + 1 (dz = -1), z, z - 1,
    // those of the chunk
    const int nz = z1 - z0, nst = nz + 2;
    auto step = [&](int st, Regs &r, auto P) {
        constexpr int p = decltype(P)::value;  // st mod 3: slot of dout plane z + 1
        const int buf = st & 1;
        commit(r, z0 - 1 + st, buf);
        fetch(r, z0 + st + 1);  // (the last two go unused)
        __syncthreads();
        const bf16 *xp = lds.x[buf] + (2 * wave) * (BW_H * 16);
        const bf16 *dp = lds.d[buf] + (2 * wave) * (BW_T * 16);
        a[p] = join(read_tr(dp, loff), read_tr(dp + BW_T * 16, loff));
        if (bias) accb = mfma(a[p], ones, accb);
        bf16x4 h[4][3];  // [row y - 1 .. y + 2][dx]
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++)
#pragma unroll
            for (int dx = 0; dx < 3; dx++) h[r4][dx] = read_tr(xp + (r4 * BW_H + dx) * 16, loff);
        bf16x8 x[9];
#pragma unroll
        for (int t = 0; t < 9; t++) {
            x[t] = join(h[t / 3][t % 3], h[t / 3 + 1][t % 3]);
            if constexpr (EDGE) x[t] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, x[t]) & keep);
        }
#pragma unroll
        for (int dz = 0; dz < 3; dz++)
            if (st >= dz && st < dz + nz)  // uniform
#pragma unroll
                for (int t = 0; t < 9; t++) acc[dz * 9 + t] = mfma(a[(p + 3 - dz) % 3], x[t], acc[dz * 9 + t]);
    };
    Regs r0, r1;
    fetch(r0, z0 - 1);
    fetch(r1, z0);
#define BW_STEP(k, r, p) \
    if (st + k < nst) step(st + k, r, std::integral_constant<int, p>())
    for (int st = 0; st < nst; st += 6) {
        BW_STEP(0, r0, 0);
        BW_STEP(1, r1, 1);
        BW_STEP(2, r0, 2);
        BW_STEP(3, r1, 0);
        BW_STEP(4, r0, 1);
        BW_STEP(5, r1, 2);
    }
#undef BW_STEP
    // D[m = co][n = ci]: lane holds co = 4 grp + r, ci = row of the tile.  The
    // eight waves' sums of BW_G taps at a time meet in LDS (plain stores and
    // ordered sums: LDS float atomics took 60 us of a 100 us launch); the bias
    // sums (every column of the ones product holds them) go with the last taps
    constexpr int G = BW_G;
#pragma unroll
    for (int t0 = 0; t0 < 28; t0 += G) {
        __syncthreads();  // the last plane, or the group before, has been read
#pragma unroll
        for (int g = 0; g < G; g++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                lds.red[wave][g * 256 + (grp * 4 + r) * 16 + row] = t0 + g < 27 ? acc[t0 + g][r] : accb[r];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < G * 256 / BW_NT; k++) {
            const int e = tid + k * BW_NT, t = t0 + (e >> 8), co = (e >> 4) & 15, ci = e & 15;
            float v = lds.red[0][e];
#pragma unroll
            for (int w = 1; w < BW_NT / 64; w++) v += lds.red[w][e];
            if (t < 27) atomicAdd(&dw[((size_t)t * cout + co0 + co) * cin + ci0 + ci], v);
            else if (bias && ci == 0) atomicAdd(&dbias[co0 + co], v);
        }
    }
}

// The same gradient for few voxels, or maps much smaller than a column: a block
// takes one tap, 64 output channels (one 16-channel tile per wave) and a chunk
// of the voxels of all samples in a row; 32 voxels at a time are staged in LDS
// (dout rows and shifted input rows), then read back transposed element by
// element as MFMA fragments.  Its work follows the voxels, whatever the shape of
// the map, where the march pays for whole 16 x 16 columns and 27 tiles of atomics
// a block: 512 samples of 2^3 voxels, 64 -> 128 channels, 31 us here against 967,
// 256 of 4^3, 64 -> 64, 40 against 296, one of 64^2 x 1, 16 -> 16, 5 against 12.
// Large maps are the march's (line in per_tap).

template <int NCI>  // input-channel tiles of 16 (cin = 16 * NCI)
__global__ __launch_bounds__(NTH) void k_conv_bwd_w_tap(const bf16 *__restrict__ dout, int cout,
                                                     const bf16 *__restrict__ ina, int ca, int upa,
                                                     const bf16 *__restrict__ inb, int cb, float *__restrict__ dw,
                                                     float *__restrict__ dbias, int D, int H, int W, long long V,
                                                     int chunk) {
    __shared__ bf16 sd[BW_KV][64 + 8];       // dout rows (64 channels of this block), padded
    __shared__ bf16 sx[BW_KV][16 * NCI + 8]; // shifted input rows
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    const int tap = blockIdx.x;  // the 27 taps of one voxel chunk run side by side and share L2
    const int co_blk = blockIdx.z * 64;
    const int cin = 16 * NCI;
    const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1;
    const long long v0 = (long long)blockIdx.y * chunk;
    const long long v1 = v0 + chunk < V ? v0 + chunk : V;
    f32x4 acc[NCI];
#pragma unroll
    for (int t = 0; t < NCI; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    const bool wave_ok = co_blk + wave * 16 < cout;
    for (long long vb = v0; vb < v1; vb += BW_KV) {
        __syncthreads();
        // stage dout[vb .. vb+32)[co_blk .. co_blk+64) : 32 x 64 bf16, 8 per thread
        {
            const int e = threadIdx.x * 8;          // 256 threads x 8 = 2048 = 32 x 64
            const int vr = e / 64, c = e % 64;
            const long long v = vb + vr;
            bf16x8 val = zero8();
            if (v < v1 && co_blk + c < cout) val = *(const bf16x8 *)(dout + v * cout + co_blk + c);
#pragma unroll
            for (int j = 0; j < 8; j++) sd[vr][c + j] = val[j];
        }
        // stage X[v + tap shift][0 .. cin) : 32 x cin bf16, 8 per thread per pass
        for (int e = threadIdx.x * 8; e < BW_KV * cin; e += NTH * 8) {
            const int vr = e / cin, c = e % cin;
            const long long v = vb + vr;
            bf16x8 val = zero8();
            if (v < v1) {
                long long t = v;
                const int x = (int)(t % W) + dx;
                t /= W;
                const int y = (int)(t % H) + dy;
                t /= H;
                const int z = (int)(t % D) + dz;
                const int n = (int)(t / D);
                if (z >= 0 && z < D && y >= 0 && y < H && x >= 0 && x < W) {
                    if (c < ca) {
                        size_t vox;
                        if (upa) vox = (((size_t)n * Dc + (z >> 1)) * Hc + (y >> 1)) * Wc + (x >> 1);
                        else vox = (((size_t)n * D + z) * H + y) * W + x;
                        val = *(const bf16x8 *)(ina + vox * ca + c);
                    } else {
                        const size_t vox = (((size_t)n * D + z) * H + y) * W + x;
                        val = *(const bf16x8 *)(inb + vox * cb + (c - ca));
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; j++) sx[vr][c + j] = val[j];
        }
        __syncthreads();
        if (wave_ok) {
            // A[m = co][k = voxel]: lane takes co = row, voxels 8*grp .. 8*grp+7
            bf16x8 afr;
#pragma unroll
            for (int j = 0; j < 8; j++) afr[j] = sd[grp * 8 + j][wave * 16 + row];
            if (tap == 13 && dbias) {
#pragma unroll
                for (int j = 0; j < 8; j++) bsum += (float)afr[j];
            }
#pragma unroll
            for (int t = 0; t < NCI; t++) {
                bf16x8 bfr;  // B[k = voxel][n = ci]
#pragma unroll
                for (int j = 0; j < 8; j++) bfr[j] = sx[grp * 8 + j][t * 16 + row];
                acc[t] = mfma(afr, bfr, acc[t]);
            }
        }
    }
    if (!wave_ok) return;
    // D[m = co][n = ci]: lane holds co = 4*grp + r, ci = row
#pragma unroll
    for (int t = 0; t < NCI; t++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int co = co_blk + wave * 16 + grp * 4 + r;
            const int ci = t * 16 + row;
            if (co < cout) atomicAdd(&dw[((size_t)tap * cout + co) * cin + ci], acc[t][r]);
        }
    if (tap == 13 && dbias) {
        // lanes with the same row hold partial sums of channel co = row over different voxel groups
        bsum += __shfl_xor(bsum, 16);
        bsum += __shfl_xor(bsum, 32);
        if (grp == 0) atomicAdd(&dbias[co_blk + wave * 16 + row], bsum);
    }
}

// ----------------------------------------------------------- elementwise
// wt[26 - tap][ci][co] = w[tap][co][ci]: the backward-data convolution is the
// forward one with flipped taps and transposed channels.
__global__ void k_flip(const bf16 *__restrict__ w, bf16 *__restrict__ wt, int cout, int cin) {
    const long long n = 27LL * cout * cin;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const int ci = (int)(e % cin);
        const int co = (int)((e / cin) % cout);
        const int tap = (int)(e / ((long long)cin * cout));
        wt[((size_t)(26 - tap) * cin + ci) * cout + co] = w[e];
    }
}

// The weights as the network's convolutions read them, from w[tap][co][ci]:
// fwd (cin a multiple of 32) in fragment order, flip as k_flip's, in fragment
// order if cout is a multiple of 32.
__global__ void k_layout(const bf16 *__restrict__ w, bf16 *__restrict__ fwd, bf16 *__restrict__ flip, int cout,
                         int cin) {
    const int per = cout * cin, n = 27 * per;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int ci = e % cin, co = e / cin % cout, tap = e / per;
        if (cin % 32 == 0) fwd[(size_t)tap * per + frag_place(co, ci, cin)] = w[e];
        flip[(size_t)(26 - tap) * per + (cout % 32 == 0 ? frag_place(ci, co, cout) : (size_t)ci * cout + co)] = w[e];
    }
}

__global__ void k_relu_bwd(bf16 *__restrict__ dy, const bf16 *__restrict__ y, long long n) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
        if (!((float)y[e] > 0.f)) dy[e] = (bf16)0.0f;
}

// 2x average pooling of a (N, D, H, W, C) tensor into (N, D/2, H/2, W/2, C),
// VEC channels of a voxel per thread.
template <int VEC>
__global__ void k_pool(const bf16 *__restrict__ in, bf16 *__restrict__ out, int C, int N, int D, int H, int W) {
    typedef __bf16 vec __attribute__((ext_vector_type(VEC)));
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1, G = C / VEC;
    const long long n = (long long)N * Dc * Hc * Wc * G;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const int c = (int)(e % G) * VEC;
        long long t = e / G;
        const int x = (int)(t % Wc);
        t /= Wc;
        const int y = (int)(t % Hc);
        t /= Hc;
        const int z = (int)(t % Dc);
        const int b = (int)(t / Dc);
        float s[VEC];
#pragma unroll
        for (int j = 0; j < VEC; j++) s[j] = 0.f;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const size_t vox = (((size_t)b * D + 2 * z + (q >> 2)) * H + 2 * y + ((q >> 1) & 1)) * W + 2 * x + (q & 1);
            const vec v = *(const vec *)(in + vox * C + c);
#pragma unroll
            for (int j = 0; j < VEC; j++) s[j] += (float)v[j];
        }
        vec o;
#pragma unroll
        for (int j = 0; j < VEC; j++) o[j] = (bf16)(0.125f * s[j]);
        *(vec *)(out + e * VEC) = o;
    }
}

// Gradient of the pooling: din[fine] += dout[parent] / 8; with a gate, din is
// then zeroed where not gate > 0.  VEC channels of a voxel per thread.
template <int VEC>
__global__ void k_pool_bwd(const bf16 *__restrict__ dout, bf16 *__restrict__ din, const bf16 *__restrict__ gate, int C,
                           int N, int D, int H, int W) {
    typedef __bf16 vec __attribute__((ext_vector_type(VEC)));
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1, G = C / VEC;
    const long long n = (long long)N * D * H * W * G;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const int c = (int)(e % G) * VEC;
        long long t = e / G;
        const int x = (int)(t % W);
        t /= W;
        const int y = (int)(t % H);
        t /= H;
        const int z = (int)(t % D);
        const int b = (int)(t / D);
        const size_t p = (((size_t)b * Dc + (z >> 1)) * Hc + (y >> 1)) * Wc + (x >> 1);
        vec v = *(vec *)(din + e * VEC);
        const vec g = *(const vec *)(dout + p * C + c);
#pragma unroll
        for (int j = 0; j < VEC; j++) v[j] = (bf16)((float)v[j] + 0.125f * (float)g[j]);
        if (gate) {
            const vec q = *(const vec *)(gate + e * VEC);
#pragma unroll
            for (int j = 0; j < VEC; j++)
                if (!((float)q[j] > 0.f)) v[j] = (bf16)0.0f;
        }
        *(vec *)(din + e * VEC) = v;
    }
}

// Split the gradient of a concatenated, partly upsampled input:
// dup[coarse][c] = sum over its 8 fine children of dx[fine][c] (c < ca), and
// dskip[fine][c - ca] = dx[fine][c] (c >= ca; the pooling path adds its share later).
// gate (may be null): dup is zeroed where not gate > 0.
__global__ void k_split_grad(const bf16 *__restrict__ dx, int ca, int cb, bf16 *__restrict__ dup,
                             bf16 *__restrict__ dskip, const bf16 *__restrict__ gate, int N, int D, int H, int W) {
    const int cin = ca + cb;
    const int Dc = D >> 1, Hc = H >> 1, Wc = W >> 1;
    const long long nc = (long long)N * Dc * Hc * Wc * ca;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nc; e += (long long)gridDim.x * blockDim.x) {
        const int c = (int)(e % ca);
        long long t = e / ca;
        const int x = (int)(t % Wc);
        t /= Wc;
        const int y = (int)(t % Hc);
        t /= Hc;
        const int z = (int)(t % Dc);
        const int b = (int)(t / Dc);
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const size_t vox = (((size_t)b * D + 2 * z + (q >> 2)) * H + 2 * y + ((q >> 1) & 1)) * W + 2 * x + (q & 1);
            s += (float)dx[vox * cin + c];
        }
        dup[e] = !gate || (float)gate[e] > 0.f ? (bf16)s : (bf16)0.0f;
    }
    if (!dskip) return;
    const long long nf = (long long)N * D * H * W * cb;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nf; e += (long long)gridDim.x * blockDim.x) {
        const int c = (int)(e % cb);
        const long long v = e / cb;
        dskip[e] = dx[v * cin + ca + c];
    }
}

// Per-sample sums over active cells: stats[2n] = sum rho^2, stats[2n+1] =
// active count (both start at zero).
__global__ void k_stats(const double *__restrict__ rho, const int8_t *__restrict__ mask, long long vs,
                        double *__restrict__ stats) {
    __shared__ double s_a[NTH / 64], s_c[NTH / 64];
    const int n = blockIdx.y;
    double a = 0.0, c = 0.0;
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < vs; v += (long long)gridDim.x * blockDim.x) {
        const long long e = n * vs + v;
        if (mask[e] == 1) {
            a += rho[e] * rho[e];
            c += 1.0;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        c += __shfl_xor(c, o);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        s_a[wv] = a;
        s_c[wv] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < NTH / 64; q++) {
            a += s_a[q];
            c += s_c[q];
        }
        atomicAdd(&stats[2 * n], a);
        atomicAdd(&stats[2 * n + 1], c);
    }
}

// Input scale of sample n: root mean square of rho over its active cells (1 if zero).
__device__ __forceinline__ double sample_scale(const double *stats, int n) {
    const double c = stats[2 * n + 1];
    const double s = c > 0.0 ? sqrt(stats[2 * n] / c) : 0.0;
    return s > 0.0 ? s : 1.0;
}

// Network input, 16 channels per voxel: rho on active cells / s, the mask, B / s, zeros.
__global__ void k_pack(const double *__restrict__ rho, const int8_t *__restrict__ mask, const double *__restrict__ B,
                       const double *__restrict__ stats, long long vs, long long total, bf16 *__restrict__ x) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        const double is = 1.0 / sample_scale(stats, (int)(e / vs));
        const bool act = mask[e] == 1;
        bf16x8 a = zero8(), b = zero8();
        a[0] = (bf16)(float)(act ? (0.0 + rho[e]) * is : 0.0);  // sums of one term: -0 becomes 0
        a[1] = (bf16)(act ? 1.0f : -1.0f);
        a[2] = (bf16)(float)((B ? 0.0 + B[e] : 0.0) * is);
        *(bf16x8 *)(x + e * 16) = a;
        *(bf16x8 *)(x + e * 16 + 8) = b;
    }
}

// Network input at 1/S resolution: mean of rho over the active fine cells of
// the block / s, +1 if more than half of the block is active (else -1), mean
// of B over the block / s, zeros.
// One sample, in one pass over the fine fields: each
// thread forms its coarse cell's sums, which wait in
// `sums` (3 per cell: of rho, of B, the active count) for the scale, and each
// block its share of k_stats' sums.  Reading rho twice and 8192 atomics on one
// line of memory took 107 + 38 us at 256^3 and S = 4; this 17 + 9 us
// (17 MB of mask and the active third of 134 MB of rho).  VEC: rows of a cell are read as 16-byte pieces and
// mask words (alignment permitting); a row with no active cell reads rho's
// first piece instead of its own.
template <int S, bool VEC>
__global__ __launch_bounds__(NTH) void k_pack_sums(const double *__restrict__ rho, const int8_t *__restrict__ mask,
                                                   const double *__restrict__ B, int Dc, int Hc, int Wc,
                                                   double *__restrict__ sums, double *__restrict__ part) {
    __shared__ double s_a[NTH / 64], s_c[NTH / 64];
    typedef double d2 __attribute__((ext_vector_type(2)));
    constexpr int P = S < 4 ? 2 : 4;  // cells of a mask word
    using word = typename std::conditional<P == 2, uint16_t, uint32_t>::type;
    const int V = Dc * Hc * Wc;
    const size_t W = (size_t)Wc * S, H = (size_t)Hc * S;
    double a = 0.0, c = 0.0;
    const int e = blockIdx.x * NTH + threadIdx.x;
    if (e < V) {
        const int cx = e % Wc, cy = e / Wc % Hc, cz = e / Wc / Hc;
        double rs = 0.0, bs = 0.0;
        int cnt = 0;
#pragma unroll 1
        for (int dz = 0; dz < S; dz++) {
            const size_t f0 = ((size_t)(cz * S + dz) * H + (size_t)cy * S) * W + (size_t)cx * S;
            double r[S][S];
            bool m[S][S];
            if constexpr (VEC) {
                word mw[S][S / P];
#pragma unroll
                for (int dy = 0; dy < S; dy++)
#pragma unroll
                    for (int q = 0; q < S / P; q++) mw[dy][q] = *(const word *)(mask + f0 + dy * W + q * P);
#pragma unroll
                for (int dy = 0; dy < S; dy++) {
                    bool any = false;
#pragma unroll
                    for (int dx = 0; dx < S; dx++) any |= (m[dy][dx] = ((mw[dy][dx / P] >> (8 * (dx % P))) & 255) == 1);
#pragma unroll
                    for (int q = 0; q < S / 2; q++) {
                        const d2 v = *(const d2 *)(any ? rho + f0 + dy * W + 2 * q : rho);
                        r[dy][2 * q] = v[0];
                        r[dy][2 * q + 1] = v[1];
                    }
                }
            } else {
#pragma unroll
                for (int dy = 0; dy < S; dy++)
#pragma unroll
                    for (int dx = 0; dx < S; dx++) {
                        m[dy][dx] = mask[f0 + dy * W + dx] == 1;
                        r[dy][dx] = rho[f0 + dy * W + dx];
                    }
            }
#pragma unroll
            for (int dy = 0; dy < S; dy++)
#pragma unroll
                for (int dx = 0; dx < S; dx++)
                    if (m[dy][dx]) {
                        rs += r[dy][dx];
                        a += r[dy][dx] * r[dy][dx];
                        cnt++;
                    }
            if (B)
#pragma unroll
                for (int dy = 0; dy < S; dy++)
#pragma unroll
                    for (int dx = 0; dx < S; dx++) bs += B[f0 + dy * W + dx];
        }
        sums[e] = rs;
        sums[(size_t)V + e] = bs;
        sums[2 * (size_t)V + e] = (double)cnt;
        c = (double)cnt;
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        c += __shfl_xor(c, o);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        s_a[wv] = a;
        s_c[wv] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < NTH / 64; q++) {
            a += s_a[q];
            c += s_c[q];
        }
        part[2 * blockIdx.x] = a;
        part[2 * blockIdx.x + 1] = c;
    }
}

// One block: stats[0], stats[1] from the np partial sums, in a fixed order.
__global__ __launch_bounds__(1024) void k_stats_sum(const double *__restrict__ part, int np,
                                                    double *__restrict__ stats) {
    __shared__ double sa[16], sc[16];
    double a = 0.0, c = 0.0;
    for (int q = threadIdx.x; q < np; q += 1024) {
        a += part[2 * q];
        c += part[2 * q + 1];
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        c += __shfl_xor(c, o);
    }
    if ((threadIdx.x & 63) == 0) {
        sa[threadIdx.x >> 6] = a;
        sc[threadIdx.x >> 6] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < 16; q++) {
            a += sa[q];
            c += sc[q];
        }
        stats[0] = a;
        stats[1] = c;
    }
}

__global__ __launch_bounds__(NTH) void k_pack_scale(const double *__restrict__ sums, const double *__restrict__ stats,
                                                    int S3, int V, bf16 *__restrict__ x) {
    const int e = blockIdx.x * NTH + threadIdx.x;
    if (e >= V) return;
    const double is = 1.0 / sample_scale(stats, 0), rs = sums[e], bs = sums[(size_t)V + e];
    const int cnt = (int)sums[2 * (size_t)V + e];
    bf16x8 a = zero8(), b = zero8();
    a[0] = (bf16)(float)(cnt > 0 ? rs / cnt * is : 0.0);
    a[1] = (bf16)(2 * cnt > S3 ? 1.0f : -1.0f);
    a[2] = (bf16)(float)(bs / S3 * is);
    *(bf16x8 *)(x + (size_t)e * 16) = a;
    *(bf16x8 *)(x + (size_t)e * 16 + 8) = b;
}

// Head: phi[v] = s_n / 256 * (sum_c w[c] x[v][c] + b), zero where a mask is
// given and the cell is inactive.
__global__ void k_head(const bf16 *__restrict__ x, const float *__restrict__ w, const float *__restrict__ b,
                       const double *__restrict__ stats, const int8_t *__restrict__ mask, double *__restrict__ phi,
                       long long vs, int N) {
    const long long V = vs * N;
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
        float s = b[0];
#pragma unroll
        for (int c = 0; c < 16; c++) s += w[c] * (float)x[v * 16 + c];
        const double sc = sample_scale(stats, (int)(v / vs)) * (1.0 / 256.0);
        phi[v] = (mask == nullptr || mask[v] == 1) ? sc * (double)s : 0.0;
    }
}

// Linear up-sampling of a cell-centred field by 2 per axis: 3/4 of the
// parent plus 1/4 of the next coarse cell on the child's side (the edge cell
// repeated past the array end); zero on inactive cells when a mask is given.
// A thread forms the two z and y children and one x pair of a coarse cell from
// its 27 neighbours and stores pairs (16 bytes with VEC): one thread per child,
// with 64-bit index divisions and 8 loads for one store, took 66 us for
// 128^3 -> 256^3, this 40 us (168 MB).  A block takes `per` coarse planes that
// fit it side by side (one where a plane fills it): 100000 planes of 3 x 3 took
// 112 us with one plane a block, 38 with a thread per child, 23 so.
template <bool VEC>
__global__ __launch_bounds__(NTH) void k_up2(const double *__restrict__ c, double *__restrict__ f, int Dc, int Hc,
                                             int Wc, int per, const int8_t *__restrict__ mask) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    const unsigned pl = (unsigned)Hc * (unsigned)Wc;     // (2^32 of them would not fit the device)
    const int q0 = per > 1 ? (int)(threadIdx.x / pl) : 0;  // plane of the block's
    const unsigned e = blockIdx.x * NTH + threadIdx.x - q0 * pl;  // row (y) and x of a coarse plane
    if (q0 >= per || e >= pl) return;
    const int py = (int)(e / (unsigned)Wc), px = (int)(e - (unsigned)py * Wc);
    const size_t base = (size_t)blockIdx.z * Dc * Hc * Wc, cpl = (size_t)Hc * Wc;
    const size_t H = 2 * (size_t)Hc, W = 2 * (size_t)Wc;
    for (int pz = (int)blockIdx.y * per + q0; pz < Dc; pz += (int)gridDim.y * per) {
        const size_t f0 = (((size_t)blockIdx.z * 2 * Dc + 2 * pz) * H + 2 * py) * W + 2 * px;
        bool act[2][2][2];
        bool any = false;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const size_t o = f0 + ((q >> 1) * H + (q & 1)) * W;
#pragma unroll
            for (int dx = 0; dx < 2; dx++) any |= (act[q >> 1][q & 1][dx] = !mask || mask[o + dx] == 1);
        }
        const auto mix = [](double near, double far) { return __builtin_fma(0.75, near, 0.25 * far); };
        const auto put = [&](int dz, int dy, double v0, double v1) {
            const size_t o = f0 + (dz * H + dy) * W;
            v0 = act[dz][dy][0] ? v0 : 0.0;
            v1 = act[dz][dy][1] ? v1 : 0.0;
            if constexpr (VEC) {
                *(d2 *)(f + o) = d2{v0, v1};
            } else {
                f[o] = v0;
                f[o + 1] = v1;
            }
        };
        if (!any) {
#pragma unroll
            for (int q = 0; q < 4; q++) put(q >> 1, q & 1, 0.0, 0.0);
            continue;
        }
        double v[3][3][3];
#pragma unroll
        for (int k = 0; k < 27; k++) {
            const int z = min(max(pz + k / 9 - 1, 0), Dc - 1), y = min(max(py + k / 3 % 3 - 1, 0), Hc - 1),
                      x = min(max(px + k % 3 - 1, 0), Wc - 1);
            v[k / 9][k / 3 % 3][k % 3] = c[base + z * cpl + (size_t)y * Wc + x];
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            double r[2];
#pragma unroll
            for (int dx = 0; dx < 2; dx++) {
                const int qz = (q >> 1) ? 2 : 0, qy = (q & 1) ? 2 : 0, qx = dx ? 2 : 0;
                r[dx] = mix(mix(mix(v[1][1][1], v[1][1][qx]), mix(v[1][qy][1], v[1][qy][qx])),
                            mix(mix(v[qz][1][1], v[qz][1][qx]), mix(v[qz][qy][1], v[qz][qy][qx])));
            }
            put(q >> 1, q & 1, r[0], r[1]);
        }
    }
}

// Coarse copy of a problem for a first guess: the mask keeps a block active
// when more than half of its S^3 cells are active (the outermost coarse layer
// is always inactive), rho is the mean over the active cells of the block and
// B the mean over the block.
__global__ void k_coarsen(const double *__restrict__ rho, const int8_t *__restrict__ mask, const double *__restrict__ B,
                          int S, int Dc, int Hc, int Wc, double *__restrict__ rho_c, int8_t *__restrict__ mask_c,
                          double *__restrict__ B_c) {
    const long long total = (long long)Dc * Hc * Wc;
    const int W = Wc * S, H = Hc * S;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        long long t = e;
        const int cx = (int)(t % Wc);
        t /= Wc;
        const int cy = (int)(t % Hc);
        const int cz = (int)(t / Hc);
        double rs = 0.0, bs = 0.0;
        int cnt = 0;
        for (int dz = 0; dz < S; dz++)
            for (int dy = 0; dy < S; dy++)
                for (int dx = 0; dx < S; dx++) {
                    const size_t f = ((size_t)(cz * S + dz) * H + cy * S + dy) * W + cx * S + dx;
                    if (mask[f] == 1) {
                        rs += rho[f];
                        cnt++;
                    }
                    if (B) bs += B[f];
                }
        const int S3 = S * S * S;
        const bool frame = cx == 0 || cy == 0 || cz == 0 || cx == Wc - 1 || cy == Hc - 1 || cz == Dc - 1;
        mask_c[e] = (!frame && 2 * cnt > S3) ? 1 : -1;
        rho_c[e] = cnt > 0 ? rs / cnt : 0.0;
        if (B_c) B_c[e] = bs / S3;
    }
}

// Loss = mean over the active cells of the batch of (y - t)^2, with y the
// head output and t = 256 target / s_n.  Writes dx (bf16; zero where x, a
// ReLU's output, is not positive), accumulates the
// head's weight and bias gradients and the loss.
// One block of 1024 threads per CU: the 18 sums take an atomic per block on one
// line of memory, and with 1024 blocks of 256 those took half of the launch
// (8 x 64^3: 50 us, now 43, for 153 MB).
constexpr int HL_NT = 1024;
__global__ __launch_bounds__(HL_NT) void k_head_loss(const bf16 *__restrict__ x, const float *__restrict__ w, const float *__restrict__ b,
                            const int8_t *__restrict__ mask, const double *__restrict__ target,
                            const double *__restrict__ stats, int N, long long vs, bf16 *__restrict__ dx,
                            float *__restrict__ dw, float *__restrict__ db, double *__restrict__ loss) {
    __shared__ float s_dw[HL_NT / 64][17];
    __shared__ double s_l[HL_NT / 64];
    double count = 0.0;
    for (int n = 0; n < N; n++) count += stats[2 * n + 1];
    const double inv_count = count > 0.0 ? 1.0 / count : 0.0;
    float ldw[17];
#pragma unroll
    for (int c = 0; c < 17; c++) ldw[c] = 0.f;
    double lsum = 0.0;
    const long long V = vs * N;
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
        float xv[16];
        float y = b[0];
#pragma unroll
        for (int c = 0; c < 16; c++) {
            xv[c] = (float)x[v * 16 + c];
            y += w[c] * xv[c];
        }
        float g = 0.f;
        if (mask[v] == 1) {
            const double t = target[v] * 256.0 / sample_scale(stats, (int)(v / vs));
            const double d = (double)y - t;
            lsum += d * d;
            g = (float)(2.0 * d * inv_count);
        }
        bf16x8 lo, hi;
#pragma unroll
        for (int c = 0; c < 8; c++) {
            lo[c] = xv[c] > 0.f ? (bf16)(g * w[c]) : (bf16)0.0f;
            hi[c] = xv[c + 8] > 0.f ? (bf16)(g * w[c + 8]) : (bf16)0.0f;
        }
        *(bf16x8 *)(dx + v * 16) = lo;
        *(bf16x8 *)(dx + v * 16 + 8) = hi;
#pragma unroll
        for (int c = 0; c < 16; c++) ldw[c] += g * xv[c];
        ldw[16] += g;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 17; c++) {
        float t = ldw[c];
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
        if (lane == 0) s_dw[wv][c] = t;
    }
    double lt = lsum;
    for (int o = 32; o > 0; o >>= 1) lt += __shfl_xor(lt, o);
    if (lane == 0) s_l[wv] = lt;
    __syncthreads();
    if (threadIdx.x < 17) {
        float t = 0.f;
        for (int q = 0; q < HL_NT / 64; q++) t += s_dw[q][threadIdx.x];
        if (threadIdx.x < 16) atomicAdd(&dw[threadIdx.x], t);
        else atomicAdd(db, t);
    }
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < HL_NT / 64; q++) t += s_l[q];
        atomicAdd(loss, t * inv_count);
    }
}

__global__ void k_fill_f32(float *__restrict__ p, long long n) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
        p[e] = 0.f;
}

__global__ void k_fill_f64(double *__restrict__ p, long long n) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
        p[e] = 0.0;
}

// AdamW on FP32 master weights, refreshing the BF16 copy (decoupled decay).
__global__ void k_adamw(float *__restrict__ p, bf16 *__restrict__ pb, const float *__restrict__ g, float *__restrict__ m,
                        float *__restrict__ v, long long n, float lr, float b1, float b2, float eps, float wd,
                        float c1, float c2) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const float gg = g[e];
        const float mm = b1 * m[e] + (1.f - b1) * gg;
        const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
        m[e] = mm;
        v[e] = vv;
        float w = p[e] * (1.f - lr * wd);
        w -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
        p[e] = w;
        if (pb) pb[e] = (bf16)w;
    }
}

// 16 x 16 x 32 self-test of the operand and result lane layouts with small
// integers (exact in BF16 and FP32): a[m][k] = (3m + k) mod 7 - 3,
// b[k][n] = (5k + 2n) mod 9 - 4, out[m][n] = sum_k a[m][k] b[k][n].
__global__ void k_mfma_selftest(float *out) {
    const int lane = threadIdx.x, row = lane & 15, grp = lane >> 4;
    bf16x8 a, b;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int k = grp * 8 + j;
        a[j] = (bf16)(float)((3 * row + k) % 7 - 3);
        b[j] = (bf16)(float)((5 * k + 2 * row) % 9 - 4);
    }
    f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
    c = mfma(a, b, c);
#pragma unroll
    for (int r = 0; r < 4; r++) out[(grp * 4 + r) * 16 + row] = c[r];
}

inline unsigned blocks_for(long long n, int per = 256) {
    long long g = (n + per - 1) / per;
    if (g > 16384) g = 16384;
    return (unsigned)(g > 0 ? g : 1);
}

template <int NCI>
void launch_bww_tap(const bf16 *dout, int cout, const bf16 *ina, int ca, int upa, const bf16 *inb, int cb, float *dw,
                    float *db, int D, int H, int W, long long V, hipStream_t s) {
    const int groups = (cout + 63) / 64;
    const long long chunk = tap_chunk(V, groups);
    dim3 grid(27, (unsigned)((V + chunk - 1) / chunk), (unsigned)groups);
    k_conv_bwd_w_tap<NCI><<<grid, NTH, 0, s>>>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, (int)chunk);
}

void launch_bww(const bf16 *dout, int cout, const bf16 *ina, int ca, int upa, const bf16 *inb, int cb, float *dw,
                float *db, int n, int D, int H, int W, hipStream_t s) {
    const long long V = (long long)n * D * H * W;
    const MarchPlan m = march_plan(n, D, H, W, ca + cb, cout);
    if (per_tap(m, ca + cb, cout, V, H, W)) {
        switch ((ca + cb) / 16) {
            case 1: launch_bww_tap<1>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            case 2: launch_bww_tap<2>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            case 3: launch_bww_tap<3>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            case 4: launch_bww_tap<4>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            case 6: launch_bww_tap<6>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            case 8: launch_bww_tap<8>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
            default: launch_bww_tap<12>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, V, s); break;
        }
        return;
    }
    dim3 grid((unsigned)(m.cols * m.nzc), (unsigned)m.tiles);
    if (W % BW_T || H % BW_T)
        k_conv_bwd_w<true><<<grid, BW_NT, 0, s>>>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, m.ntx, m.nty,
                                                  m.nzc, m.zc);
    else
        k_conv_bwd_w<false><<<grid, BW_NT, 0, s>>>(dout, cout, ina, ca, upa, inb, cb, dw, db, D, H, W, m.ntx, m.nty,
                                                   m.nzc, m.zc);
}

// ------------------------------------------------ host launchers (nn_core.h)
static bool dims_ok(int n, int d, int h, int w) { return n > 0 && d > 0 && h > 0 && w > 0; }

template <int CK, int NTC>
void launch_tile(const bf16 *ina, int ca, int upa, const bf16 *inb, int cb, const bf16 *w, const float *bias, bf16 *out,
                 int cout, int relu, const ConvOut &eo, int n, int D, int H, int W, hipStream_t s, int frag) {
    const int ntx = (W + TX - 1) / TX, nty = (H + TY - 1) / TY, ntz = (D + TZ - 1) / TZ;
    const int nblk = n * ntx * nty * ntz;
    dim3 grid((unsigned)nblk, (unsigned)(cout / (16 * NTC)));
    if constexpr (CK == 32) {
        if ((ca + cb) % 32 == 16) {
            k_conv_tile<CK, NTC, true><<<grid, NTH, 0, s>>>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, D, H, W,
                                                            ntx, nty, ntz, nblk, eo, 0);
            return;
        }
    }
    k_conv_tile<CK, NTC><<<grid, NTH, 0, s>>>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, D, H, W, ntx, nty, ntz,
                                              nblk, eo, frag);
}

template <int CK>
void launch_tile_ck(const bf16 *ina, int ca, int upa, const bf16 *inb, int cb, const bf16 *w, const float *bias,
                    bf16 *out, int cout, int relu, const ConvOut &eo, int n, int D, int H, int W, hipStream_t s,
                    int frag) {
    // widest output tiling that still gives about 1024 blocks
    const long long nblk = (long long)n * ((W + TX - 1) / TX) * ((H + TY - 1) / TY) * ((D + TZ - 1) / TZ);
    const int tiles = cout / 16;
    int ntc = 4;
    while (ntc > 1 && (tiles % ntc || nblk * (tiles / ntc) < 1024)) ntc--;
    if (ntc == 4) launch_tile<CK, 4>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, eo, n, D, H, W, s, frag);
    else if (ntc == 3) launch_tile<CK, 3>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, eo, n, D, H, W, s, frag);
    else if (ntc == 2) launch_tile<CK, 2>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, eo, n, D, H, W, s, frag);
    else launch_tile<CK, 1>(ina, ca, upa, inb, cb, w, bias, out, cout, relu, eo, n, D, H, W, s, frag);
}

static bool conv_run(const void *in_a, int ca, int up_a, const void *in_b, int cb, const void *w, const float *bias,
                     void *out, int cout, int relu, const ConvOut &eo, int n, int d, int h, int wd, hipStream_t s,
                     bool frag) {
    if (!in_a || !w || !out || ca <= 0 || cb < 0 || (cb > 0 && !in_b) || ca % 8 || cb % 8 || cout <= 0 ||
        cout % 16 || !dims_ok(n, d, h, wd) || (up_a && (d % 2 || h % 2 || wd % 2))) {
        set_error("conv3d: invalid arguments (input channels multiples of 8, output channels of 16)");
        return false;
    }
    const bf16 *A = (const bf16 *)in_a, *B = (const bf16 *)in_b, *W = (const bf16 *)w;
    bf16 *O = (bf16 *)out;
    if (frag && (ca + cb) % 32) {
        set_error("conv3d: weights in fragment order need input channels in multiples of 32");
        return false;
    }
    if (ca + cb <= 16) launch_tile_ck<16>(A, ca, up_a, B, cb, W, bias, O, cout, relu, eo, n, d, h, wd, s, 0);
    else launch_tile_ck<32>(A, ca, up_a, B, cb, W, bias, O, cout, relu, eo, n, d, h, wd, s, frag ? 1 : 0);
    return hip_ok(hipGetLastError(), "conv3d launch");
}

bool conv_fwd(const void *in_a, int ca, int up_a, const void *in_b, int cb, const void *w, const float *bias,
              void *out, int cout, int relu, int n, int d, int h, int wd, hipStream_t s, bool frag) {
    return conv_run(in_a, ca, up_a, in_b, cb, w, bias, out, cout, relu, ConvOut{}, n, d, h, wd, s, frag);
}

bool conv_grad(const void *dout, int cout, const void *wf, const void *gate, void *dx, int cin, int n, int d, int h,
               int wd, hipStream_t s) {
    ConvOut eo;
    eo.gate = (const bf16 *)gate;
    return conv_run(dout, cout, 0, nullptr, 0, wf, nullptr, dx, cin, 0, eo, n, d, h, wd, s, cout % 32 == 0);
}

bool conv_grad_split(const void *dout, int cout, const void *wf, int ca, int cb, const void *gate, void *dup,
                     void *dskip, int n, int d, int h, int wd, hipStream_t s) {
    if (!dup || !dskip || ca % 16 || cb % 16 || d % 2 || h % 2 || wd % 2) {
        set_error("conv3d split gradient: invalid arguments");
        return false;
    }
    ConvOut eo;
    eo.gate = (const bf16 *)gate;
    eo.up = (bf16 *)dup;
    eo.cup = ca;
    return conv_run(dout, cout, 0, nullptr, 0, wf, nullptr, dskip, ca + cb, 0, eo, n, d, h, wd, s, cout % 32 == 0);
}

bool conv_bwd_weight(const void *dout, int cout, const void *in_a, int ca, int up_a, const void *in_b, int cb,
                     float *dw, float *dbias, int n, int d, int h, int wd, hipStream_t s) {
    const int cin = ca + cb;
    if (!dout || !in_a || !dw || cout <= 0 || cout % 16 || ca <= 0 || ca % 8 || cb < 0 || cb % 8 ||
        (cb > 0 && !in_b) || cin % 16 || !dims_ok(n, d, h, wd) || (up_a && (d % 2 || h % 2 || wd % 2))) {
        set_error("conv3d weight gradient: invalid arguments (input channels a multiple of 16, output of 16)");
        return false;
    }
    const bf16 *G = (const bf16 *)dout, *A = (const bf16 *)in_a, *B = (const bf16 *)in_b;
    if (cin != 16 && cin != 32 && cin != 48 && cin != 64 && cin != 96 && cin != 128 && cin != 192) {
        set_error("conv3d weight gradient: input channels must be 16, 32, 48, 64, 96, 128 or 192");
        return false;
    }
    launch_bww(G, cout, A, ca, up_a, B, cb, dw, dbias, n, d, h, wd, s);
    return hip_ok(hipGetLastError(), "conv3d weight gradient launch");
}

bool weight_flip(const void *w, int cout, int cin, void *wt, hipStream_t s) {
    const long long n = 27LL * cout * cin;
    k_flip<<<blocks_for(n), 256, 0, s>>>((const bf16 *)w, (bf16 *)wt, cout, cin);
    return hip_ok(hipGetLastError(), "weight flip launch");
}

bool weight_layout(const void *w, int cout, int cin, void *fwd, void *flip, hipStream_t s) {
    k_layout<<<blocks_for(27LL * cout * cin), 256, 0, s>>>((const bf16 *)w, (bf16 *)fwd, (bf16 *)flip, cout, cin);
    return hip_ok(hipGetLastError(), "weight layout launch");
}

bool relu_bwd(void *dy, const void *y, long long count, hipStream_t s) {
    k_relu_bwd<<<blocks_for(count), 256, 0, s>>>((bf16 *)dy, (const bf16 *)y, count);
    return hip_ok(hipGetLastError(), "relu backward launch");
}

bool pool2(const void *in, void *out, int c, int n, int d, int h, int wd, hipStream_t s) {
    const long long cnt = (long long)n * (d / 2) * (h / 2) * (wd / 2) * c;
    // 16-byte accesses where every voxel's channels allow them (8 x 64^3 x 16: 22 -> 14 us)
    if (c % 8 == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0)
        k_pool<8><<<blocks_for(cnt / 8), 256, 0, s>>>((const bf16 *)in, (bf16 *)out, c, n, d, h, wd);
    else
        k_pool<1><<<blocks_for(cnt), 256, 0, s>>>((const bf16 *)in, (bf16 *)out, c, n, d, h, wd);
    return hip_ok(hipGetLastError(), "pool launch");
}

bool pool2_bwd(const void *dout, void *din, const void *gate, int c, int n, int d, int h, int wd, hipStream_t s) {
    const long long cnt = (long long)n * d * h * wd * c;
    // 16-byte accesses where every voxel's channels allow them: at 8 x 64^3 x 16
    // 102 us with one channel a thread (the index divisions) plus 50 us for the
    // gate as a pass of its own, 32 us with both
    const bool vec = c % 8 == 0 && (((uintptr_t)dout | (uintptr_t)din | (uintptr_t)gate) & 15) == 0;
    if (vec)
        k_pool_bwd<8><<<blocks_for(cnt / 8), 256, 0, s>>>((const bf16 *)dout, (bf16 *)din, (const bf16 *)gate, c, n, d,
                                                          h, wd);
    else
        k_pool_bwd<1><<<blocks_for(cnt), 256, 0, s>>>((const bf16 *)dout, (bf16 *)din, (const bf16 *)gate, c, n, d, h,
                                                      wd);
    return hip_ok(hipGetLastError(), "pool backward launch");
}

bool split_grad(const void *dx, int ca, int cb, void *dup, void *dskip, const void *gate, int n, int d, int h, int wd,
                hipStream_t s) {
    const long long cnt = (long long)n * d * h * wd * (ca > cb ? ca : cb);
    k_split_grad<<<blocks_for(cnt), 256, 0, s>>>((const bf16 *)dx, ca, cb, (bf16 *)dup, (bf16 *)dskip,
                                                (const bf16 *)gate, n, d, h, wd);
    return hip_ok(hipGetLastError(), "split gradient launch");
}

bool stats(const double *rho, const int8_t *mask, long long vs, int n, double *st, hipStream_t s) {
    k_fill_f64<<<1, 64, 0, s>>>(st, 2LL * n);
    // two atomics a block on one line of memory (about 10 ns each)
    dim3 grid(std::min(blocks_for(vs, 4096), 1024u), (unsigned)n);
    k_stats<<<grid, NTH, 0, s>>>(rho, mask, vs, st);
    return hip_ok(hipGetLastError(), "stats launch");
}

bool pack(const double *rho, const int8_t *mask, const double *B, const double *st, int n, long long vs, void *x,
          hipStream_t s) {
    k_pack<<<blocks_for(vs * n), 256, 0, s>>>(rho, mask, B, st, vs, vs * n, (bf16 *)x);
    return hip_ok(hipGetLastError(), "pack launch");
}

template <int S>
static void launch_pack_sums(const double *rho, const int8_t *mask, const double *B, int dc, int hc, int wc,
                             double *sums, double *part, unsigned g, hipStream_t s) {
    if (((uintptr_t)rho & 15) == 0 && ((uintptr_t)mask & 3) == 0)
        k_pack_sums<S, true><<<g, NTH, 0, s>>>(rho, mask, B, dc, hc, wc, sums, part);
    else
        k_pack_sums<S, false><<<g, NTH, 0, s>>>(rho, mask, B, dc, hc, wc, sums, part);
}

long long pack_coarse_words(int dc, int hc, int wc) {
    const long long v = (long long)dc * hc * wc;
    return 3 * v + 2 * ((v + NTH - 1) / NTH);
}

bool pack_coarse(const double *rho, const int8_t *mask, const double *B, double *st, int S, int dc, int hc, int wc,
                 double *work, void *x, hipStream_t s) {
    const long long v = (long long)dc * hc * wc;
    const unsigned g = (unsigned)((v + NTH - 1) / NTH);
    double *part = work + 3 * v;
    if (S == 2) launch_pack_sums<2>(rho, mask, B, dc, hc, wc, work, part, g, s);
    else if (S == 4) launch_pack_sums<4>(rho, mask, B, dc, hc, wc, work, part, g, s);
    else launch_pack_sums<8>(rho, mask, B, dc, hc, wc, work, part, g, s);
    k_stats_sum<<<1, 1024, 0, s>>>(part, (int)g, st);
    k_pack_scale<<<g, NTH, 0, s>>>(work, st, S * S * S, (int)v, (bf16 *)x);
    return hip_ok(hipGetLastError(), "pack launch");
}

bool head(const void *x, const float *w, const float *b, const double *st, const int8_t *mask, double *phi,
          long long vs, int n, hipStream_t s) {
    k_head<<<blocks_for(vs * n), 256, 0, s>>>((const bf16 *)x, w, b, st, mask, phi, vs, n);
    return hip_ok(hipGetLastError(), "head launch");
}

bool up2(const double *c, double *f, int n, int dc, int hc, int wc, const int8_t *mask, hipStream_t s) {
    const long long pl = (long long)hc * wc;
    const int per = pl < NTH ? (int)std::min<long long>(NTH / pl, dc) : 1;
    const dim3 grid((unsigned)((pl + NTH - 1) / NTH), (unsigned)std::min((dc + per - 1) / per, 65535), (unsigned)n);
    if (((uintptr_t)f & 15) == 0) k_up2<true><<<grid, NTH, 0, s>>>(c, f, dc, hc, wc, per, mask);
    else k_up2<false><<<grid, NTH, 0, s>>>(c, f, dc, hc, wc, per, mask);
    return hip_ok(hipGetLastError(), "up-sampling launch");
}

bool coarsen(const double *rho, const int8_t *mask, const double *B, int S, int dc, int hc, int wc, double *rho_c,
             int8_t *mask_c, double *B_c, hipStream_t s) {
    k_coarsen<<<blocks_for((long long)dc * hc * wc), 256, 0, s>>>(rho, mask, B, S, dc, hc, wc, rho_c, mask_c, B_c);
    return hip_ok(hipGetLastError(), "coarsen launch");
}

bool head_loss(const void *x, const float *w, const float *b, const int8_t *mask, const double *target,
               const double *st, int n, long long vs, void *dx, float *dw, float *db, double *loss, hipStream_t s) {
    k_head_loss<<<std::min(blocks_for(vs * n, HL_NT), 256u), HL_NT, 0, s>>>((const bf16 *)x, w, b, mask, target, st, n, vs, (bf16 *)dx,
                                                         dw, db, loss);
    return hip_ok(hipGetLastError(), "loss launch");
}

bool fill_f32(float *p, long long n, hipStream_t s) {
    k_fill_f32<<<blocks_for(n), 256, 0, s>>>(p, n);
    return hip_ok(hipGetLastError(), "fill launch");
}

bool fill_f64(double *p, long long n, hipStream_t s) {
    k_fill_f64<<<blocks_for(n), 256, 0, s>>>(p, n);
    return hip_ok(hipGetLastError(), "fill launch");
}

bool adamw(float *p, void *pb, const float *g, float *m, float *v, long long n, float lr, float b1, float b2, float eps,
           float wd, int step, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    k_adamw<<<blocks_for(n), 256, 0, s>>>(p, (bf16 *)pb, g, m, v, n, lr, b1, b2, eps, wd, c1, c2);
    return hip_ok(hipGetLastError(), "adamw launch");
}

}  // namespace nn
}  // namespace mg

using namespace mg;

#define NN_RET(x) return (x) ? MG_OK : MG_ERR_HIP

extern "C" {

mg_status mg_nn_conv3d_fwd(const void *in_a, int32_t ca, int32_t up_a, const void *in_b, int32_t cb, const void *w,
                           const float *bias, void *out, int32_t cout, int32_t relu, int32_t n, int32_t d, int32_t h,
                           int32_t wd, void *stream) {
    if (!in_a || !w || !out || ca <= 0 || cb < 0 || (cb > 0 && !in_b) || ca % 8 || cb % 8 || cout <= 0 || cout % 16 ||
        n <= 0 || d <= 0 || h <= 0 || wd <= 0 || (up_a && (d % 2 || h % 2 || wd % 2))) {
        set_error("mg_nn_conv3d_fwd: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::conv_fwd(in_a, ca, up_a, in_b, cb, w, bias, out, cout, relu, n, d, h, wd, (hipStream_t)stream));
}

mg_status mg_nn_conv3d_bwd_weight(const void *dout, int32_t cout, const void *in_a, int32_t ca, int32_t up_a,
                                  const void *in_b, int32_t cb, float *dw, float *dbias, int32_t n, int32_t d,
                                  int32_t h, int32_t wd, void *stream) {
    const int cin = ca + cb;
    const bool cin_ok = cin == 16 || cin == 32 || cin == 48 || cin == 64 || cin == 96 || cin == 128 || cin == 192;
    if (!dout || !in_a || !dw || cout <= 0 || cout % 16 || ca <= 0 || ca % 8 || cb < 0 || cb % 8 ||
        (cb > 0 && !in_b) || !cin_ok || n <= 0 || d <= 0 || h <= 0 || wd <= 0 ||
        (up_a && (d % 2 || h % 2 || wd % 2))) {
        set_error("mg_nn_conv3d_bwd_weight: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::conv_bwd_weight(dout, cout, in_a, ca, up_a, in_b, cb, dw, dbias, n, d, h, wd, (hipStream_t)stream));
}

mg_status mg_nn_weight_flip(const void *w, int32_t cout, int32_t cin, void *wt, void *stream) {
    if (!w || !wt || cout <= 0 || cin <= 0) {
        set_error("mg_nn_weight_flip: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::weight_flip(w, cout, cin, wt, (hipStream_t)stream));
}

mg_status mg_nn_relu_bwd(void *dy, const void *y, int64_t count, void *stream) {
    if (!dy || !y || count <= 0) {
        set_error("mg_nn_relu_bwd: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::relu_bwd(dy, y, count, (hipStream_t)stream));
}

mg_status mg_nn_pool2(const void *in, void *out, int32_t c, int32_t n, int32_t d, int32_t h, int32_t wd, void *stream) {
    if (!in || !out || c <= 0 || n <= 0 || d <= 0 || h <= 0 || wd <= 0 || d % 2 || h % 2 || wd % 2) {
        set_error("mg_nn_pool2: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::pool2(in, out, c, n, d, h, wd, (hipStream_t)stream));
}

mg_status mg_nn_pool2_bwd(const void *dout, void *din, int32_t c, int32_t n, int32_t d, int32_t h, int32_t wd,
                          void *stream) {
    if (!dout || !din || c <= 0 || n <= 0 || d <= 0 || h <= 0 || wd <= 0 || d % 2 || h % 2 || wd % 2) {
        set_error("mg_nn_pool2_bwd: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::pool2_bwd(dout, din, nullptr, c, n, d, h, wd, (hipStream_t)stream));
}

mg_status mg_nn_split_grad(const void *dx, int32_t ca, int32_t cb, void *dup, void *dskip, int32_t n, int32_t d,
                           int32_t h, int32_t wd, void *stream) {
    if (!dx || !dup || ca <= 0 || cb < 0 || (cb > 0 && !dskip) || n <= 0 || d <= 0 || h <= 0 || wd <= 0 || d % 2 ||
        h % 2 || wd % 2) {
        set_error("mg_nn_split_grad: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::split_grad(dx, ca, cb, dup, dskip, nullptr, n, d, h, wd, (hipStream_t)stream));
}

mg_status mg_nn_adamw(float *param, void *param_bf16, const float *grad, float *m, float *v, int64_t count, float lr,
                      float beta1, float beta2, float eps, float weight_decay, int32_t step, void *stream) {
    if (!param || !grad || !m || !v || count <= 0 || step < 1) {
        set_error("mg_nn_adamw: invalid arguments");
        return MG_ERR_ARG;
    }
    NN_RET(nn::adamw(param, param_bf16, grad, m, v, count, lr, beta1, beta2, eps, weight_decay, step,
                     (hipStream_t)stream));
}

mg_status mg_nn_mfma_selftest(float *out_dev, void *stream) {
    if (!out_dev) {
        set_error("mg_nn_mfma_selftest: null output");
        return MG_ERR_ARG;
    }
    nn::k_mfma_selftest<<<1, 64, 0, (hipStream_t)stream>>>(out_dev);
    return hip_ok(hipGetLastError(), "mfma selftest launch") ? MG_OK : MG_ERR_HIP;
}

}  // extern "C"
