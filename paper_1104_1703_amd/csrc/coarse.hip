// Small coarse levels in one workgroup.
//
// Below a few thousand cells a level is far too small to fill the GPU, and
// one launch per half-sweep would cost more than the work.  This kernel runs
// one whole multigrid call MG(ls) (Sec. 2 enumerated recipe, with N_cycles
// recursive calls per level and n_coarse passes on the deepest level) for the
// levels ls..last inside one 1024-thread workgroup, with every level's x, f
// and diagonal resident in LDS.  Red-black Gauss-Seidel is done in place with
// a barrier between the colours (a colour only reads the other colour).
#include <algorithm>

#include "coarse_core.h"

namespace mg {

namespace {

using namespace small;

constexpr int NTC = 1024;  // 16 waves: four per SIMD to hide LDS and FP64 latency

template <typename T>
__global__ __launch_bounds__(NTC) void k_coarse(SmallLevels<T> S) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (S.halt && *S.halt) return;
    T *sm = reinterpret_cast<T *>(smem_raw);
    if (S.fast) small_fast<T, NTC>(sm, S, S.f0, S.x0, S.load_x != 0);
    else small_tail<T, NTC>(sm, S, S.f0, S.x0, S.load_x != 0);
}

// Column blockIdx.x of the deepest level's relaxation matrix (deep_solve):
// `passes` passes from zero on the unit right-hand side of that cell.
__global__ __launch_bounds__(DEEP_MAX) void k_deep_matrix(Lv<double> L, const double *__restrict__ d, int passes,
                                                         double *__restrict__ M, float *__restrict__ M32) {
    __shared__ double sx[DEEP_MAX], sf[DEEP_MAX], sd[DEEP_MAX];
    const int e = threadIdx.x, j = blockIdx.x;
    if (e < L.n) {
        sx[e] = 0.0;
        sd[e] = d[e];
        sf[e] = e == j && sd[e] != 0.0 ? 1.0 : 0.0;
    }
    L.x = sx;
    L.f = sf;
    L.d = sd;
    __syncthreads();
    smooth<double, DEEP_MAX>(L, passes);
    if (e < L.n) {
        M[e * L.n + j] = sx[e];
        if (M32) M32[e * L.n + j] = (float)sx[e];
    }
}

template <typename T>
void launch_impl(const mg_hierarchy *H, int order, int ls, bool zero_start, const T *f0, T *x0, hipStream_t s,
                 bool f32) {
    SmallLevels<T> S{};
    const int last = H->nlev[order] - 1;
    S.n = last - ls + 1;
    int off = 0;
    for (int q = 0; q < S.n; q++) {
        const Level &L = H->lev[ls + q];
        S.nx[q] = L.nx;
        S.ny[q] = L.ny;
        S.nz[q] = L.nz;
        S.mx[q] = div_magic((unsigned)L.nx);
        S.mxy[q] = div_magic((unsigned)(L.nx * L.ny));
        S.mh[q] = div_magic((unsigned)((L.nx + 1) / 2));
        S.mhy[q] = div_magic((unsigned)((L.nx + 1) / 2 * L.ny));
        S.h2[q] = (T)(L.h * L.h);
        S.ih2[q] = (T)(1.0 / (L.h * L.h));
        S.d[q] = f32 ? (const T *)L.od[order].d32 : (const T *)L.od[order].d;
        if (q < 2) S.rd[q] = f32 ? (const T *)L.od[order].rd32 : (const T *)L.od[order].rd;
        S.off[q] = off;
        off += 3 * (int)L.n;
    }
    S.f0 = f0;
    S.x0 = x0;
    S.load_x = zero_start ? 0 : 1;
    S.deep = f32 ? (const T *)H->lev[last].od[order].deep32 : (const T *)H->lev[last].od[order].deep;
    S.halt = H->lev[0].halt;
    S.n_pre = H->opt.n_pre;
    S.n_post = H->opt.n_post;
    S.n_cycles = H->opt.n_cycles;
    S.n_coarse = H->opt.n_coarse_sweeps;
    S.fast = small_fast_levels(H, order, ls) ? 1 : 0;
    const size_t bytes = small_lds_bytes(H, order, ls, f32);
    k_coarse<T><<<1, NTC, bytes, s>>>(S);
}

}  // namespace

bool small_direct(const mg_hierarchy *H, int order, int ls) {
    const int last = H->nlev[order] - 1;
    return deep_product(last - ls + 1, H->lev[last].n, (long long)H->opt.n_cycles * H->opt.n_coarse_sweeps);
}

void launch_deep_matrix(const Level &L, const OrderData &od, int passes, hipStream_t s) {
    Lv<double> v{};
    v.nx = L.nx;
    v.ny = L.ny;
    v.nz = L.nz;
    v.n = (int)L.n;
    v.mx = div_magic((unsigned)L.nx);
    v.mxy = div_magic((unsigned)(L.nx * L.ny));
    v.hx = (L.nx + 1) / 2;
    v.mh = div_magic((unsigned)v.hx);
    v.mhy = div_magic((unsigned)(v.hx * L.ny));
    v.h2 = L.h * L.h;
    v.ih2 = 1.0 / (L.h * L.h);
    k_deep_matrix<<<(unsigned)L.n, DEEP_MAX, 0, s>>>(v, od.d, passes, od.deep, od.deep32);
}

__global__ void k_reciprocals(const double *__restrict__ d, size_t n, double *__restrict__ rd,
                              float *__restrict__ rd32) {
    const size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (p >= n) return;
    rd[p] = d[p] != 0.0 ? 1.0 / d[p] : 0.0;
    if (rd32) rd32[p] = d[p] != 0.0 ? 1.0f / (float)d[p] : 0.0f;
}

void launch_reciprocals(const Level &L, const OrderData &od, hipStream_t s) {
    k_reciprocals<<<(unsigned)((L.n + 255) / 256), 256, 0, s>>>(od.d, L.n, od.rd, od.rd32);
}

namespace {

// Dims of the levels ls .. last (at most three) for fast_fits / fast_lds.
struct SmallDims {
    int n = 0, nx[3], ny[3], nz[3];
    bool direct = false;
    SmallDims(const mg_hierarchy *H, int order, int ls) {
        const int last = H->nlev[order] - 1;
        n = last - ls + 1;
        for (int q = 0; q < n && q < 3; q++) {
            const Level &L = H->lev[ls + q];
            nx[q] = L.nx, ny[q] = L.ny, nz[q] = L.nz;
        }
        direct = small_direct(H, order, ls);
    }
};

}  // namespace

bool small_fast_levels(const mg_hierarchy *H, int order, int ls) {
    const SmallDims d(H, order, ls);
    return fast_fits(d.n, d.direct, d.nx, d.ny, d.nz, NTC);
}

size_t small_lds_bytes(const mg_hierarchy *H, int order, int ls, bool f32) {
    size_t n = 0;
    for (int l = ls; l < H->nlev[order]; l++) n += 3 * H->lev[l].n;
    const SmallDims d(H, order, ls);
    if (fast_fits(d.n, d.direct, d.nx, d.ny, d.nz, NTC))
        n = std::max(n, (size_t)fast_lds(d.n, d.direct, d.nx, d.ny, d.nz).end);
    return n * (f32 ? sizeof(float) : sizeof(double));
}

// Largest dynamic LDS the one-workgroup kernel may use on the current device
// (0 if it cannot run).  Any refused request is cleared so that no error is
// left pending for the caller's next HIP call.
int small_init() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    int lim = std::min(v, SMALL_LDS_MAX) - 1024;  // room for the kernel's static LDS
    if (lim > 64 * 1024 - 1024) {
        if (hipFuncSetAttribute((const void *)k_coarse<double>, hipFuncAttributeMaxDynamicSharedMemorySize, lim) !=
                hipSuccess ||
            hipFuncSetAttribute((const void *)k_coarse<float>, hipFuncAttributeMaxDynamicSharedMemorySize, lim) !=
                hipSuccess) {
            (void)hipGetLastError();
            lim = 64 * 1024 - 1024;
        }
    }
    return lim > 0 ? lim : 0;
}

void launch_small(const mg_hierarchy *H, int order, int ls, bool zero_start, const double *f0, double *x0,
                  hipStream_t s) {
    launch_impl<double>(H, order, ls, zero_start, f0, x0, s, false);
}

void launch_small32(const mg_hierarchy *H, int order, int ls, bool zero_start, const float *f0, float *x0,
                    hipStream_t s) {
    launch_impl<float>(H, order, ls, zero_start, f0, x0, s, true);
}

}  // namespace mg
