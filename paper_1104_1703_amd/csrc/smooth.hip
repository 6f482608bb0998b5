// Masked red-black Gauss-Seidel smoother (Sec. 2: red-black ordering of the
// 7-point Laplacian; Sec. 3: ghost-modified operator near the boundary).
//
// One launch performs one full pass (red half-sweep, then black) over the
// active segments of a level.  Relaxing an active cell i solves its own
// equation (1/h^2)(sum_{j active} x_j - d_i x_i) = f_i for x_i; inactive
// cells hold x = 0, so the neighbour sum runs over all six neighbours.
//
// Work item: a TX x TY column of cells marching up a z range.  The block keeps
// a ring of four planes in LDS: x with a 2-cell xy halo, f and the diagonal
// (or the finest-level neighbour code) with a 1-cell halo.  At step k it
// relaxes red cells of plane k+1 on the tile plus a 1-cell ring (redundantly
// with the neighbouring work items, from identical inputs), then black cells
// of plane k on the tile, and writes plane k.  Red cells only read black ones
// and vice versa, so each plane is updated in place; reads come from `xin`
// and writes go to `xout` (ping-pong), so concurrent work items never see
// each other's results.  Global loads of the planes needed two and three
// steps ahead are in flight in registers while a step computes, so the
// compute phases touch LDS only.  Loads go through buffer resources and are
// masked per 16-cell row granule by the item's precomputed activity masks:
// granules without an active cell (outside the domain, inside holes, halo rows
// of inactive neighbours) are never fetched, and inactive cells are never
// stored.  Net HBM traffic per pass: one read of x, f and the code/diagonal
// and one write of x, on granules holding active cells.
#include <hip/hip_ext.h>

#include "cube_core.h"
#include "mg_core.h"
#include "smooth2_core.h"
#include "smooth_res_core.h"
#include "transfer_core.h"

namespace mg {

namespace {

using namespace rb;

// Five blocks per CU (LDS); the finest float passes (16-19 KB of LDS, 62
// registers) eight, so that the 2048 items of a 256^3 pass run in one round.
template <typename T, bool FINE, int SEGZ, bool PRO = false, int AUX = 0>
__global__ __launch_bounds__(NT, FINE && sizeof(T) == 4 ? 8 : 5) void k_rbgs(
    const T *__restrict__ xin, T *__restrict__ xout, const T *__restrict__ f, const uint8_t *__restrict__ code,
    const T *__restrict__ dco, int nx, int ny, int nz, T h2, const Seg *__restrict__ segs,
    const unsigned long long *__restrict__ pm, int nsegs, const int *__restrict__ halt, const T *__restrict__ xc = nullptr,
    int cnx = 0, int cny = 0, int cnz = 0) {
    __shared__ RbgsLds<T, FINE, PRO> lds;
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= nsegs || (halt && *halt)) return;
    rbgs_item<T, FINE, SEGZ, PRO, false, AUX>(lds, xin, xout, f, code, dco, nx, ny, nz, h2, segs[item],
                                              pm + (size_t)item * (SEGZ + 4), xc, cnx, cny, cnz);
}

// The finest pass that also forms the residual-norm partials of its input,
// one per work item, as the residual-norm march does.
template <int SZ, int AUX>
__global__ __launch_bounds__(NT, 5) void k_rbgs_norm(const double *__restrict__ xin, double *__restrict__ xout,
                                                   const double *__restrict__ f, const uint8_t *__restrict__ code,
                                                   int nx, int ny, int nz, double h2, double ih2,
                                                   const Seg *__restrict__ segs,
                                                   const unsigned long long *__restrict__ pm, int nsegs,
                                                   const int *__restrict__ halt, double *__restrict__ part) {
    __shared__ RbgsLds<double, true, false> lds;
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= nsegs || (halt && *halt)) return;
    const double sq = rbgs_item<double, true, SZ, false, true, AUX>(lds, xin, xout, f, code, nullptr, nx, ny, nz, h2,
                                                                    segs[item], pm + (size_t)item * (SZ + 4), nullptr,
                                                                    0, 0, 0, ih2);
    const double t = tr::block_sum(sq);
    if (threadIdx.x == 0) part[item] = t;
}

// The finest pass that also forms the residual of its result and restricts
// it onto level 1 (smooth_res_core.h): four FP64 blocks per CU (LDS), six
// FP32 blocks.
template <typename T, int SEGZ, int AUX>
__global__ __launch_bounds__(NT, sizeof(T) == 8 ? 4 : 6) void k_rbgs_res(
    const T *__restrict__ xin, T *__restrict__ xout, const T *__restrict__ f, const uint8_t *__restrict__ code, int nx,
    int ny, int nz, T h2, T ih2, const Seg *__restrict__ segs, const unsigned long long *__restrict__ pm, int nsegs,
    const int *__restrict__ halt, const T *__restrict__ cd, int cnx, int cny, T *__restrict__ fc) {
    __shared__ rbr::Lds<T> lds;
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= nsegs || (halt && *halt)) return;
    rbr::rbgs_res_item<T, SEGZ, AUX>(lds, xin, xout, f, code, nx, ny, nz, h2, ih2, segs[item],
                                     pm + (size_t)item * (SEGZ + 2 * rbr::H), cd, cnx, cny, fc);
}

// Two passes per launch (smooth2_core.h): LDS allows two FP64 blocks per CU.
template <typename T, bool FINE, int SEGZ, bool PRO = false>
__global__ __launch_bounds__(NT, 2) void k_rbgs2(const T *__restrict__ xin, T *__restrict__ xout,
                                               const T *__restrict__ f, const uint8_t *__restrict__ code,
                                               const T *__restrict__ dco, int nx, int ny, int nz, T h2,
                                               const Seg *__restrict__ segs, const unsigned long long *__restrict__ pm,
                                               int nsegs, const int *__restrict__ halt,
                                               const T *__restrict__ xc = nullptr, int cnx = 0, int cny = 0,
                                               int cnz = 0) {
    __shared__ rb2::Lds<T, FINE, PRO> lds;
    const int item = xcd_item(blockIdx.x, gridDim.x);
    if (item >= nsegs || (halt && *halt)) return;
    rb2::rbgs2_item<T, FINE, SEGZ, PRO>(lds, xin, xout, f, code, dco, nx, ny, nz, h2, segs[item],
                                        pm + (size_t)item * (SEGZ + 2 * rb2::H), xc, cnx, cny, cnz);
}

// Origin of cube `item` (four per active 32 x 8 x 8 tile); false past the last
// cube and for cubes of a tile wider than the level.
struct CubeAt {
    int x0, y0, z0;
};
__device__ __forceinline__ bool cube_at(int item, const int *tiles, int ntiles, int ntx, int nty, int nx, CubeAt &c) {
    if (item >= 4 * ntiles) return false;
    const int tile = tiles[item >> 2];
    c.x0 = (tile % ntx) * TX + (item & 3) * cube::C;
    c.y0 = (tile / ntx) % nty * TY;
    c.z0 = tile / (ntx * nty) * TZ;
    return c.x0 < nx;
}

// Pass over 8 x 8 x 8 cubes, each loaded whole: cube_core.h.
template <typename T, bool FINE, bool PRO>
__global__ __launch_bounds__(cube::NT) void k_rbgs_cube(const T *__restrict__ xin, T *__restrict__ xout,
                                                      const T *__restrict__ f,
                                                      const cube::DiagT<T, FINE> *__restrict__ d, int nx, int ny,
                                                      int nz, int ntx, int nty, T h2, const int *__restrict__ tiles,
                                                      int ntiles, const int *__restrict__ halt,
                                                      const T *__restrict__ xc, int cnx, int cny, int cnz) {
    __shared__ cube::Lds<T, FINE, PRO> lds;
    CubeAt c;
    if (!cube_at(xcd_item(blockIdx.x, gridDim.x), tiles, ntiles, ntx, nty, nx, c) || (halt && *halt)) return;
    cube::rbgs_cube<T, FINE, PRO>(lds, xin, xout, f, d, nx, ny, nz, h2, c.x0, c.y0, c.z0, xc, cnx, cny, cnz);
}

// The cube pass that also forms the residual and its R1 restriction onto
// the next coarser level (the last pre-smoothing pass of a cube level).
template <typename T, bool FINE>
__global__ __launch_bounds__(cube::NT) void k_rbgs_cube_restrict(
    const T *__restrict__ xin, T *__restrict__ xout, const T *__restrict__ f,
    const cube::DiagT<T, FINE> *__restrict__ d, int nx, int ny, int nz, int ntx, int nty, T h2, T ih2,
    const int *__restrict__ tiles, int ntiles, const int *__restrict__ halt, const T *__restrict__ cd,
    T *__restrict__ fc, int cnx, int cny, int cnz) {
    __shared__ cube::LdsRes<T, FINE> lds;
    CubeAt c;
    if (!cube_at(xcd_item(blockIdx.x, gridDim.x), tiles, ntiles, ntx, nty, nx, c) || (halt && *halt)) return;
    cube::rbgs_cube_restrict<T, FINE>(lds, xin, xout, f, d, nx, ny, nz, h2, ih2, c.x0, c.y0, c.z0, cd, fc, cnx, cny,
                                      cnz);
}

// A finest cube pass whose launch also forms the residual-norm partials of
// its input: the first nitems blocks take one work item's partial each (as
// launch_resnorm does), the others one cube.
__global__ __launch_bounds__(cube::NT) void k_rbgs_cube_norm(
    const double *__restrict__ xin, double *__restrict__ xout, const double *__restrict__ f,
    const uint8_t *__restrict__ code, int nx, int ny, int nz, int ntx, int nty, double h2, double ih2,
    const int *__restrict__ tiles, int ntiles, const Seg *__restrict__ segs, int nitems, const int *__restrict__ halt,
    double *__restrict__ part) {
    __shared__ cube::Lds<double, true, false> lds;
    if (halt && *halt) return;
    const int b = blockIdx.x;
    if (b < nitems) {  // uniform per block
        const double t = tr::block_sum(tr::item_norm(segs[b], xin, f, code, nx, ny, nz, ih2));
        if (threadIdx.x == 0) part[b] = t;
        return;
    }
    CubeAt c;
    if (!cube_at(xcd_item(b - nitems, gridDim.x - nitems), tiles, ntiles, ntx, nty, nx, c)) return;
    cube::rbgs_cube<double, true, false>(lds, xin, xout, f, code, nx, ny, nz, h2, c.x0, c.y0, c.z0);
}

inline unsigned grid8(int items) { return (unsigned)(((items + 7) / 8) * 8); }

template <typename T>
struct same_t {
    using type = T;
};
// Launches kernel k over `grid` blocks of NT threads; with events, through
// hipExtLaunchKernel so that e0 and e1 take the kernel's own start and end.
template <typename... P>
hipError_t launch_k(void (*k)(P...), unsigned grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                    typename same_t<P>::type... a) {
    if (!e0 && !e1) {
        k<<<grid, NT, 0, s>>>(a...);
        return hipSuccess;
    }
    void *args[] = {(void *)&a...};
    return hipExtLaunchKernel((const void *)k, dim3(grid), dim3(NT), args, 0, s, e0, e1, 0);
}

}  // namespace

// The level's diagonal as the cube kernels take it.
template <typename T, bool FINE>
const cube::DiagT<T, FINE> *cube_diag(const Level &L, const OrderData &od) {
    if constexpr (FINE) return L.code;
    else if constexpr (sizeof(T) == 8) return od.d;
    else return od.d32;
}

template <typename T, bool FINE>
hipError_t launch_cube_restrict(const T *xin, T *xout, const T *f, const Level &L, const OrderData &od,
                                const Level &C, const T *cd, T *fc, hipStream_t s, hipEvent_t e0 = nullptr,
                                hipEvent_t e1 = nullptr) {
    if (od.ntiles == 0) return hipSuccess;
    return launch_k(k_rbgs_cube_restrict<T, FINE>, grid8(4 * od.ntiles), s, e0, e1, xin, xout, f,
                    cube_diag<T, FINE>(L, od), L.nx, L.ny, L.nz, L.ntx, L.nty, (T)(L.h * L.h),
                    (T)(1.0 / (L.h * L.h)), od.tiles, od.ntiles, L.halt, cd, fc, C.nx, C.ny, C.nz);
}

template <typename T, bool FINE, bool PRO = false>
hipError_t launch_cube(const T *xin, T *xout, const T *f, const Level &L, const OrderData &od, hipStream_t s,
                       hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr, const T *xc = nullptr,
                       const Level *C = nullptr) {
    static_assert(TX == 4 * cube::C && TY == cube::C && TZ == cube::C, "a tile holds four cubes");
    if (od.ntiles == 0) return hipSuccess;
    return launch_k(k_rbgs_cube<T, FINE, PRO>, grid8(4 * od.ntiles), s, e0, e1, xin, xout, f,
                    cube_diag<T, FINE>(L, od), L.nx, L.ny, L.nz, L.ntx, L.nty, (T)(L.h * L.h), od.tiles, od.ntiles,
                    L.halt, xc, C ? C->nx : 0, C ? C->ny : 0, C ? C->nz : 0);
}

void launch_rbgs_restrict(const Level &L, const Level &C, int order, const OrderData &od, const double *xin,
                          double *xout, const double *f, double *fc, hipStream_t s) {
    (void)launch_cube_restrict<double, false>(xin, xout, f, L, od, C, C.od[order].d, fc, s);
}

void launch_rbgs_restrict32(const Level &L, const Level &C, int order, const OrderData &od, const float *xin,
                            float *xout, const float *f, float *fc, hipStream_t s) {
    (void)launch_cube_restrict<float, false>(xin, xout, f, L, od, C, C.od[order].d32, fc, s);
}

// Calls launch with a finest pass's item depth and the cache policy of its
// stores.  The result is stored non-temporally when what a pass touches (x in
// and out, f and the code, on active cells) is more than the 256 MiB last-level
// cache holds: the next pass then finds nothing of it there anyway.  Below that
// size it reads the result back from that cache.  At 512^3 porous the FP32
// passes take 1-4% less time so (plain 475 -> 458 us, residual 666 -> 653,
// prolongation 605 -> 588), the passes with the larger halos also reading less
// (residual 1.72 -> 1.58 GB); the FP64 plain pass
// 890 -> 866 us, though it reads 4% more.  Solve times, without and with: FP64
// 192^3 porous (166 MB) 12.57 / 13.69 ms, 256^3 holes (152 MB) 12.56 / 13.26,
// 256^3 porous (394 MB) 25.7 / 25.1, 384^3 holes (510 MB) 38.7 / 38.4, 512^3
// holes (1.2 GB) 89.8 / 87.9; mixed precision (with the update's outputs always
// stored so) 256^3 porous (205 MB) 20.5 / 21.6, 320^3 (400 MB) 44.0 / 43.5,
// 512^3 (1.6 GB) 163.6 / 162.2.
template <typename T, typename F>
void with_fine_pass(const OrderData &od, F &&launch) {
    const bool stream = (size_t)od.nact * (3 * sizeof(T) + 1) > ((size_t)256 << 20);
    with_fine_depth(od.depth, [&](auto Z) {
        if (stream) launch(Z, std::integral_constant<int, STREAM>{});
        else launch(Z, std::integral_constant<int, 0>{});
    });
}

template <typename T>
hipError_t launch_fine_res(const Level &L, const OrderData &od, const T *xin, T *xout, const T *f, const Level &C,
                           const T *cd, T *fc, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    if (od.few_wide()) return launch_cube_restrict<T, true>(xin, xout, f, L, od, C, cd, fc, s, e0, e1);
    const T h2 = (T)(L.h * L.h), ih2 = (T)(1.0 / (L.h * L.h));
    hipError_t err = hipSuccess;
    with_fine_pass<T>(od, [&](auto Z, auto P) {
        err = launch_k(k_rbgs_res<T, decltype(Z)::value, decltype(P)::value>, grid8(od.nsegs), s, e0, e1, xin, xout, f, L.code, L.nx,
                       L.ny, L.nz, h2, ih2, od.segs, od.pmask3, od.nsegs, L.halt, cd, C.nx, C.ny, fc);
    });
    return err;
}

hipError_t launch_rbgs_res_fine(const Level &L, const Level &C, int order, const OrderData &od, const double *xin,
                                double *xout, const double *f, double *fc, hipStream_t s, hipEvent_t e0,
                                hipEvent_t e1) {
    return launch_fine_res<double>(L, od, xin, xout, f, C, C.od[order].d, fc, s, e0, e1);
}

hipError_t launch_rbgs_res_fine32(const Level &L, const Level &C, int order, const OrderData &od, const float *xin,
                                  float *xout, const float *f, float *fc, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1) {
    return launch_fine_res<float>(L, od, xin, xout, f, C, C.od[order].d32, fc, s, e0, e1);
}

// Coarse levels: the kernel instance for the level's item depth.
template <typename T, bool PRO = false>
void launch_coarse(int depth, const T *xin, T *xout, const T *f, const T *d, const Level &L, const OrderData &od,
                   T h2, hipStream_t s, const T *xc = nullptr, const Level *C = nullptr) {
    const int cnx = C ? C->nx : 0, cny = C ? C->ny : 0, cnz = C ? C->nz : 0;
    if (depth == 8)
        k_rbgs<T, false, 8, PRO><<<grid8(od.nsegs), NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2,
                                                               od.segs, od.pmask, od.nsegs, L.halt, xc, cnx, cny, cnz);
    else if (depth == 2)
        k_rbgs<T, false, 2, PRO><<<grid8(od.nsegs), NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2,
                                                               od.segs, od.pmask, od.nsegs, L.halt, xc, cnx, cny, cnz);
    else
        k_rbgs<T, false, 4, PRO><<<grid8(od.nsegs), NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2,
                                                               od.segs, od.pmask, od.nsegs, L.halt, xc, cnx, cny, cnz);
}
static_assert((SEGZ_COARSE1 == 2 || SEGZ_COARSE1 == 4 || SEGZ_COARSE1 == 8) &&
                  (SEGZ_COARSE == 2 || SEGZ_COARSE == 4 || SEGZ_COARSE == 8),
              "coarse item depths have kernel instances for 2, 4 and 8 planes");

// A finest-level pass; with events, launched so that e0 and e1 take the
// kernel's own start and end times.
template <typename T>
hipError_t launch_fine(const Level &L, const OrderData &od, const T *xin, T *xout, const T *f, T h2, hipStream_t s,
                       hipEvent_t e0, hipEvent_t e1) {
    if (od.few) return launch_cube<T, true>(xin, xout, f, L, od, s, e0, e1);
    hipError_t err = hipSuccess;
    with_fine_pass<T>(od, [&](auto Z, auto P) {
        err = launch_k(k_rbgs<T, true, decltype(Z)::value, false, decltype(P)::value>, grid8(od.nsegs), s, e0, e1, xin, xout, f, L.code,
                       (const T *)nullptr, L.nx, L.ny, L.nz, h2, od.segs, od.pmask, od.nsegs, L.halt,
                       (const T *)nullptr, 0, 0, 0);
    });
    return err;
}

hipError_t launch_rbgs(const Level &L, int level, const OrderData &od, const double *xin, double *xout,
                       const double *f, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    const double h2 = L.h * L.h;
    if (level == 0)
        return launch_fine<double>(L, od, xin, xout, f, h2, s, e0, e1);
    else if (od.cubes())
        return launch_cube<double, false>(xin, xout, f, L, od, s);
    else
        launch_coarse<double>(od.depth, xin, xout, f, od.d, L, od, h2, s);
    return hipSuccess;
}

hipError_t launch_rbgs_norm(const Level &L, const OrderData &od, const double *xin, double *xout, const double *f,
                            double *part, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    if (od.few_wide())
        return launch_k(k_rbgs_cube_norm, (unsigned)od.nsegs + grid8(4 * od.ntiles), s, e0, e1, xin, xout, f, L.code,
                        L.nx, L.ny, L.nz, L.ntx, L.nty, L.h * L.h, 1.0 / (L.h * L.h), od.tiles, od.ntiles, od.segs,
                        od.nsegs, L.halt, part);
    hipError_t err = hipSuccess;
    with_fine_pass<double>(od, [&](auto Z, auto P) {
        err = launch_k(k_rbgs_norm<decltype(Z)::value, decltype(P)::value>, grid8(od.nsegs), s, e0, e1, xin, xout, f, L.code, L.nx, L.ny,
                       L.nz, L.h * L.h, 1.0 / (L.h * L.h), od.segs, od.pmask, od.nsegs, L.halt, part);
    });
    return err;
}

hipError_t launch_rbgs_prolong(const Level &L, int level, const OrderData &od, const Level &C, const double *xc,
                               const double *xin, double *xout, const double *f, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    if (od.few_prolong(level, false))
        return level == 0 ? launch_cube<double, true, true>(xin, xout, f, L, od, s, e0, e1, xc, &C)
                          : launch_cube<double, false, true>(xin, xout, f, L, od, s, e0, e1, xc, &C);
    const double h2 = L.h * L.h;
    hipError_t err = hipSuccess;
    if (level == 0)
        with_fine_pass<double>(od, [&](auto Z, auto P) {
            err = launch_k(k_rbgs<double, true, decltype(Z)::value, true, decltype(P)::value>, grid8(od.nsegs), s, e0, e1, xin, xout, f,
                           L.code, (const double *)nullptr, L.nx, L.ny, L.nz, h2, od.segs, od.pmask, od.nsegs, L.halt,
                           xc, C.nx, C.ny, C.nz);
        });
    else if (level == 1 && od.nsegs8 > 0)  // whole tiles: one round at 4 blocks per CU
        k_rbgs<double, false, TZ, true><<<grid8(od.nsegs8), NT, 0, s>>>(xin, xout, f, nullptr, od.d, L.nx, L.ny, L.nz,
                                                                      h2, od.segs8, od.pmask8, od.nsegs8, L.halt, xc,
                                                                      C.nx, C.ny, C.nz);
    else
        launch_coarse<double, true>(od.depth, xin, xout, f, od.d, L, od, h2, s, xc, &C);
    return err;
}

hipError_t launch_rbgs_prolong32(const Level &L, int level, const OrderData &od, const Level &C, const float *xc,
                                 const float *xin, float *xout, const float *f, hipStream_t s, hipEvent_t e0,
                                 hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    if (od.few_prolong(level, true))
        return level == 0 ? launch_cube<float, true, true>(xin, xout, f, L, od, s, e0, e1, xc, &C)
                          : launch_cube<float, false, true>(xin, xout, f, L, od, s, e0, e1, xc, &C);
    const float h2 = (float)(L.h * L.h);
    hipError_t err = hipSuccess;
    if (level == 0)
        with_fine_pass<float>(od, [&](auto Z, auto P) {
            err = launch_k(k_rbgs<float, true, decltype(Z)::value, true, decltype(P)::value>, grid8(od.nsegs), s, e0, e1, xin, xout, f,
                           L.code, (const float *)nullptr, L.nx, L.ny, L.nz, h2, od.segs, od.pmask, od.nsegs, L.halt,
                           xc, C.nx, C.ny, C.nz);
        });
    else
        launch_coarse<float, true>(od.depth, xin, xout, f, od.d32, L, od, h2, s, xc, &C);
    return err;
}

template <typename T>
void launch_fused(const Level &L, int level, const OrderData &od, const T *xin, T *xout, const T *f, const T *d,
                  T h2, hipStream_t s) {
    if (od.nsegs == 0) return;
    const unsigned g = grid8(od.nsegs);
    if (level == 0)
        k_rbgs2<T, true, SEG_TILES_FINE * TZ><<<g, NT, 0, s>>>(xin, xout, f, L.code, nullptr, L.nx, L.ny, L.nz, h2,
                                                               od.segs, od.pmask2, od.nsegs, L.halt);
    else if (od.depth == 8)
        k_rbgs2<T, false, 8><<<g, NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2, od.segs, od.pmask2,
                                              od.nsegs, L.halt);
    else if (od.depth == 4)
        k_rbgs2<T, false, 4><<<g, NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2, od.segs, od.pmask2,
                                              od.nsegs, L.halt);
    else
        k_rbgs2<T, false, 2><<<g, NT, 0, s>>>(xin, xout, f, nullptr, d, L.nx, L.ny, L.nz, h2, od.segs, od.pmask2,
                                              od.nsegs, L.halt);
}

void launch_rbgs2(const Level &L, int level, const OrderData &od, const double *xin, double *xout, const double *f,
                  hipStream_t s) {
    launch_fused<double>(L, level, od, xin, xout, f, od.d, L.h * L.h, s);
}

void launch_rbgs2_32(const Level &L, int level, const OrderData &od, const float *xin, float *xout, const float *f,
                     hipStream_t s) {
    launch_fused<float>(L, level, od, xin, xout, f, od.d32, (float)(L.h * L.h), s);
}

void launch_rbgs2_prolong(const Level &L, const OrderData &od, const Level &C, const double *xc, const double *xin,
                          double *xout, const double *f, hipStream_t s) {
    if (od.nsegs == 0) return;
    k_rbgs2<double, true, SEG_TILES_FINE * TZ, true><<<grid8(od.nsegs), NT, 0, s>>>(
        xin, xout, f, L.code, nullptr, L.nx, L.ny, L.nz, L.h * L.h, od.segs, od.pmask2, od.nsegs, L.halt, xc, C.nx,
        C.ny, C.nz);
}

void launch_rbgs2_prolong32(const Level &L, const OrderData &od, const Level &C, const float *xc, const float *xin,
                            float *xout, const float *f, hipStream_t s) {
    if (od.nsegs == 0) return;
    k_rbgs2<float, true, SEG_TILES_FINE * TZ, true><<<grid8(od.nsegs), NT, 0, s>>>(
        xin, xout, f, L.code, nullptr, L.nx, L.ny, L.nz, (float)(L.h * L.h), od.segs, od.pmask2, od.nsegs, L.halt,
        xc, C.nx, C.ny, C.nz);
}

hipError_t launch_rbgs32(const Level &L, int level, const OrderData &od, const float *xin, float *xout,
                         const float *f, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (od.nsegs == 0) return hipSuccess;
    const float h2 = (float)(L.h * L.h);
    if (level == 0)
        return launch_fine<float>(L, od, xin, xout, f, h2, s, e0, e1);
    else if (od.cubes())
        return launch_cube<float, false>(xin, xout, f, L, od, s);
    else
        launch_coarse<float>(od.depth, xin, xout, f, od.d32, L, od, h2, s);
    return hipSuccess;
}

}  // namespace mg
