// Core of the one-workgroup multigrid call on small levels, shared by the
// per-level path (coarse.hip) and the batched phase kernels (batch.hip).
#pragma once

#include "mg_core.h"
#include "small_rule.h"
#include "smooth_core.h"

namespace mg {
namespace small {

// One fused multiply-add in T (named, so that every path rounds alike).
template <typename T>
__device__ __forceinline__ T fma_t(T a, T b, T c) {
    if constexpr (sizeof(T) == 8) return __builtin_fma(a, b, c);
    else return __builtin_fmaf(a, b, c);
}

template <typename T>
struct SmallLevels {
    int n;                 // number of levels held (ls..last)
    int nx[MAXS], ny[MAXS], nz[MAXS];
    unsigned long long mx[MAXS], mxy[MAXS];  // division magics, see qdiv
    unsigned long long mh[MAXS], mhy[MAXS];  // ... of hx = ceil(nx / 2) and hx * ny
    T h2[MAXS];            // h^2 per level
    T ih2[MAXS];           // 1/h^2 per level
    const T *d[MAXS];      // diagonal per level (global), 0 off the domain
    const T *rd[2];        // reciprocals 1/d of the first two levels (global; small_fast)
    int fast;              // the call takes small_fast
    int off[MAXS];         // LDS offset (elements) of the level's x; f and d follow
    const T *f0;           // right-hand side of level ls (global)
    T *x0;                 // iterate of level ls (global, in/out)
    int load_x;            // 1: start from x0, 0: start from zero
    const T *deep;         // matrix of the deepest level's relaxation (deep_solve), nullptr: relax it
    const int *halt;       // the solve loop's halt flag (nullable): the call does nothing when set
    int n_pre, n_post, n_cycles, n_coarse;
};

template <typename T>
struct Lv {
    T *x, *f, *d;
    int nx, ny, nz, n;
    unsigned long long mx, mxy;  // ceil(2^32 / nx), ceil(2^32 / (nx*ny))
    int hx;                      // cells of one colour per row, at most: ceil(nx / 2)
    unsigned long long mh, mhy;  // ceil(2^32 / hx), ceil(2^32 / (hx*ny))
    T h2, ih2;
};

// Division magics of a level for the host: ceil(2^32 / v).
inline unsigned long long div_magic(unsigned v) { return (0x100000000ull + v - 1) / v; }

// Exact quotient e / d for e * d < 2^32, with m = ceil(2^32 / d): the error
// of e * m / 2^32 is below e / 2^32 < 1/d, too small to reach the next integer.
__device__ __forceinline__ int qdiv(int e, unsigned long long m) {
    return (int)(((unsigned long long)(unsigned)e * m) >> 32);
}

template <typename T>
__device__ __forceinline__ void cell_ijk(const Lv<T> &L, int e, int &i, int &j, int &k) {
    k = qdiv(e, L.mxy);
    const int r = e - k * L.nx * L.ny;
    j = qdiv(r, L.mx);
    i = r - j * L.nx;
}

template <typename T>
__device__ __forceinline__ T nb_sum(const T *x, int i, int j, int k, int nx, int ny, int nz) {
    const int p = (k * ny + j) * nx + i;
    const T xm = i > 0 ? x[p - 1] : T(0);
    const T xp = i < nx - 1 ? x[p + 1] : T(0);
    const T ym = j > 0 ? x[p - nx] : T(0);
    const T yp = j < ny - 1 ? x[p + nx] : T(0);
    const T zm = k > 0 ? x[p - nx * ny] : T(0);
    const T zp = k < nz - 1 ? x[p + nx * ny] : T(0);
    return (xm + xp) + (ym + yp) + (zm + zp);
}

// The three relaxation paths below (one wave, cells in registers, slots in
// turn) are chosen by level size and thread count; each evaluates
// ((x-neighbour pair) + (y pair) + (z pair) - h^2 f) / d with h^2 f rounded
// on its own (no fused multiply-add) and the quotient correctly rounded (by
// a division, or, where a cell's diagonal stays in registers over the passes,
// from its correctly rounded reciprocal with one correction step: rb::
// div_small), so every path, for any thread count, gives the same value bit
// for bit.

// Red-black half-sweep of colour `col` over slots first, first + step, ...
// (slot m of row (j, k) is cell i = 2m + ((col + j + k) mod 2)).
template <typename T>
__device__ __forceinline__ void half_sweep(const Lv<T> &L, int col, int first, int step) {
#pragma clang fp contract(off)
    const int slots = L.hx * L.ny * L.nz;
    for (int s = first; s < slots; s += step) {
        const int k = qdiv(s, L.mhy);
        const int r = s - k * L.hx * L.ny;
        const int j = qdiv(r, L.mh);
        const int i = 2 * (r - j * L.hx) + ((col + j + k) & 1);
        if (i >= L.nx) continue;
        const int e = (k * L.ny + j) * L.nx + i;
        const T d = L.d[e];
        if (d == T(0)) continue;
        L.x[e] = (nb_sum(L.x, i, j, k, L.nx, L.ny, L.nz) - L.h2 * L.f[e]) / d;
    }
}

// Levels with at most 64 cells of one colour are relaxed by the first wave
// alone, each lane owning at most one cell per colour: its index, neighbour
// validity, diagonal and h^2 f stay in registers for all passes.  A wave's LDS
// accesses complete in order, so its half-sweeps need no workgroup barrier
// between them (the other waves wait once at the end).
constexpr int WAVE_SLOTS = 64;

template <typename T>
__device__ __forceinline__ void smooth_wave(const Lv<T> &L, int passes) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x;
    const int nxy = L.nx * L.ny;
    int e[2] = {-1, -1};
    unsigned nb[2] = {0u, 0u};  // valid neighbours: -x, +x, -y, +y, -z, +z
    T dg[2] = {T(1), T(1)}, yr[2] = {T(1), T(1)}, rhs[2] = {T(0), T(0)};
#pragma unroll
    for (int col = 0; col < 2; col++) {
        if (lane >= L.hx * L.ny * L.nz) continue;
        const int k = qdiv(lane, L.mhy);
        const int r = lane - k * L.hx * L.ny;
        const int j = qdiv(r, L.mh);
        const int i = 2 * (r - j * L.hx) + ((col + j + k) & 1);
        if (i >= L.nx) continue;
        const int c = (k * L.ny + j) * L.nx + i;
        if (L.d[c] == T(0)) continue;
        e[col] = c;
        dg[col] = L.d[c];
        yr[col] = T(1) / dg[col];
        rhs[col] = L.h2 * L.f[c];
        nb[col] = (unsigned)(i > 0) | (unsigned)(i < L.nx - 1) << 1 | (unsigned)(j > 0) << 2 |
                  (unsigned)(j < L.ny - 1) << 3 | (unsigned)(k > 0) << 4 | (unsigned)(k < L.nz - 1) << 5;
    }
    for (int p = 0; p < passes; p++)
#pragma unroll
        for (int col = 0; col < 2; col++) {
            const int c = e[col];
            if (c >= 0) {
                const unsigned m = nb[col];
                const T *x = L.x;
                const T xm = (m & 1u) ? x[c - 1] : T(0);
                const T xp = (m & 2u) ? x[c + 1] : T(0);
                const T ym = (m & 4u) ? x[c - L.nx] : T(0);
                const T yp = (m & 8u) ? x[c + L.nx] : T(0);
                const T zm = (m & 16u) ? x[c - nxy] : T(0);
                const T zp = (m & 32u) ? x[c + nxy] : T(0);
                L.x[c] = rb::div_small<T>(((xm + xp) + (ym + yp) + (zm + zp)) - rhs[col], dg[col], yr[col]);
            }
            // keep the next half-sweep's LDS reads behind this one's writes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
}

// Levels with at most two cells of one colour per thread: each thread keeps
// its cells' index, neighbour validity, diagonal and f in registers for all
// passes of the call (the same expression as half_sweep).
template <typename T, int NTH>
__device__ void smooth_regs(const Lv<T> &L, int passes) {
#pragma clang fp contract(off)
    const int slots = L.hx * L.ny * L.nz;
    const int nxy = L.nx * L.ny;
    int e[2][2];
    unsigned nb[2][2];
    T dg[2][2], yr[2][2], fv[2][2];
#pragma unroll
    for (int col = 0; col < 2; col++)
#pragma unroll
        for (int u = 0; u < 2; u++) {
            e[col][u] = -1;
            nb[col][u] = 0u;
            dg[col][u] = T(1);
            yr[col][u] = T(1);
            fv[col][u] = T(0);
            const int s = threadIdx.x + u * NTH;
            if (s >= slots) continue;
            const int k = qdiv(s, L.mhy);
            const int r = s - k * L.hx * L.ny;
            const int j = qdiv(r, L.mh);
            const int i = 2 * (r - j * L.hx) + ((col + j + k) & 1);
            if (i >= L.nx) continue;
            const int c = (k * L.ny + j) * L.nx + i;
            const T d = L.d[c];
            if (d == T(0)) continue;
            e[col][u] = c;
            dg[col][u] = d;
            yr[col][u] = T(1) / d;
            fv[col][u] = L.f[c];
            nb[col][u] = (unsigned)(i > 0) | (unsigned)(i < L.nx - 1) << 1 | (unsigned)(j > 0) << 2 |
                         (unsigned)(j < L.ny - 1) << 3 | (unsigned)(k > 0) << 4 | (unsigned)(k < L.nz - 1) << 5;
        }
    for (int p = 0; p < passes; p++)
#pragma unroll
        for (int col = 0; col < 2; col++) {
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int c = e[col][u];
                if (c < 0) continue;
                const unsigned m = nb[col][u];
                const T *x = L.x;
                const T xm = (m & 1u) ? x[c - 1] : T(0);
                const T xp = (m & 2u) ? x[c + 1] : T(0);
                const T ym = (m & 4u) ? x[c - L.nx] : T(0);
                const T yp = (m & 8u) ? x[c + L.nx] : T(0);
                const T zm = (m & 16u) ? x[c - nxy] : T(0);
                const T zp = (m & 32u) ? x[c + nxy] : T(0);
                L.x[c] = rb::div_small<T>(((xm + xp) + (ym + yp) + (zm + zp)) - L.h2 * fv[col][u], dg[col][u],
                                          yr[col][u]);
            }
            __syncthreads();
        }
}

// Red-black passes; each half-sweep visits only the cells of its colour.
// WAVE: a level of at most WAVE_SLOTS slots per colour runs on one wave with
// no block barrier (levels in LDS only; with levels in global memory every
// half-sweep ends at a block barrier).
template <typename T, int NTH, bool WAVE = true>
__device__ void smooth(const Lv<T> &L, int passes) {
    const int slots = L.hx * L.ny * L.nz;
    if (WAVE && slots <= WAVE_SLOTS) {
        if (threadIdx.x < 64) smooth_wave(L, passes);
        __syncthreads();
        return;
    }
    if (slots <= 2 * NTH) {
        smooth_regs<T, NTH>(L, passes);
        return;
    }
    for (int p = 0; p < passes; p++)
        for (int col = 0; col < 2; col++) {
            half_sweep(L, col, threadIdx.x, NTH);
            __syncthreads();
        }
}

// The deepest level's whole share of a cycle as one matrix product.  Its
// n_cycles x n_coarse passes start from zero and are linear in f, so they are
// x = M f with M formed once per hierarchy (column j: the passes applied to the
// unit right-hand side of cell j, k_deep_matrix).  16 lanes share a row, lane q
// summing columns q, q + 16, ... in order, then an exchange tree: the same sums
// for any thread count.  A cell whose right-hand side does not reach a row
// (another part of the domain, or out of the passes' reach) has a zero there and
// is left out, so that an infinity or a NaN of its stays with the cells that the
// passes would carry it to.  Taken where deep_product (small_rule.h) says so.
template <typename T>
__device__ __forceinline__ T deep_term(T m, T f, T s) {
    return fma_t<T>(m, m != T(0) ? f : T(0), s);  // (selected ahead of the chain of sums)
}

template <typename T, int NTH>
__device__ void deep_solve(const Lv<T> &L, const T *__restrict__ M) {
    const int q = threadIdx.x & 15;
    for (int row0 = 0; row0 < L.n; row0 += NTH / 16) {
        const int row = row0 + (int)(threadIdx.x >> 4);
        T s = T(0);
        if (row < L.n)
            for (int j = q; j < L.n; j += 16) s = deep_term<T>(M[row * L.n + j], L.f[j], s);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (row < L.n && q == 0) L.x[row] = L.d[row] != T(0) ? s : T(0);
    }
    __syncthreads();
}

// f_c = -(1/8) sum over active children of (L x - f); x_c = 0.
template <typename T, int NTH>
__device__ void restrict_to(const Lv<T> &L, const Lv<T> &C) {
    for (int E = threadIdx.x; E < C.n; E += NTH) {
        int I, J, K;
        cell_ijk(C, E, I, J, K);
        T s = T(0);
        if (C.d[E] != T(0)) {
#pragma unroll
            for (int c = 0; c < 8; c++) {
                const int i = 2 * I + (c & 1), j = 2 * J + ((c >> 1) & 1), k = 2 * K + (c >> 2);
                const int p = (k * L.ny + j) * L.nx + i;
                const T d = L.d[p];
                if (d != T(0))
                    s += fma_t<T>(fma_t<T>(-d, L.x[p], nb_sum(L.x, i, j, k, L.nx, L.ny, L.nz)), L.ih2, -L.f[p]);
            }
            s = -s / T(8);
        }
        C.f[E] = s;
        C.x[E] = T(0);
    }
    __syncthreads();
}

// x += P2(x_c) on active cells (weights 3/4, 1/4 per axis; 0 off the box).
template <typename T, int NTH>
__device__ void prolong_from(const Lv<T> &L, const Lv<T> &C) {
    const T w[2] = {T(0.75), T(0.25)};
    for (int e = threadIdx.x; e < L.n; e += NTH) {
        if (L.d[e] == T(0)) continue;
        int i, j, k;
        cell_ijk(L, e, i, j, k);
        const int I = i >> 1, J = j >> 1, K = k >> 1;
        const int sx = (i & 1) ? 1 : -1, sy = (j & 1) ? 1 : -1, sz = (k & 1) ? 1 : -1;
        T s = T(0);
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int a = 0; a < 2; a++) {
                    const int ci = I + a * sx, cj = J + b * sy, ck = K + c * sz;
                    T v = T(0);
                    if (ci >= 0 && ci < C.nx && cj >= 0 && cj < C.ny && ck >= 0 && ck < C.nz)
                        v = C.x[(ck * C.ny + cj) * C.nx + ci];
                    s = fma_t<T>(w[a] * w[b] * w[c], v, s);
                }
        L.x[e] += s;
    }
    __syncthreads();
}

// ---- the call on one to three levels with the cells in registers ----
// One CU issues the whole call, so its instructions and LDS cycles decide: a
// phase of the general path spends most of its instructions on cell indices,
// box-edge selects and reciprocals, once per phase and level, and its x rows
// put the cells of one colour 16 bytes apart (two-way bank conflicts).  Here
// each thread owns the same cells throughout (up to two of each colour on the
// first level A, one of each on the second, B), holds their diagonal, its
// reciprocal (formed once per hierarchy) and right-hand side in registers, and
// x lies in LDS inside a ring of zeros, A's colours in arrays of their own, so a
// relaxation is six conflict-free reads, the sum and the quotient.  The deepest
// level D is the matrix of deep_solve.  Every value is formed by the expression,
// in the order, of the general path (bit for bit).
// Levels A, D or A, B (relaxed n_coarse times, no matrix) or A, B, D; A alone,
// relaxed n_coarse times, is small_one, with up to four cells of a colour per
// thread.
// 16^3 + 8^3 + 4^3: 14 us a call at a 32^3 or 64^3 finest level and 17 us at
// 256^3, against 25 and 29 us in the general path (30 and 32 us with the
// deepest level relaxed); in a W-cycle 17 against 57 us; 17 x 9 x 13 relaxed 32
// times 22 against 25 us, 6 x 32 x 32 in a batch 35 against 99 us.  The general
// path stays for four levels and more, for single levels of more than 8192 cells
// and for blocks of fewer threads.
struct FastLds {  // offsets in elements
    int ra, xb, rb, xd, fd, end;
};

__host__ __device__ constexpr int padded(int nx, int ny, int nz) { return (nx + 2) * (ny + 2) * (nz + 2); }
// one colour of a level with its ring
__host__ __device__ constexpr int padded_half(int nx, int ny, int nz) { return padded((nx + 1) >> 1, ny, nz); }

// The LDS of the levels with these dims (A's colours come first).  direct: the
// deepest level has its matrix.
__host__ __device__ inline FastLds fast_lds(int n, bool direct, const int *nx, const int *ny, const int *nz) {
    FastLds o{};
    const bool hasb = n == 3 || (n == 2 && !direct);
    const int d = n - 1;
    o.ra = 2 * padded_half(nx[0], ny[0], nz[0]);
    o.xb = o.ra + (n > 1 ? nx[0] * ny[0] * nz[0] : 0);
    o.rb = o.xb + (hasb ? padded(nx[1], ny[1], nz[1]) : 0);
    o.xd = o.rb + (n == 3 ? nx[1] * ny[1] * nz[1] : 0);
    o.fd = o.xd + (direct ? padded(nx[d], ny[d], nz[d]) : 0);
    o.end = o.fd + (direct ? nx[d] * ny[d] * nz[d] : 0);
    return o;
}
// Whether blocks of nth threads can run these levels this way.
inline bool fast_fits(int n, bool direct, const int *nx, const int *ny, const int *nz, int nth) {
    if (n < 1 || n > 3 || (n == 3 && !direct)) return false;
    if (((nx[0] + 1) >> 1) * ny[0] * nz[0] > (n == 1 ? 4 : 2) * nth) return false;
    return n == 1 || (n == 2 && direct) || ((nx[1] + 1) >> 1) * ny[1] * nz[1] <= nth;
}

// ((x pair) + (y pair) + (z pair) - h^2 f) / d at LDS cell x (strides sy, sz).
template <typename T>
__device__ __forceinline__ T relaxed(const T *x, int sy, int sz, T h2, T f, T d, T y) {
#pragma clang fp contract(off)
    const T sum = (x[-1] + x[1]) + (x[-sy] + x[sy]) + (x[-sz] + x[sz]);
    return rb::div_small<T>(sum - h2 * f, d, y);
}

// L x - f at LDS cell x.
template <typename T>
__device__ __forceinline__ T residual_at(const T *x, int sy, int sz, T ih2, T f, T d) {
    const T sum = (x[-1] + x[1]) + (x[-sy] + x[sy]) + (x[-sz] + x[sz]);
    return fma_t<T>(fma_t<T>(-d, x[0], sum), ih2, -f);
}

// -(1/8) of the sum of the 8 children's residuals (0 on inactive ones) from r,
// whose row and plane strides are nx and nxy; b: the first child.
template <typename T>
__device__ __forceinline__ T coarse_rhs(const T *r, int b, int nx, int nxy) {
    T s = T(0);
#pragma unroll
    for (int c = 0; c < 8; c++) s += r[b + (c & 1) + ((c >> 1) & 1) * nx + (c >> 2) * nxy];
    return -s / T(8);
}

// P2 at a fine cell of parities (i, j, k): v = the parent in its ring-padded
// level of strides sy, sz.
template <typename T>
__device__ __forceinline__ T interpolated(const T *v, int i, int j, int k, int sy, int sz) {
    const T w[2] = {T(0.75), T(0.25)};
    const int ox = (i & 1) ? 1 : -1, oy = (j & 1) ? sy : -sy, oz = (k & 1) ? sz : -sz;
    T s = T(0);
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int a = 0; a < 2; a++)
                s = fma_t<T>(w[a] * w[b] * w[c], v[(a ? ox : 0) + (b ? oy : 0) + (c ? oz : 0)], s);
    return s;
}

// Cells of one slot of a level: slot s = (row m, j, k), colour c at
// i = 2m + ((c + j + k) mod 2).
struct SlotAt {
    int m, j, k;
    __device__ __forceinline__ int i(int c) const { return 2 * m + ((c + j + k) & 1); }
};
__device__ __forceinline__ SlotAt slot_at(int s, int hx, int ny, unsigned long long mh, unsigned long long mhy) {
    SlotAt t;
    t.k = qdiv(s, mhy);
    const int r = s - t.k * hx * ny;
    t.j = qdiv(r, mh);
    t.m = r - t.j * hx;
    return t;
}

// Level A: this thread's U slots, tid + u NTH, both colours.  Colour c of slot
// (m, j, k) is element (k + 1) sz + (j + 1) sy + m + 1 of the array x[c]; its x
// neighbours are the other colour's slots m - 1 + q and m + q of the row, q the
// cell's i mod 2 (for red, (j + k) mod 2; for black the other), its y and z
// neighbours the same m of the neighbouring rows.
template <typename T, int NTH, int U>
struct Finest {
    T *x[2];
    int nx, ny, hx, sy, sz, slots;
    T h2;
    int p[U];
    SlotAt at[U];
    T d[U][2], y[U][2], f[U][2];

    __device__ __forceinline__ void init(T *sm, const SmallLevels<T> &S) {
        nx = S.nx[0], ny = S.ny[0], hx = (nx + 1) >> 1, sy = hx + 2, sz = sy * (ny + 2);
        slots = hx * ny * S.nz[0];
        h2 = S.h2[0];
        x[0] = sm;
        x[1] = sm + sz * (S.nz[0] + 2);
    }
    __device__ __forceinline__ int cell(int u, int c) const {  // -1: none
        const int i = at[u].i(c);
        return (int)threadIdx.x + u * NTH < slots && i < nx ? (at[u].k * ny + at[u].j) * nx + i : -1;
    }
    // diagonals, reciprocals and right-hand sides; v: the start (0 unless load_x)
    __device__ __forceinline__ void load(const SmallLevels<T> &S, const T *__restrict__ f0, const T *__restrict__ x0,
                                         bool load_x, T (&v)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int s = (int)threadIdx.x + u * NTH;
            at[u] = slot_at(s < slots ? s : 0, hx, ny, S.mh[0], S.mhy[0]);
            p[u] = (at[u].k + 1) * sz + (at[u].j + 1) * sy + at[u].m + 1;
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int e = cell(u, c);
                d[u][c] = e >= 0 ? S.d[0][e] : T(0);
                y[u][c] = e >= 0 ? S.rd[0][e] : T(0);
                f[u][c] = e >= 0 ? f0[e] : T(0);
                v[u][c] = e >= 0 && load_x ? x0[e] : T(0);
            }
        }
    }
    __device__ __forceinline__ T sum(int u, int c) const {
#pragma clang fp contract(off)
        const T *o = x[c ^ 1];
        const int l = p[u] - 1 + ((c + at[u].j + at[u].k) & 1);
        return (o[l] + o[l + 1]) + (o[p[u] - sy] + o[p[u] + sy]) + (o[p[u] - sz] + o[p[u] + sz]);
    }
    __device__ __forceinline__ T relaxed(int u, int c) const {
#pragma clang fp contract(off)
        return rb::div_small<T>(sum(u, c) - h2 * f[u][c], d[u][c], y[u][c]);
    }
    __device__ __forceinline__ void smooth(int passes) {
        for (int n = 0; n < passes; n++)
#pragma unroll
            for (int c = 0; c < 2; c++) {
#pragma unroll
                for (int u = 0; u < U; u++)
                    if (d[u][c] != T(0)) x[c][p[u]] = relaxed(u, c);
                __syncthreads();
            }
    }
    __device__ __forceinline__ T residual(int u, int c, T ih2) const {
        return fma_t<T>(fma_t<T>(-d[u][c], x[c][p[u]], sum(u, c)), ih2, -f[u][c]);
    }
    __device__ __forceinline__ void set(const T (&v)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int c = 0; c < 2; c++)
                if (cell(u, c) >= 0) x[c][p[u]] = v[u][c];
    }
    __device__ __forceinline__ void store(T *__restrict__ x0) const {
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int e = cell(u, c);
                if (e >= 0) x0[e] = x[c][p[u]];
            }
    }
};

// A single level, relaxed n_coarse times.
template <typename T, int NTH, int U>
__device__ __forceinline__ void small_one(T *sm, const SmallLevels<T> &S, const T *__restrict__ f0,
                                          T *__restrict__ x0, bool load_x) {
    Finest<T, NTH, U> A;
    T v[U][2];
    A.init(sm, S);
    A.load(S, f0, x0, load_x, v);
    for (int e = threadIdx.x; e < 2 * A.sz * (S.nz[0] + 2); e += NTH) sm[e] = T(0);
    __syncthreads();
    if (load_x) {
        A.set(v);
        __syncthreads();
    }
    A.smooth(S.n_coarse);
    A.store(x0);
}

template <typename T, int NTH>
__device__ __forceinline__ void small_fast(T *sm, const SmallLevels<T> &S, const T *__restrict__ f0,
                                           T *__restrict__ x0, bool load_x) {
    if (S.n == 1) {
        if (((S.nx[0] + 1) >> 1) * S.ny[0] * S.nz[0] <= 2 * NTH) small_one<T, NTH, 2>(sm, S, f0, x0, load_x);
        else small_one<T, NTH, 4>(sm, S, f0, x0, load_x);
        return;
    }
    constexpr int U = 2;
    const int tid = threadIdx.x;
    const bool direct = S.deep != nullptr;
    const bool three = S.n == 3, hasb = three || !direct;
    const FastLds o = fast_lds(S.n, direct, S.nx, S.ny, S.nz);
    T *const ra = sm + o.ra, *const xb = sm + o.xb, *const rbs = sm + o.rb, *const xd = sm + o.xd,
             *const fd = sm + o.fd;
    Finest<T, NTH, U> A;
    {
        T v[U][2];
        A.init(sm, S);
        A.load(S, f0, x0, load_x, v);
        for (int e = tid; e < o.end; e += NTH) sm[e] = T(0);
        __syncthreads();
        if (load_x) {
            A.set(v);
            __syncthreads();
        }
    }
    const int nxa = A.nx, nxya = A.nx * A.ny;
    // level B: one slot; its first child in A's cells
    int pb[2] = {0, 0}, eb[2] = {0, 0}, cb[2] = {0, 0};
    SlotAt tb{0, 0, 0};
    T db[2] = {T(0), T(0)}, yb[2] = {T(0), T(0)}, fb[2] = {T(0), T(0)};
    const int nxb = S.nx[1], nyb = S.ny[1], nxyb = nxb * nyb;
    const int syb = nxb + 2, szb = syb * (nyb + 2);
    if (hasb) {
        const int hxb = (nxb + 1) >> 1;
        if (tid < hxb * nyb * S.nz[1]) {
            tb = slot_at(tid, hxb, nyb, S.mh[1], S.mhy[1]);
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int i = tb.i(c);
                if (i >= nxb) continue;
                eb[c] = (tb.k * nyb + tb.j) * nxb + i;
                pb[c] = (tb.k + 1) * szb + (tb.j + 1) * syb + i + 1;
                cb[c] = 2 * tb.k * nxya + 2 * tb.j * nxa + 2 * i;
                db[c] = S.d[1][eb[c]];
                yb[c] = S.rd[1][eb[c]];
            }
        }
    }
    // level D: the matrix (in registers for a level of up to 64 cells)
    const int ld = S.n - 1, nd = S.nx[ld] * S.ny[ld] * S.nz[ld];
    const int q = tid & 15;
    T mreg[4] = {T(0), T(0), T(0), T(0)};
    const bool inreg = direct && nd <= 64 && NTH >= 1024;
    if (inreg && (tid >> 4) < nd)
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (q + 16 * k < nd) mreg[k] = S.deep[(tid >> 4) * nd + q + 16 * k];
    const T h2b = S.h2[1];
    auto smooth_b = [&](int passes) {
        for (int n = 0; n < passes; n++)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                if (db[c] != T(0)) xb[pb[c]] = relaxed<T>(xb + pb[c], syb, szb, h2b, fb[c], db[c], yb[c]);
                __syncthreads();
            }
    };
    // D's right-hand side from r of the level above (row and plane strides fx, fxy)
    const int nxd = S.nx[ld], nyd = S.ny[ld], nxyd = nxd * nyd, syd = nxd + 2, szd = syd * (nyd + 2);
    auto solve_d = [&](const T *r, int fx, int fxy) {
        for (int e = tid; e < nd; e += NTH) {
            const int k = qdiv(e, S.mxy[ld]), r2 = e - k * nxyd, j = qdiv(r2, S.mx[ld]), i = r2 - j * nxd;
            fd[e] = S.d[ld][e] != T(0) ? coarse_rhs<T>(r, 2 * k * fxy + 2 * j * fx + 2 * i, fx, fxy) : T(0);
        }
        __syncthreads();
        for (int row0 = 0; row0 < nd; row0 += NTH / 16) {
            const int row = row0 + (tid >> 4);
            T s = T(0);
            if (row < nd) {
                if (inreg) {
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        if (q + 16 * k < nd) s = deep_term<T>(mreg[k], fd[q + 16 * k], s);
                } else {
                    for (int j = q; j < nd; j += 16) s = deep_term<T>(S.deep[row * nd + j], fd[j], s);
                }
            }
#pragma unroll
            for (int w = 8; w > 0; w >>= 1) s += __shfl_xor(s, w);
            if (row < nd && q == 0 && S.d[ld][row] != T(0)) {
                const int k = qdiv(row, S.mxy[ld]), r2 = row - k * nxyd, j = qdiv(r2, S.mx[ld]), i = r2 - j * nxd;
                xd[(k + 1) * szd + (j + 1) * syd + i + 1] = s;
            }
        }
        __syncthreads();
    };
    A.smooth(S.n_pre);
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int c = 0; c < 2; c++)
            if (A.d[u][c] != T(0)) ra[A.cell(u, c)] = A.residual(u, c, S.ih2[0]);
    __syncthreads();
    if (hasb) {
#pragma unroll
        for (int c = 0; c < 2; c++)
            if (db[c] != T(0)) fb[c] = coarse_rhs<T>(ra, cb[c], nxa, nxya);
        if (three) {
            for (int n = 0; n < S.n_cycles; n++) {  // (x starts at zero, later visits go on from it)
                smooth_b(S.n_pre);
#pragma unroll
                for (int c = 0; c < 2; c++)
                    if (db[c] != T(0)) rbs[eb[c]] = residual_at<T>(xb + pb[c], syb, szb, S.ih2[1], fb[c], db[c]);
                __syncthreads();
                solve_d(rbs, nxb, nxyb);
#pragma unroll
                for (int c = 0; c < 2; c++)
                    if (db[c] != T(0)) {
                        const int i = tb.i(c);
                        xb[pb[c]] += interpolated<T>(
                            xd + ((tb.k >> 1) + 1) * szd + ((tb.j >> 1) + 1) * syd + (i >> 1) + 1, i, tb.j, tb.k, syd, szd);
                    }
                __syncthreads();
                smooth_b(S.n_post);
            }
        } else {
            for (int n = 0; n < S.n_cycles; n++) smooth_b(S.n_coarse);
        }
    } else {
        solve_d(ra, nxa, nxya);
    }
    {
        const T *xc = hasb ? xb : xd;
        const int syc = hasb ? syb : syd, szc = hasb ? szb : szd;
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int c = 0; c < 2; c++)
                if (A.d[u][c] != T(0)) {
                    const int i = A.at[u].i(c), j = A.at[u].j, k = A.at[u].k;
                    A.x[c][A.p[u]] += interpolated<T>(
                        xc + ((k >> 1) + 1) * szc + ((j >> 1) + 1) * syc + (i >> 1) + 1, i, j, k, syc, szc);
                }
        __syncthreads();
    }
    A.smooth(S.n_post);
    A.store(x0);
}

// One call MG(ls) for the levels held in S, all resident at `sm`: in LDS
// (WAVE: the one-wave path relies on a wave's in-order LDS accesses), or in
// a global-memory area of the block's own (!WAVE: block barriers only); f0 is
// level ls's right-hand side and x0 its iterate (in/out), started from zero
// unless load_x.  Called by all NTH threads of a block.
template <typename T, int NTH, bool WAVE = true>
__device__ void small_tail(T *sm, const SmallLevels<T> &S, const T *f0, T *x0, bool load_x) {
    // level descriptors live in LDS (dynamic indexing without private memory)
    __shared__ int s_nx[MAXS], s_ny[MAXS], s_nz[MAXS], s_off[MAXS];
    __shared__ unsigned long long s_mx[MAXS], s_mxy[MAXS], s_mh[MAXS], s_mhy[MAXS];
    __shared__ T s_h2[MAXS], s_ih2[MAXS];
    __shared__ const T *s_d[MAXS];
    if (threadIdx.x < (unsigned)S.n) {
        const int l = threadIdx.x;
        s_nx[l] = S.nx[l];
        s_ny[l] = S.ny[l];
        s_nz[l] = S.nz[l];
        s_off[l] = S.off[l];
        s_mx[l] = S.mx[l];
        s_mxy[l] = S.mxy[l];
        s_mh[l] = S.mh[l];
        s_mhy[l] = S.mhy[l];
        s_h2[l] = S.h2[l];
        s_ih2[l] = S.ih2[l];
        s_d[l] = S.d[l];
    }
    __syncthreads();
    auto level = [&](int l) {
        Lv<T> v;
        v.nx = s_nx[l];
        v.ny = s_ny[l];
        v.nz = s_nz[l];
        v.n = v.nx * v.ny * v.nz;
        v.mx = s_mx[l];
        v.mxy = s_mxy[l];
        v.hx = (v.nx + 1) >> 1;
        v.mh = s_mh[l];
        v.mhy = s_mhy[l];
        v.x = sm + s_off[l];
        v.f = v.x + v.n;
        v.d = v.f + v.n;
        v.h2 = s_h2[l];
        v.ih2 = s_ih2[l];
        return v;
    };
    // Copy-in: every level's cells as one flat range, U elements per thread
    // loaded before any is stored, so that their global loads overlap.
    auto cells = [&](int l) { return s_nx[l] * s_ny[l] * s_nz[l]; };
    int tot = 0;
    for (int l = 0; l < S.n; l++) tot += cells(l);
    constexpr int U = 8;
    for (int q0 = threadIdx.x; q0 < tot; q0 += U * NTH) {
        T dv[U], fv[U], xv[U];
        int lv[U], ev[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            int l = 0, e = q0 + u * NTH;
            lv[u] = -1;
            if (e >= tot) continue;
            while (e >= cells(l)) {
                e -= cells(l);
                l++;
            }
            lv[u] = l;
            ev[u] = e;
            dv[u] = s_d[l][e];
            fv[u] = l == 0 ? f0[e] : T(0);
            xv[u] = (l == 0 && load_x) ? x0[e] : T(0);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (lv[u] < 0) continue;
            const Lv<T> v = level(lv[u]);
            v.d[ev[u]] = dv[u];
            v.x[ev[u]] = xv[u];
            if (lv[u] == 0) v.f[ev[u]] = fv[u];
        }
    }
    __syncthreads();
    // iterative form of the recursion MG(l): pre-smooth, restrict, N_cycles x
    // MG(l+1) from zero, prolong, post-smooth; the deepest level is relaxed.
    // visits: 3 bits per level (N_cycles <= 4).
    const int last = S.n - 1;
    const bool direct = last > 0 && S.deep;  // (a single level may start from a non-zero iterate)
    unsigned visits = 0;
    int l = 0;
    bool down = true;
    while (true) {
        if (down) {
            if (l == last) {
                if (direct) deep_solve<T, NTH>(level(l), S.deep);
                else smooth<T, NTH, WAVE>(level(l), S.n_coarse);
                down = false;
                continue;
            }
            smooth<T, NTH, WAVE>(level(l), S.n_pre);
            restrict_to<T, NTH>(level(l), level(l + 1));
            visits &= ~(7u << (3 * (l + 1)));
            l++;
            continue;
        }
        if (l == 0) break;
        const unsigned vc = ((visits >> (3 * l)) & 7u) + 1u;
        visits = (visits & ~(7u << (3 * l))) | (vc << (3 * l));
        if ((int)vc < S.n_cycles && !(direct && l == last)) {  // (the matrix holds all its visits)
            down = true;
            continue;
        }
        prolong_from<T, NTH>(level(l - 1), level(l));
        smooth<T, NTH, WAVE>(level(l - 1), S.n_post);
        l--;
    }
    const Lv<T> top = level(0);
    for (int e = threadIdx.x; e < top.n; e += NTH) x0[e] = top.x[e];
    __syncthreads();
}

}  // namespace small
}  // namespace mg
