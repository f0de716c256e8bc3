// Kernels on the 8^3-cell blocks of AMR levels: operator apply, residual and
// red-black half-sweep (one workgroup per block, block plus a one-cell face and
// edge halo staged in LDS), restriction, prolongation, coarse-fine ghost fill,
// refluxing and per-problem norm reductions.
#include "common.h"
#include <type_traits>
#include "stencil.h"
#include "sweep.h"

namespace ohm {

namespace {

constexpr int TW = NB + 2;             // tile edge with a one-cell halo
constexpr int TC = TW * TW * TW;       // tile cells

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous
// run of blocks (blocks are in Z-order, so a compact region whose halo stays
// in that XCD's L2).
__device__ __forceinline__ int xcd_block(int w, int n)
{
    int q = n / NXCD, r = n % NXCD;
    int x = w % NXCD, i = w / NXCD;
    return x * q + min(x, r) + i;
}

// The loads in front of a block's fields -- its problem, that problem's active
// flag, its neighbours -- are what a small launch waits for, one after the
// other: a handle of one problem passes no problem table, and the neighbour
// entries are requested before the flag is known.
__device__ __forceinline__ int problem_of(const int *prob_of, int b) { return prob_of ? prob_of[b] : 0; }
__device__ __forceinline__ int load_nbr(const int *nbr_tab, int b)
{
    return threadIdx.x < 27 ? nbr_tab[27 * (long long)b + threadIdx.x] : 0;
}

__device__ __forceinline__ int side(int c) { return c < 0 ? -1 : (c >= NB ? 1 : 0); }

// B (3 components) and eta of block b plus the one-cell halo into LDS: each of
// the first 200 (500) of 256 (512) threads owns a tile column (x, y) and five
// (two) consecutive z, issues all its global loads, then stores them (ghost
// blocks for negative neighbour entries, zeros for absent corner blocks)
template <typename T, int THREADS>
__device__ __forceinline__ void load_tile_b_eta(T (*sB)[TC], T *sE, const T *f, const T *g, long long cs,
                                                long long gcs, const T *eta, const T *etag, const int *nbr)
{
    constexpr int EACH = THREADS == 512 ? 2 : 5;
    const int u = threadIdx.x;
    if (u >= TW / EACH * TW * TW) return;
    const int col = u % (TW * TW), zh = u / (TW * TW);
    const int x = col % TW - 1, y = col / TW - 1;
    const int sx = side(x), sy = side(y);
    const int lxy = (x - NB * sx) + NB * (y - NB * sy);
    const int sxy = (sx + 1) + 3 * (sy + 1);
    T v[EACH][4];
#pragma unroll
    for (int k = 0; k < EACH; ++k) {
        const int z = EACH * zh + k - 1, sz = side(z);
        const int n = nbr[sxy + 9 * (sz + 1)];
        const int li = lxy + NB * NB * (z - NB * sz);
        if (n >= 0) {
            const long long gi = (long long)n * NC + li;
            v[k][0] = f[gi];
            v[k][1] = f[cs + gi];
            v[k][2] = f[2 * cs + gi];
            v[k][3] = eta[gi];
        } else if (n != NBR_NONE) {
            const long long gi = (long long)(-1 - n) * NC + li;
            v[k][0] = g[gi];
            v[k][1] = g[gcs + gi];
            v[k][2] = g[2 * gcs + gi];
            v[k][3] = etag[gi];
        } else {
            v[k][0] = v[k][1] = v[k][2] = v[k][3] = T(0);
        }
    }
#pragma unroll
    for (int k = 0; k < EACH; ++k) {
        const int t = col + TW * TW * (EACH * zh + k);
        sB[0][t] = v[k][0];
        sB[1][t] = v[k][1];
        sB[2][t] = v[k][2];
        sE[t] = v[k][3];
    }
}

// THREADS 256 or 512: two cells or one a thread (see launch_blk_stencil)
template <typename T, int MODE, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_blk_stencil(int nblk, const int *__restrict__ nbr_tab, const int *__restrict__ prob_of,
              const uint8_t *__restrict__ cov_zero, const int *__restrict__ active,
              const double *__restrict__ inv_h2_p,
            const double *__restrict__ coef_p, double coef_v,
              const T *__restrict__ B, const T *__restrict__ Bg, long long cs, long long gcs,
              const T *__restrict__ S, const T *__restrict__ eta, const T *__restrict__ etag,
              T *__restrict__ out, int colour, double *__restrict__ partials, StencilDots dots,
              const int *__restrict__ dense_map, const DenseProbDev *__restrict__ dp, long long ccs)
{
    __shared__ __align__(8) T sB[3][TC];
    __shared__ T sE[1][TC];
    __shared__ int snbr[27];
    const int b = xcd_block(blockIdx.x, nblk);
    const int mine = load_nbr(nbr_tab, b);
    const int pr = problem_of(prob_of, b);
    if (active && !active[pr]) {
        if (MODE == MODE_APPLY && threadIdx.x < dots.ndot) dots.dot_part[(long long)b * dots.ndot + threadIdx.x] = 0.0;
        return;
    }
    if (threadIdx.x < 27) snbr[threadIdx.x] = mine;
    __syncthreads();
    load_tile_b_eta<T, THREADS>(sB, sE[0], B, Bg, cs, gcs, eta, etag, snbr);
    // values read per cell after the stencil (S, or the other vector of the
    // first fused dot product that has one), loaded with the tile so that
    // their latency overlaps it
    constexpr bool HAS_S = MODE != MODE_APPLY;   // MODE_MEAN: the old value of out
    constexpr int H = NC / THREADS;
    T pS[H][3];
    double pY[H][3];
    const long long g0 = (long long)b * NC + threadIdx.x;
    int qy = -1;
    if (HAS_S) {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) pS[h][c] = (MODE == MODE_MEAN ? out : S)[c * cs + g0 + THREADS * h];
    }
    if (MODE == MODE_APPLY) {
        for (int q = dots.ndot - 1; q >= 0; --q)
            if (dots.dot_y[q]) qy = q;
        if (qy >= 0)
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int c = 0; c < 3; ++c) pY[h][c] = dots.dot_y[qy][c * cs + g0 + THREADS * h];
    }
    __syncthreads();
    const T cih2 = T(coef_of(coef_p[pr], coef_v)) * T(inv_h2_p[pr]);
    const T c8 = cih2 * T(0.125), c2 = cih2 * T(0.5);
    const uint8_t cov = cov_zero ? cov_zero[b] : 0;
    T o[H][3];   // outputs kept for the fused dot products, restriction and norms
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int cell = threadIdx.x + THREADS * h;
        const int x = cell & 7, y = (cell >> 3) & 7, z = cell >> 6;
        const int p = (x + 1) + TW * ((y + 1) + TW * (z + 1));
        const bool zero = (cov >> ((x >> 2) + 2 * (y >> 2) + 4 * (z >> 2))) & 1;
        const long long gi = g0 + THREADS * h;
        T dvs[3], als[3];
        divF_all<T, TW>(sB[0], sB[1], sB[2], sE[0], p, dvs, als);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T LB = fma(c8, dvs[c], sB[c][p]);
            if (MODE == MODE_APPLY) {
                o[h][c] = zero ? T(0) : LB;
                out[c * cs + gi] = o[h][c];
            } else if (MODE == MODE_MEAN) {
                out[c * cs + gi] = T(0.5) * (pS[h][c] + LB);
            } else if (MODE == MODE_RESID_RESTRICT) {
                o[h][c] = zero ? T(0) : pS[h][c] - LB;
            } else if (MODE == MODE_RESID) {
                o[h][c] = zero ? T(0) : pS[h][c] - LB;
                if (out) out[c * cs + gi] = o[h][c];
            } else {  // smoother half-sweep
                T v = sB[c][p];
                if (in_colour(x, y, z, colour)) v = relax_point(v, pS[h][c], dvs[c], als[c], c8, c2);
                out[c * cs + gi] = v;
            }
        }
    }
    if (MODE == MODE_APPLY && dots.ndot > 0) {
        // column (x, y) of the block, plane by plane, then the 64 columns (the
        // order of the marching stencil): a plane's products of each column go
        // through LDS, where the tile is no longer needed
        double *col = (double *)sB;
        __syncthreads();
        for (int q = 0; q < dots.ndot; ++q)
#pragma unroll
            for (int h = 0; h < H; ++h) {
                double acc = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double y = q == qy ? pY[h][c]
                                     : (dots.dot_y[q] ? dots.dot_y[q][c * cs + g0 + THREADS * h] : (double)o[h][c]);
                    acc = fma((double)o[h][c], y, acc);
                }
                col[NC * q + threadIdx.x + THREADS * h] = acc;
            }
        __syncthreads();
        const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
        if (q < dots.ndot) {
            double a = col[NC * q + lane];
#pragma unroll
            for (int z = 1; z < NB; ++z) a += col[NC * q + lane + 64 * z];
            for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
            if (lane == 0) dots.dot_part[(long long)b * dots.ndot + q] = a;
        }
    }
    if (MODE == MODE_RESID_RESTRICT) {
        // r through LDS (the tile is no longer needed), then the mean of the 8
        // children of each coarse cell in the order of the restriction kernel
        __syncthreads();
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) sB[c][threadIdx.x + THREADS * h] = o[h][c];
        __syncthreads();
        if (threadIdx.x < 64) {
            const int t = threadIdx.x;
            const int i = t & 3, j = (t >> 2) & 3, k = t >> 4;
            const DenseProbDev q = dp[pr];
            const long long cidx = dense_map[b] + i + (long long)q.nx * (j + (long long)q.ny * k);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                T a = T(0);
#pragma unroll
                for (int dz = 0; dz < 2; ++dz)
#pragma unroll
                    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                        for (int dx = 0; dx < 2; ++dx) a += sB[c][(2 * i + dx) + NB * ((2 * j + dy) + NB * (2 * k + dz))];
                out[c * ccs + cidx] = a * T(0.125);
            }
        }
    }
    if (MODE == MODE_RESID && partials) {
        // r through LDS (the tile is no longer needed); a wavefront takes a sum
        // or a maximum, each lane up a column of the block, then the 64 columns
        // (1 or 2 of the 6 reductions over lanes a wavefront.  All six in every
        // one, plane by plane, us: FP64 1,331 blocks 24.6 instead of 19.5, 4,096
        // blocks 59 instead of 46; FP32 21.3 instead of 14.4, 47 instead of 28)
        __syncthreads();
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) sB[c][threadIdx.x + THREADS * h] = o[h][c];
        __syncthreads();
        const int lane = threadIdx.x & 63;
        for (int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); k < 6; k += THREADS / 64) {
            const T *r = sB[k % 3] + lane;
            const bool sum = k < 3;
            double v = 0.0;
#pragma unroll
            for (int z = 0; z < NB; ++z) {
                const double x = (double)r[64 * z];
                v = sum ? fma(x, x, v) : fmax(v, fabs(x));
            }
            for (int off = 32; off > 0; off >>= 1) {
                const double w = __shfl_down(v, off, 64);
                v = sum ? v + w : fmax(v, w);
            }
            if (lane == 0) partials[6 * (long long)b + k] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// Fused red-black sweep on the blocks of a level whose blocks have all 26
// neighbours (the tile body is in sweep.h, shared with the dense levels)
// ---------------------------------------------------------------------------
struct BlockAddr {
    static constexpr bool ghosts = false;
    const int *nbr;   // 27 neighbour entries of the block (LDS)
    int b;
    __device__ __forceinline__ long long at(int x, int y, int z) const
    {
        const int sx = side(x), sy = side(y), sz = side(z);
        const int n = nbr[(sx + 1) + 3 * (sy + 1) + 9 * (sz + 1)];
        return (long long)n * NC + (x - NB * sx) + NB * ((y - NB * sy) + NB * (z - NB * sz));
    }
};

// Same, on a level whose neighbour entries may name coarse-fine ghost blocks
// (never absent ones); at() is used for level cells only.
template <typename T>
struct GhostBlockAddr {
    static constexpr bool ghosts = true;
    const int *nbr;
    const T *G;       // ghost blocks, component stride gcs
    long long gcs;
    const T *EG;      // resistivity of the ghost blocks
    __device__ __forceinline__ int entry(int x, int y, int z) const
    {
        return nbr[(side(x) + 1) + 3 * (side(y) + 1) + 9 * (side(z) + 1)];
    }
    __device__ __forceinline__ int local(int x, int y, int z) const
    {
        const int sx = side(x), sy = side(y), sz = side(z);
        return (x - NB * sx) + NB * ((y - NB * sy) + NB * (z - NB * sz));
    }
    __device__ __forceinline__ long long at(int x, int y, int z) const
    {
        return (long long)entry(x, y, z) * NC + local(x, y, z);
    }
};

// DIRECT (plain FP64 sweeps, MODE 0): the tile is staged by loads that write
// LDS directly instead of passing through registers.
// MODE 0: sweep B -> out; 1: zero input (B not read); 2: sweep of B plus the
// prolonged correction from the first dense level (coarse), B -> out; MODE 3
// and 4 as 0 and 1 on a level with coarse-fine ghost blocks (Bg, etag).  With
// O64 (MODE 0 or 2 of an FP32 sweep) the result is written as FP64.
template <typename T, int MODE, bool O64, bool DIRECT, typename Tl>
__global__ void __launch_bounds__(Tl::THREADS)
k_blk_sweep(int nblk, const int *__restrict__ nbr_tab, const int *__restrict__ prob_of,
            const int *__restrict__ active, const double *__restrict__ inv_h2_p,
            const double *__restrict__ coef_p, double coef_v,
            const T *__restrict__ B, long long cs, const T *__restrict__ S, const T *__restrict__ eta,
            void *__restrict__ out, const int *__restrict__ ijk, const DenseProbDev *__restrict__ dp,
            const T *__restrict__ coarse, long long ccs, const T *__restrict__ Bg, long long gcs,
            const T *__restrict__ etag)
{
    using TO = typename std::conditional<O64, double, T>::type;
    using Addr = typename std::conditional<(MODE >= 3), GhostBlockAddr<T>, BlockAddr>::type;
    using Part = typename std::conditional<Tl::whole, Addr, PartAddr<Addr>>::type;
    using Coarse = typename std::conditional<MODE == 2, TileCoarse<T, Tl>, NoCoarse<T>>::type;
    constexpr int TS = Tl::N + (DIRECT && Tl::whole ? 64 : 0);
    __shared__ T sB[3][TS];
    __shared__ T sE[TS];
    __shared__ T sC[MODE == 2 ? 3 * Tl::NCOARSE : 1];
    __shared__ int snbr[27];
    const int w = xcd_block(blockIdx.x, nblk * Tl::PARTS), b = w / Tl::PARTS, part = w % Tl::PARTS;
    const int mine = load_nbr(nbr_tab, b);
    const int pr = problem_of(prob_of, b);
    if (active && !active[pr]) return;
    if (threadIdx.x < 27) snbr[threadIdx.x] = mine;
    __syncthreads();
    const T cih2 = T(coef_of(coef_p[pr], coef_v)) * T(inv_h2_p[pr]);
    Part A;
    if constexpr (MODE >= 3) static_cast<Addr &>(A) = Addr{snbr, Bg, gcs, etag};
    else static_cast<Addr &>(A) = Addr{snbr, b};
    if constexpr (!Tl::whole) A.y0 = Tl::y0(part), A.z0 = Tl::z0(part);
    Coarse cor;
    if constexpr (MODE == 2)
        cor = {coarse, ccs, dp[pr], 4 * ijk[3 * b] - 2, 4 * ijk[3 * b + 1] - 2 + Tl::y0(part) / 2,
               4 * ijk[3 * b + 2] - 2 + Tl::z0(part) / 2, sC, {}};
    fused_sweep_tile<T, MODE == 1 || MODE == 4, Part, Coarse, TO, Tl, TS, DIRECT>(A, B, cs, S, eta, (TO *)out, cih2,
                                                                                  sB, sE, cor);
}

// residual + restriction to the first dense level by parts of the blocks of a
// complete level 0
template <typename T, typename Tl>
__global__ void __launch_bounds__(Tl::THREADS)
k_blk_down(int nblk, const int *__restrict__ nbr_tab, const int *__restrict__ prob_of, const int *__restrict__ active,
           const double *__restrict__ inv_h2_p, const double *__restrict__ coef_p, double coef_v, const T *B, long long cs,
           const T *__restrict__ S, const T *__restrict__ eta, const int *__restrict__ dense_map,
           const DenseProbDev *__restrict__ dp, T *__restrict__ coarse, long long ccs)
{
    using Dn = DownTile<Tl>;
    __shared__ T sB[3][Dn::N];
    __shared__ T sE[Dn::N];
    __shared__ T sR[3][Dn::CELLS];
    __shared__ int snbr[27];
    const int w = xcd_block(blockIdx.x, nblk * Tl::PARTS), b = w / Tl::PARTS, part = w % Tl::PARTS;
    const int mine = load_nbr(nbr_tab, b);
    const int pr = problem_of(prob_of, b);
    if (active && !active[pr]) return;
    if (threadIdx.x < 27) snbr[threadIdx.x] = mine;
    __syncthreads();
    PartAddr<BlockAddr> A;
    static_cast<BlockAddr &>(A) = BlockAddr{snbr, b};
    A.y0 = Tl::y0(part), A.z0 = Tl::z0(part);
    down_tile<T, false, Tl>(A, const_cast<T *>(B), cs, S, eta, T(coef_of(coef_p[pr], coef_v)) * T(inv_h2_p[pr]), sB, sE, sR);
    if (threadIdx.x < 3 * Dn::NC8) {
        const int c = threadIdx.x / Dn::NC8, m = threadIdx.x % Dn::NC8;
        const int i = m & 3, j = A.y0 / 2 + (m >> 2) % (Tl::TY / 2), k = A.z0 / 2 + m / (2 * Tl::TY);
        const DenseProbDev q = dp[pr];
        coarse[c * ccs + dense_map[b] + i + (long long)q.nx * (j + (long long)q.ny * k)] = restrict_part<T, Tl>(sR[c], m);
    }
}

// ---------------------------------------------------------------------------
// restriction: fine block -> the octant of its parent block (AMR levels), and
// level-0 block -> the first dense level
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64)
k_restrict_blk(int nfine, const int *__restrict__ parent, const int *__restrict__ octant,
               const int *__restrict__ fprob, const int *__restrict__ active, const T *__restrict__ fine,
               long long fcs, T *__restrict__ coarse, long long ccs, int ncomp)
{
    const int b = xcd_block(blockIdx.x, nfine);
    if (active && !active[problem_of(fprob, b)]) return;
    const int t = threadIdx.x;          // 4^3 coarse cells of the octant
    const int i = t & 3, j = (t >> 2) & 3, k = t >> 4;
    const int o = octant[b];
    const int ci = 4 * (o & 1) + i, cj = 4 * ((o >> 1) & 1) + j, ck = 4 * (o >> 2) + k;
    const long long cidx = (long long)parent[b] * NC + ci + NB * (cj + NB * ck);
    for (int c = 0; c < ncomp; ++c) {
        const T *f = fine + c * fcs + (long long)b * NC;
        T s = T(0);
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) s += f[(2 * i + dx) + NB * ((2 * j + dy) + NB * (2 * k + dz))];
        coarse[c * ccs + cidx] = s * T(0.125);
    }
}

template <typename T>
__global__ void __launch_bounds__(64)
k_restrict_blk0_dense(int nblk, const int *__restrict__ dense_map, const int *__restrict__ prob_of,
                      const DenseProbDev *__restrict__ dp, const int *__restrict__ active,
                      const T *__restrict__ fine, long long fcs, T *__restrict__ coarse, long long ccs,
                      int ncomp)
{
    const int b = xcd_block(blockIdx.x, nblk);
    const int pr = problem_of(prob_of, b);
    if (active && !active[pr]) return;
    const int t = threadIdx.x;
    const int i = t & 3, j = (t >> 2) & 3, k = t >> 4;
    const DenseProbDev q = dp[pr];
    const long long cidx = dense_map[b] + i + (long long)q.nx * (j + (long long)q.ny * k);
    for (int c = 0; c < ncomp; ++c) {
        const T *f = fine + c * fcs + (long long)b * NC;
        T s = T(0);
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) s += f[(2 * i + dx) + NB * ((2 * j + dy) + NB * (2 * k + dz))];
        coarse[c * ccs + cidx] = s * T(0.125);
    }
}

// ---------------------------------------------------------------------------
// prolongation (cell-centred trilinear, 27/9/3/1 over 64) into fine blocks or
// ghost blocks from their parent block (and its neighbours) one level coarser.
// A chain of three loads (parent, neighbour, values), each requested for the
// whole block at once and the values added to ahead of it: 2,240 FP64 ghost
// blocks 10.8 -> 9.3 us, a correction added to 1,232 blocks 9.1 -> 8.4.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_prolong_blk(int nfine, const int *__restrict__ parent, const int *__restrict__ octant,
              const int *__restrict__ fprob, const int *__restrict__ active, const int *__restrict__ cnbr,
              const T *__restrict__ coarse, long long ccs, T *fine, long long fcs, int ncomp, int accumulate)
{
    // coarse region of the octant plus a one-cell halo: 6^3 cells
    __shared__ T sc[3][216];
    const int b = xcd_block(blockIdx.x, nfine);
    if (active && !active[problem_of(fprob, b)]) return;
    const int pb = parent[b], o = octant[b];
    // the values that are added to, two cells a thread (three components at most)
    T old[2][3];
    if (accumulate)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) old[h][c] = fine[min(c, ncomp - 1) * fcs + (long long)b * NC + threadIdx.x + 256 * h];
    {
        const int t = min((int)threadIdx.x, 215);
        const int x = 4 * (o & 1) - 1 + t % 6, y = 4 * ((o >> 1) & 1) - 1 + (t / 6) % 6, z = 4 * (o >> 2) - 1 + t / 36;
        const int sx = side(x), sy = side(y), sz = side(z);
        const int n = cnbr[27 * (long long)pb + (sx + 1) + 3 * (sy + 1) + 9 * (sz + 1)];
        const long long li = (long long)max(n, 0) * NC + (x - NB * sx) + NB * ((y - NB * sy) + NB * (z - NB * sz));
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T v = coarse[min(c, ncomp - 1) * ccs + li];
            sc[c][t] = n >= 0 ? v : T(0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int cell = threadIdx.x + 256 * h;
        const int x = cell & 7, y = (cell >> 3) & 7, z = cell >> 6;
        // parent cell in the 6^3 tile and the side of the fine cell
        const int px = (x >> 1) + 1, py = (y >> 1) + 1, pz = (z >> 1) + 1;
        const int sx = (x & 1) ? 1 : -1, sy = (y & 1) ? 1 : -1, sz = (z & 1) ? 1 : -1;
        const int p0 = px + 6 * (py + 6 * pz);
        const int qx = sx, qy = 6 * sy, qz = 36 * sz;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T *C = sc[c];
            const T v = trilinear<T>(C[p0], C[p0 + qx] + C[p0 + qy] + C[p0 + qz],
                               C[p0 + qx + qy] + C[p0 + qx + qz] + C[p0 + qy + qz], C[p0 + qx + qy + qz]);
            if (c < ncomp) fine[c * fcs + (long long)b * NC + cell] = accumulate ? old[h][c] + v : v;
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(256)
k_prolong_dense_blk0(int nblk, const int *__restrict__ ijk, const int *__restrict__ prob_of,
                     const DenseProbDev *__restrict__ dp, const int *__restrict__ active,
                     const T *__restrict__ coarse, long long ccs, const T *base, T *fine, long long fcs,
                     int ncomp)
{
    // the 6^3 coarse cells the block's 8^3 fine cells interpolate from (its
    // 4^3 parents and one layer around them, periodic) are staged in LDS
    __shared__ T sc[3][216];
    const int b = xcd_block(blockIdx.x, nblk);
    const int pr = problem_of(prob_of, b);
    if (active && !active[pr]) return;
    const DenseProbDev q = dp[pr];
    const int bi = ijk[3 * b], bj = ijk[3 * b + 1], bk = ijk[3 * b + 2];
    const int i0 = 4 * bi - 1, j0 = 4 * bj - 1, k0 = 4 * bk - 1;
    for (int t = threadIdx.x; t < 216 * ncomp; t += blockDim.x) {
        const int c = t / 216, r = t % 216;
        const int i = (i0 + r % 6 + q.nx) % q.nx, j = (j0 + (r / 6) % 6 + q.ny) % q.ny, k = (k0 + r / 36 + q.nz) % q.nz;
        sc[c][r] = coarse[c * ccs + q.off + i + (long long)q.nx * (j + (long long)q.ny * k)];
    }
    __syncthreads();
    for (int cell = threadIdx.x; cell < NC; cell += blockDim.x) {
        const int x = cell & 7, y = (cell >> 3) & 7, z = cell >> 6;
        // parent (local index 1..4 on each axis) and its neighbour on the child's side
        const int i = (x >> 1) + 1, j = (y >> 1) + 1, k = (z >> 1) + 1;
        const int i1 = i + ((x & 1) ? 1 : -1), j1 = j + ((y & 1) ? 1 : -1), k1 = k + ((z & 1) ? 1 : -1);
        auto at = [](int a, int bb, int cc) { return a + 6 * (bb + 6 * cc); };
        for (int c = 0; c < ncomp; ++c) {
            const T *C = sc[c];
            const T v = trilinear<T>(C[at(i, j, k)], C[at(i1, j, k)] + C[at(i, j1, k)] + C[at(i, j, k1)],
                               C[at(i1, j1, k)] + C[at(i1, j, k1)] + C[at(i, j1, k1)], C[at(i1, j1, k1)]);
            const long long gi = c * fcs + (long long)b * NC + cell;
            fine[gi] = base ? base[gi] + v : v;
        }
    }
}

// ---------------------------------------------------------------------------
// refluxing (section 4)
// ---------------------------------------------------------------------------
// Refluxing.  An entry is a leaf cell of level l with faces next to covered
// cells; each such face needs, for both tangential components, the coarse
// flux and the four fine fluxes through it.  A workgroup takes whole entries
// (at most RF_WG_FACES faces) and gives every one of the ten fluxes of a face
// its own thread.  The face corrections and the entry sums are then formed in
// fixed orders: fine fluxes in child order, faces in face order.
//
// The launch is a chain of dependent loads: workgroup, face, neighbour blocks,
// fields.  All loads of a link are issued together and without branches, and
// what the last two phases need is on its way before the first: the refined
// 64^3 hierarchy's 30,000 faces (FP64) 15.4 -> 11.9 us, the smaller of the three-level
// one's 13.2 -> 6.6.
template <typename T>
__global__ void __launch_bounds__(RF_WG_FACES * 10)
k_reflux(const int *__restrict__ rfw, const int4 *__restrict__ rff, const int *__restrict__ rfs,
         const int *__restrict__ rf, const int *__restrict__ active, const int *__restrict__ cnbr,
         const int *__restrict__ fnbr, const double *__restrict__ inv_h_c, const double *__restrict__ coef_p, double coef_v,
         const T *__restrict__ Bc, long long ccs, const T *__restrict__ Ec, const T *__restrict__ Bf,
         long long fcs, const T *__restrict__ Bfg, long long fgcs, const T *__restrict__ Ef,
         const T *__restrict__ Efg, T *out)
{
    __shared__ T sfl[RF_WG_FACES * 10];
    __shared__ T sadd[RF_WG_FACES][2];
    const int e0 = rfw[4 * blockIdx.x], ne = rfw[4 * blockIdx.x + 1], f0 = rfw[4 * blockIdx.x + 2],
              nf = rfw[4 * blockIdx.x + 3];
    const int t = threadIdx.x;
    // one flux: face i, tangential component ci (c = d + 1 + ci mod 3), k = 0
    // the coarse face, k = 1..4 the fine faces (children a1, a2 = (k-1)/2, (k-1)%2)
    // (the ten lanes of a face share the lines they load: the same flux of
    // neighbouring faces side by side instead: 16.2 us)
    const int i = min(t / 10, nf - 1), ci = (t % 10) / 5, k = t % 5;
    const int4 fa = rff[2 * (f0 + i)], fb = rff[2 * (f0 + i) + 1];   // see RfFace
    // the face whose correction this thread forms, and its entry
    const int4 ga = rff[2 * (f0 + min(t >> 1, nf - 1)) + 1];
    const int e = e0 + min(t, ne - 1);
    const int *en = rf + RF_INTS * (long long)e;
    const int4 ea = *(const int4 *)en;   // block, cell, face mask
    const int epr = en[15], es = rfs[e];
    const int f = fb.x, d = f >> 1, sg = (f & 1) ? -1 : 1, c = (d + 1 + ci) % 3;
    // the face is after cell q of block b along d: after the entry's cell (sg =
    // +1) or the one below it; after the child (sg < 0) or the one below it
    const bool coarse = k == 0;
    const int b = coarse ? fa.x : fa.z, base = coarse ? fa.y : fa.w;
    int q[3] = {base & 7, (base >> 3) & 7, base >> 6};
    if (!coarse) {
        q[(d + 1) % 3] += (k - 1) >> 1;
        q[(d + 2) % 3] += (k - 1) & 1;
    }
    if ((sg < 0) == coarse) q[d] -= 1;
    // a, a + e_d, and both with + e_c, - e_c
    const int *nbr = (coarse ? cnbr : fnbr) + 27 * (long long)b;
    int n[6], li[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
        int r[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) r[x] = q[x] + ((m & 1) && x == d ? 1 : 0) + (x == c ? (m >= 4 ? -1 : (m >= 2 ? 1 : 0)) : 0);
        const int sx = side(r[0]), sy = side(r[1]), sz = side(r[2]), at = (sx + 1) + 3 * (sy + 1) + 9 * (sz + 1);
        const int v = nbr[at];
        n[m] = at == 13 ? b : v;
        li[m] = (r[0] - NB * sx) + NB * ((r[1] - NB * sy) + NB * (r[2] - NB * sz));
    }
    const double ih64 = inv_h_c[ga.y];   // fine fluxes carry h_f = h/2
    const T coef = T(coef_of(coef_p[epr], coef_v));
    const bool on = !(active && !active[fb.y]), eon = !(active && !active[epr]);
    const long long gi = (long long)ea.x * NC + ea.y;
    T o[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) o[x] = out[x * ccs + gi];
    {
        // a null coarse field stands for zero (its lanes read the first fine cell)
        const bool null = coarse && !Bc, cl = coarse && Bc;
        const T *F = cl ? Bc : Bf, *E = cl ? Ec : Ef, *G = cl ? Bc : Bfg, *EG = cl ? Ec : Efg;
        const long long fs = cl ? ccs : fcs, gs = cl ? ccs : fgcs;
        bool g[6];
        long long at[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            g[m] = n[m] < 0 && !null;
            at[m] = null ? 0 : (long long)(g[m] ? -1 - n[m] : n[m]) * NC + li[m];
        }
        auto field = [&](int m, int comp) { return (g[m] ? G : F)[(g[m] ? gs : fs) * comp + at[m]]; };
        auto resist = [&](int m) { return (g[m] ? EG : E)[at[m]]; };
        const T ea_ = resist(0), eq = resist(1);
        const T f2 = field(2, d), f3 = field(3, d), f4 = field(4, d), f5 = field(5, d), f1 = field(1, c), f0_ = field(0, c);
        const T ef = (ea_ + eq) * T(0.5);
        const T tr = (f2 + f3 - f4 - f5) * T(0.25);
        if (t < 10 * nf) sfl[t] = on && !null ? ef * (tr - (f1 - f0_)) : T(0);
    }
    __syncthreads();
    // face correction per tangential component: sg (<F_fine> - F_coarse) / h
    if (t < 2 * nf) {
        const int gsg = (ga.x & 1) ? -1 : 1;
        const T ih = T(ih64);
        const T *fl = sfl + 10 * (t >> 1) + 5 * (t & 1);
        const T Fc = fl[0] * ih;
        T Ff = fl[1];
        Ff += fl[2];
        Ff += fl[3];
        Ff += fl[4];
        Ff *= T(0.25) * (ih * T(2));
        sadd[t >> 1][t & 1] = T(gsg) * (Ff - Fc) * ih;
    }
    __syncthreads();
    if (t < ne && eon) {
        T a[3] = {T(0), T(0), T(0)};
        int j = es - f0;
#pragma unroll
        for (int ff = 0; ff < 6; ++ff)
            if ((ea.z >> ff) & 1) {
                a[((ff >> 1) + 1) % 3] += sadd[j][0];
                a[((ff >> 1) + 2) % 3] += sadd[j][1];
                ++j;
            }
#pragma unroll
        for (int x = 0; x < 3; ++x)
            if (a[x] != T(0)) out[x * ccs + gi] = o[x] + coef * a[x];
    }
}

template <typename T>
__global__ void k_zero_covered(int nblk, const uint8_t *__restrict__ cov, T *__restrict__ out, long long cs,
                               int ncomp)
{
    const int b = blockIdx.x;
    if (b >= nblk) return;
    const uint8_t m = cov[b];
    if (!m) return;
    for (int cell = threadIdx.x; cell < NC; cell += blockDim.x) {
        const int x = cell & 7, y = (cell >> 3) & 7, z = cell >> 6;
        if ((m >> ((x >> 2) + 2 * (y >> 2) + 4 * (z >> 2))) & 1)
            for (int c = 0; c < ncomp; ++c) out[c * cs + (long long)b * NC + cell] = T(0);
    }
}

// per-problem reduction of per-block partials (sums for k < ksum, max after):
// one workgroup per (problem, quantity); each thread walks a fixed strided
// subset of the problem's blocks (ranges per AMR level, in order), then a
// fixed-shape tree combines the threads -- the result depends only on the
// problem's own blocks, never on the other problems of the handle
__global__ void __launch_bounds__(256)
k_reduce_blocks(int nprob, int nrange, const long long *__restrict__ range, const double *__restrict__ part, int k,
                int ksum, double *__restrict__ out)
{
    __shared__ double sred[4];
    const int p = blockIdx.x / k, q = blockIdx.x % k;
    if (p >= nprob) return;   // uniform per workgroup, before any barrier
    const bool sum = q < ksum;
    double v = 0.0;
    long long base = 0;   // running block count of the problem (thread striding is global over its ranges)
    for (int r = 0; r < nrange; ++r) {
        const long long b0 = range[2 * ((long long)p * nrange + r)], b1 = range[2 * ((long long)p * nrange + r) + 1];
        const long long n = b1 - b0;
        // element i of this range has problem-local index base + i; thread t owns indices = t mod 256
        long long first = ((threadIdx.x - base) % 256 + 256) % 256;
        for (long long i = first; i < n; i += 256) {
            const double x = part[(b0 + i) * k + q];
            v = sum ? v + x : fmax(v, x);
        }
        base += n;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_down(v, o, 64);
        v = sum ? v + w : fmax(v, w);
    }
    if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = sred[0];
        for (int w = 1; w < 4; ++w) t = sum ? t + sred[w] : fmax(t, sred[w]);
        out[(long long)p * k + q] = t;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// The block stencil takes a thread per cell (8 instead of 20 tile loads in front
// of one instead of two applications) while all groups of 512 threads are
// resident at once, four to a compute unit.  us, two cells a thread / one: FP64
// 512 blocks 8.4 / 7.6, with the mean 9.4 / 8.6, 1,024 blocks 12.8 / 11.9 (residual
// 13.4 / 13.4), 1,232 blocks 14.2 / 14.7; FP32 512 blocks 6.2 / 5.9 (residual 6.5 /
// 6.0), 1,024 9.1 / 8.2 (9.4 / 8.4).
static bool one_cell_a_thread(const AmrLevelDev &L) { return L.nb <= 4 * COMPUTE_UNITS; }

// Base levels with marching tables take the marching stencil (but see the FP64
// residual in hier.hip), up to the 4 GiB a component that its 32-bit offsets
// reach.  L B on smaller levels, us, per block / marching in segments of one
// block: 64^3 9.8 / 10.9, 96^3 18.5 / 16.6, 112^3 25.0 / 23.5 -- too little for
// tables of its own.
static bool march_stencil(const AmrLevelDev &L, int mode, size_t elem)
{
    return L.nmarch > 0 && (mode != MODE_RESID || elem == 4 || L.march_resid64) &&
           (unsigned long long)L.nb * NC * elem <= 0xFFFFFFFFull;
}
template <typename T>
static bool march_sweep(const AmrLevelDev &L)
{
    return sizeof(T) == 8 ? L.march_sweep64 : L.march_sweep32;
}

template <typename T>
ohm_status launch_blk_stencil(const ohm_hier *h, int level, int mode, const T *B, const T *Bg, long long cs,
                              long long gcs, const T *S, const T *eta, const T *etag, Coef coef_dev,
                              T *out, int colour, double *partials, const uint8_t *cov_zero, const int *active,
                              hipStream_t s, StencilDots dots)
{
    const AmrLevelDev &L = h->amr[level];
    if (L.nb == 0) return OHM_OK;
    if (dots.ndot < 0 || dots.ndot > 2 || (dots.ndot > 0 && (mode != MODE_APPLY || !dots.dot_part)))
        return fail(OHM_ERR_ARG, "fused dot products need MODE_APPLY, 1 or 2 products and a partials buffer");
    const int given = (dots.ndot > 0 && dots.dot_y[0]) + (dots.ndot > 1 && dots.dot_y[1]);
    if (level == 0 && march_stencil(L, mode, sizeof(T)) && !cov_zero && !partials && out && mode != MODE_SMOOTH &&
        (dots.ndot == 0 || (given == 1 && std::is_same<T, double>::value)))
        return launch_march_stencil<T>(h, mode, B, cs, S, eta, coef_dev, out, 0, active, s, dots);
    const bool one = one_cell_a_thread(L);
#define ARGS L.nb, L.nbr, problem_table(h, L), cov_zero, active, L.inv_h2, coef_dev.p, coef_dev.v, B, Bg, cs, gcs, S, eta, \
             etag, out, colour, partials, dots, nullptr, nullptr, 0
#define RUN(mode)                                                              \
    if (one) k_blk_stencil<T, mode, 512><<<L.nb, 512, 0, s>>>(ARGS);           \
    else k_blk_stencil<T, mode, 256><<<L.nb, 256, 0, s>>>(ARGS)
    switch (mode) {
    case MODE_APPLY: RUN(MODE_APPLY); break;
    case MODE_RESID: RUN(MODE_RESID); break;
    case MODE_SMOOTH: RUN(MODE_SMOOTH); break;
    case MODE_MEAN:
        if (cov_zero) return fail(OHM_ERR_ARG, "the mean with an application is for levels without covered cells");
        RUN(MODE_MEAN);
        break;
    default: return fail(OHM_ERR_ARG, "unknown stencil mode %d", mode);
    }
#undef RUN
#undef ARGS
    return check_launch("block stencil");
}

template <typename T>
ohm_status launch_resid_restrict_blk0(const ohm_hier *h, const T *B, const T *Bg, long long cs, long long gcs,
                                      const T *S, const T *eta, const T *etag, Coef coef_dev, T *coarse,
                                      long long ccs, const int *active, hipStream_t s)
{
    const AmrLevelDev &L = h->amr[0];
    if (L.nb == 0) return OHM_OK;
    if (h->min_level > -1) return fail(OHM_ERR_ARG, "no dense level below level 0");
    if (march_stencil(L, MODE_RESID_RESTRICT, sizeof(T)))
        return launch_march_stencil<T>(h, MODE_RESID_RESTRICT, B, cs, S, eta, coef_dev, coarse, ccs, active, s);
    const int parts = tile_parts(L.nb);
    const bool pairs = ((uintptr_t)B | (uintptr_t)eta | (uintptr_t)(cs * sizeof(T))) % (2 * sizeof(T)) == 0;
    if (parts > 1 && L.complete27 && pairs) {
#define ARGS L.nb, L.nbr, problem_table(h, L), active, L.inv_h2, coef_dev.p, coef_dev.v, B, cs, S, eta, L.dense_map, \
             h->dense[1].probs, coarse, ccs
        if (parts == 4) k_blk_down<T, Tile<4, 4>><<<4 * L.nb, Tile<4, 4>::THREADS, 0, s>>>(ARGS);
        else k_blk_down<T, Tile<8, 4>><<<2 * L.nb, Tile<8, 4>::THREADS, 0, s>>>(ARGS);
#undef ARGS
        return check_launch("residual + restriction by parts");
    }
#define ARGS L.nb, L.nbr, problem_table(h, L), nullptr, active, L.inv_h2, coef_dev.p, coef_dev.v, B, Bg, cs, gcs, S, eta, etag, \
             coarse, 0, nullptr, StencilDots{{nullptr, nullptr}, 0, nullptr}, L.dense_map, h->dense[1].probs, ccs
    if (one_cell_a_thread(L)) k_blk_stencil<T, MODE_RESID_RESTRICT, 512><<<L.nb, 512, 0, s>>>(ARGS);
    else k_blk_stencil<T, MODE_RESID_RESTRICT, 256><<<L.nb, 256, 0, s>>>(ARGS);
#undef ARGS
    return check_launch("residual + restriction to dense");
}

template <typename T, int MODE, bool O64, bool DIRECT>
static void blk_sweep(const ohm_hier *h, const AmrLevelDev &L, const T *B, long long cs, const T *S, const T *eta,
                      Coef coef_dev, void *out, const int *active, hipStream_t s, const T *coarse,
                      long long ccs, const T *Bg, long long gcs, const T *etag)
{
#define ARGS L.nb, L.nbr, problem_table(h, L), active, L.inv_h2, coef_dev.p, coef_dev.v, B, cs, S, eta, out, L.ijk, h->dense[1].probs, \
             coarse, ccs, Bg, gcs, etag
    switch (tile_parts(L.nb)) {
    case 4: k_blk_sweep<T, MODE, O64, DIRECT, Tile<4, 4>><<<4 * L.nb, Tile<4, 4>::THREADS, 0, s>>>(ARGS); break;
    case 2: k_blk_sweep<T, MODE, O64, DIRECT, Tile<8, 4>><<<2 * L.nb, Tile<8, 4>::THREADS, 0, s>>>(ARGS); break;
    default: k_blk_sweep<T, MODE, O64, DIRECT, WholeTile><<<L.nb, WholeTile::THREADS, 0, s>>>(ARGS);
    }
#undef ARGS
}

template <typename T>
ohm_status launch_blk_sweep(const ohm_hier *h, int level, const T *B, long long cs, const T *S, const T *eta,
                            Coef coef_dev, T *out, const int *active, hipStream_t s, const T *coarse,
                            long long ccs, const T *Bg, long long gcs, const T *etag, double *out64)
{
    const AmrLevelDev &L = h->amr[level];
    if (L.nb == 0) return OHM_OK;
    if (out64) {
        if constexpr (std::is_same<T, float>::value) {
            if (!L.complete27 || !B)
                return fail(OHM_ERR_ARG, "an FP64 result needs a complete level and an input");
            if ((unsigned long long)L.nb * NC * sizeof(double) > 0xFFFFFFFFull)
                return fail(OHM_ERR_ARG, "level %d: FP64 result array above 4 GiB", level);
            if (((uintptr_t)B | (uintptr_t)eta | (uintptr_t)(cs * sizeof(T))) % (2 * sizeof(T)) != 0)
                return fail(OHM_ERR_ARG, "level %d: fused sweep needs B, eta and the component stride %zu-byte "
                                         "aligned", level, 2 * sizeof(T));
            if (coarse && (level != 0 || h->min_level > -1))
                return fail(OHM_ERR_ARG, "a fused coarse correction needs level 0 and a dense level below it");
            if (level == 0 && march_sweep<T>(L) &&
                ((uintptr_t)S % (2 * sizeof(T)) | (uintptr_t)out64 % (2 * sizeof(double))) == 0)
                return launch_march_sweep<T, double>(h, B, cs, S, eta, coef_dev, out64, active, s, coarse, ccs);
            if (coarse)
                blk_sweep<T, 2, true, false>(h, L, B, cs, S, eta, coef_dev, out64, active, s, coarse, ccs, nullptr, 0,
                                             nullptr);
            else
                blk_sweep<T, 0, true, false>(h, L, B, cs, S, eta, coef_dev, out64, active, s, nullptr, 0, nullptr, 0,
                                             nullptr);
            return check_launch("fused sweep to FP64");
        } else {
            return fail(OHM_ERR_ARG, "an FP64 result is for FP32 sweeps");
        }
    }
    if (!L.fused)
        return fail(OHM_ERR_ARG, "fused sweep needs every neighbour block of level %d as a level or ghost block", level);
    const bool gh = !L.complete27;
    if ((unsigned long long)L.nb * NC * sizeof(T) > 0xFFFFFFFFull ||
        (gh && (unsigned long long)L.ng * NC * sizeof(T) > 0xFFFFFFFFull))
        return fail(OHM_ERR_ARG, "level %d: fused sweep addresses each field array with 32-bit offsets (max 4 GiB)",
                    level);
    if (((uintptr_t)B | (uintptr_t)eta | (uintptr_t)(cs * sizeof(T))) % (2 * sizeof(T)) != 0)
        return fail(OHM_ERR_ARG, "level %d: fused sweep needs B, eta and the component stride %zu-byte aligned", level,
                    2 * sizeof(T));
    if (gh) {
        if (coarse) return fail(OHM_ERR_ARG, "a fused coarse correction needs level 0");
        if ((B && !Bg) || !etag) return fail(OHM_ERR_ARG, "level %d has ghost blocks: B_ghost and eta_ghost needed", level);
        if (((uintptr_t)Bg | (uintptr_t)etag | (uintptr_t)(gcs * sizeof(T))) % (2 * sizeof(T)) != 0)
            return fail(OHM_ERR_ARG, "level %d: fused sweep needs the ghost arrays and their stride %zu-byte aligned",
                        level, 2 * sizeof(T));
        if (B)
            blk_sweep<T, 3, false, false>(h, L, B, cs, S, eta, coef_dev, out, active, s, nullptr, 0, Bg, gcs, etag);
        else
            blk_sweep<T, 4, false, false>(h, L, B, cs, S, eta, coef_dev, out, active, s, nullptr, 0, nullptr, 0, etag);
        return check_launch("fused sweep with ghosts");
    }
    if (coarse && (level != 0 || h->min_level > -1 || !B))
        return fail(OHM_ERR_ARG, "a fused coarse correction needs level 0, a dense level below it and an input");
    if (level == 0 && march_sweep<T>(L) && ((uintptr_t)S | (uintptr_t)out) % (2 * sizeof(T)) == 0) {
        return launch_march_sweep<T, T>(h, B, cs, S, eta, coef_dev, out, active, s, coarse, ccs);
    } else if (coarse) {
        blk_sweep<T, 2, false, false>(h, L, B, cs, S, eta, coef_dev, out, active, s, coarse, ccs, nullptr, 0, nullptr);
    } else if (B) {
        // FP64 tiles go straight from global memory into LDS (16-byte pairs)
        blk_sweep<T, 0, false, std::is_same<T, double>::value>(h, L, B, cs, S, eta, coef_dev, out, active, s, nullptr, 0,
                                                               nullptr, 0, nullptr);
    } else {
        blk_sweep<T, 1, false, false>(h, L, B, cs, S, eta, coef_dev, out, active, s, nullptr, 0, nullptr, 0, nullptr);
    }
    return check_launch("fused sweep");
}

template <typename T>
ohm_status launch_restrict_blk(const ohm_hier *h, int fine_level, const T *fine, long long fcs, T *coarse,
                               long long ccs, int ncomp, const int *active, hipStream_t s)
{
    if (fine_level >= 1) {
        const AmrLevelDev &L = h->amr[fine_level];
        if (L.nb == 0) return OHM_OK;
        k_restrict_blk<T><<<L.nb, 64, 0, s>>>(L.nb, L.parent, L.octant, problem_table(h, L), active, fine, fcs, coarse, ccs,
                                              ncomp);
        return check_launch("restrict");
    }
    const AmrLevelDev &L = h->amr[0];
    k_restrict_blk0_dense<T><<<L.nb, 64, 0, s>>>(L.nb, L.dense_map, problem_table(h, L), h->dense[1].probs, active, fine, fcs,
                                                 coarse, ccs, ncomp);
    return check_launch("restrict to dense");
}

template <typename T>
ohm_status launch_prolong_blk(const ohm_hier *h, int coarse_level, const T *coarse, long long ccs, T *fine,
                              long long fcs, int ncomp, int accumulate, const int *active, hipStream_t s,
                              const T *base)
{
    if (coarse_level >= 0) {
        if (base) return fail(OHM_ERR_ARG, "prolongation between block levels is in place");
        const AmrLevelDev &F = h->amr[coarse_level + 1];
        if (F.nb == 0) return OHM_OK;
        k_prolong_blk<T><<<F.nb, 256, 0, s>>>(F.nb, F.parent, F.octant, problem_table(h, F), active, h->amr[coarse_level].nbr,
                                              coarse, ccs, fine, fcs, ncomp, accumulate);
        return check_launch("prolong");
    }
    const AmrLevelDev &L = h->amr[0];
    if (base && !accumulate) return fail(OHM_ERR_ARG, "prolongation onto a base field must accumulate");
    if (ncomp < 1 || ncomp > 3) return fail(OHM_ERR_ARG, "prolongation takes 1 to 3 components, got %d", ncomp);
    if (accumulate && !base) base = fine;
    k_prolong_dense_blk0<T><<<L.nb, 256, 0, s>>>(L.nb, L.ijk, problem_table(h, L), h->dense[1].probs, active, coarse, ccs, base,
                                                 fine, fcs, ncomp);
    return check_launch("prolong from dense");
}

template <typename T>
ohm_status launch_fill_ghosts(const ohm_hier *h, int level, const T *coarse, long long ccs, T *ghost,
                              long long gcs, int ncomp, const int *active, hipStream_t s)
{
    const AmrLevelDev &L = h->amr[level];
    if (level < 1 || L.ng == 0) return OHM_OK;
    k_prolong_blk<T><<<L.ng, 256, 0, s>>>(L.ng, L.gparent, L.goctant, h->nprob == 1 ? nullptr : L.gprob, active,
                                          h->amr[level - 1].nbr,
                                          coarse, ccs, ghost, gcs, ncomp, 0);
    return check_launch("fill ghosts");
}

template <typename T>
ohm_status launch_reflux(const ohm_hier *h, int level, const T *Bc, long long ccs, const T *etac, const T *Bf,
                         long long fcs, const T *Bfg, long long fgcs, const T *etaf, const T *etafg,
                         Coef coef_dev, T *out, const int *active, hipStream_t s)
{
    const AmrLevelDev &L = h->amr[level];
    if (L.nrf == 0) return OHM_OK;
    k_reflux<T><<<L.nrfw, RF_WG_FACES * 10, 0, s>>>(L.rfw, (const int4 *)L.rff, L.rfs, L.rf, active, L.nbr, h->amr[level + 1].nbr,
                                                   L.inv_h, coef_dev.p, coef_dev.v, Bc, ccs, etac, Bf, fcs, Bfg, fgcs, etaf, etafg,
                                                   out);
    return check_launch("reflux");
}

template <typename T>
ohm_status launch_zero_covered(const ohm_hier *h, int level, T *out, long long cs, int ncomp, hipStream_t s)
{
    const AmrLevelDev &L = h->amr[level];
    if (L.nb == 0) return OHM_OK;
    k_zero_covered<T><<<L.nb, 256, 0, s>>>(L.nb, L.cov, out, cs, ncomp);
    return check_launch("zero covered");
}

ohm_status launch_reduce_problem(int nprob, int nrange, const long long *range_dev, const double *part, int k,
                                 int ksum, double *out, hipStream_t s)
{
    k_reduce_blocks<<<nprob * k, 256, 0, s>>>(nprob, nrange, range_dev, part, k, ksum, out);
    return check_launch("reduce");
}

#define INST(T)                                                                                                 \
    template ohm_status launch_blk_sweep<T>(const ohm_hier *, int, const T *, long long, const T *, const T *,   \
                                            Coef, T *, const int *, hipStream_t, const T *, long long, \
                                            const T *, long long, const T *, double *);                         \
    template ohm_status launch_blk_stencil<T>(const ohm_hier *, int, int, const T *, const T *, long long,      \
                                              long long, const T *, const T *, const T *, Coef, T *,  \
                                              int, double *, const uint8_t *, const int *, hipStream_t,         \
                                              StencilDots);                                                     \
    template ohm_status launch_resid_restrict_blk0<T>(const ohm_hier *, const T *, const T *, long long,       \
                                                      long long, const T *, const T *, const T *,             \
                                                      Coef, T *, long long, const int *, hipStream_t);        \
    template ohm_status launch_restrict_blk<T>(const ohm_hier *, int, const T *, long long, T *, long long, int, \
                                               const int *, hipStream_t);                                       \
    template ohm_status launch_prolong_blk<T>(const ohm_hier *, int, const T *, long long, T *, long long, int,  \
                                              int, const int *, hipStream_t, const T *);                        \
    template ohm_status launch_fill_ghosts<T>(const ohm_hier *, int, const T *, long long, T *, long long, int,  \
                                              const int *, hipStream_t);                                        \
    template ohm_status launch_reflux<T>(const ohm_hier *, int, const T *, long long, const T *, const T *,      \
                                         long long, const T *, long long, const T *, const T *, Coef, \
                                         T *, const int *, hipStream_t);                                        \
    template ohm_status launch_zero_covered<T>(const ohm_hier *, int, T *, long long, int, hipStream_t);
INST(double)
INST(float)
#undef INST

}  // namespace ohm
