// One fused red-black sweep (eq. 19 with alpha of eqs. 21-23) of an 8^3 tile, or
// of a part of one.
//
// The tile and a two-cell halo are staged in LDS.  The red half-sweep is
// computed on the tile and, redundantly, on the red cells of the first halo
// layer that face the tile (their neighbours come from the second layer); the
// black half-sweep on the tile then reads those updated red values.  This is
// the same arithmetic as two separate half-sweeps.  `Addr::at(x, y, z)` gives
// the element offset of tile-local cell (x, y, z), -2 <= x, y, z <= 9, inside a
// component of the field.  Without `Addr::ghosts` every such cell is a level
// cell; with it, `Addr::entry(x, y, z)` is the neighbour entry of the cell's
// block (a level block, or ghost block -1-entry of the ghost arrays A.G, A.EG
// with component stride A.gcs), tile values of ghost blocks are loaded from
// those arrays, and first-layer red cells of ghost blocks keep their values
// (ghost values are fixed during smoothing).
// With ZERO the input field is zero and is not read (B may be null; so must
// be the ghost values): the red update reduces to S / diag and the tile starts
// from zeros, which gives the same values as a sweep over an explicitly zeroed
// field.  A `Coarse` object
// with active = true adds a coarse-grid correction to every tile value as it
// is loaded (prolongation fused into the first post-smoothing sweep); its
// load() issues the global reads of whatever it stages, stage() stores them in
// LDS (a barrier follows) and add(x, y, z, c, v) returns v plus the correction.
#pragma once

#include "common.h"
#include "stencil.h"

namespace ohm {

// What one group of a sweep updates: a tile of 8 x TY x TZ cells (8^3, or a part
// of one), staged with its two-cell halo by THREADS threads.
template <int TY_, int TZ_>
struct Tile {
    static constexpr int TY = TY_, TZ = TZ_, PARTS = (8 / TY) * (8 / TZ);
    static constexpr bool whole = PARTS == 1;
    static constexpr int THREADS = whole ? 512 : 384;
    static constexpr int W = 8 + 4, P = W * (TY + 4), N = P * (TZ + 4);   // row, plane and tile with the halo
    // coarse cells under the tile and its halo, with one more layer around
    static constexpr int CY = TY / 2 + 4, CZ = TZ / 2 + 4, NCOARSE = 8 * CY * CZ;
    // part q of an 8^3 tile starts at these cells of it
    static __device__ __forceinline__ int y0(int q) { return TY * (q % (8 / TY)); }
    static __device__ __forceinline__ int z0(int q) { return TZ * (q / (8 / TY)); }
    static __device__ __forceinline__ int at(int x, int y, int z) { return (x + 2) + W * ((y + 2) + (TY + 4) * (z + 2)); }
    // red cells: HALF of the tile, then those beyond its faces of x, y and z
    static constexpr int HALF = 4 * TY * TZ, FX = TY * TZ / 2, FY = 4 * TZ, FZ = 4 * TY, NRED = HALF + 2 * (FX + FY + FZ);
    static __device__ __forceinline__ void red_cell(int u, int &x, int &y, int &z)
    {
        if (u < HALF) {
            z = u / (4 * TY);
            y = (u >> 2) % TY;
            x = 2 * (u & 3) + ((y + z) & 1);
        } else if (whole) {
            const int w = u - HALF, f = w >> 5, k = w & 31;
            const int d = f >> 1, s = (f & 1) ? 8 : -1;
            const int bb = k >> 2, a = 2 * (k & 3) + ((s + bb) & 1);
            if (d == 0) { x = s; y = a; z = bb; }
            else if (d == 1) { x = a; y = s; z = bb; }
            else { x = a; y = bb; z = s; }
        } else if (int w = u - HALF; w < 2 * FX) {
            const int k = w % FX;
            x = w < FX ? -1 : 8;
            z = k / (TY / 2);
            y = 2 * (k % (TY / 2)) + ((x + z) & 1);
        } else if ((w -= 2 * FX) < 2 * FY) {
            y = w < FY ? -1 : TY;
            z = (w >> 2) % TZ;
            x = 2 * (w & 3) + ((y + z) & 1);
        } else {
            w -= 2 * FY;
            z = w < FZ ? -1 : TZ;
            y = (w >> 2) % TY;
            x = 2 * (w & 3) + ((y + z) & 1);
        }
    }
};
using WholeTile = Tile<8, 8>;

// Groups a tile is split over in a launch of `tiles`: as many as find a compute
// unit each.  A group alone on its unit waits out its chain (neighbour list,
// tile, red cells, black cells, store), of which the updates take longer the
// more cells it has; with every unit taken the parts' larger share of halo
// cells costs more than that gives.  Steps of six iterations (2 + 5 sweeps, 1
// below the base) with the base level's tiles whole, halved and quartered, us:
// FP64 32^3 (64 tiles) 1184, 1130 and 1099, 40^3 (125) 1295, 1256 and 1290, 48^3
// (216) 1481, 1566 and 1798; mixed 1036, 1025 and 1007, 1134, 1124 and 1158, 1308,
// 1341 and 1405.  With the dense levels of a 64^3 box (64, 8 and 1 tiles) so: FP64
// 2073, 1924 and 1850, mixed 1627, 1621 and 1579.
constexpr int COMPUTE_UNITS = 256;
inline int tile_parts(int tiles) { return 4 * tiles <= COMPUTE_UNITS ? 4 : 2 * tiles <= COMPUTE_UNITS ? 2 : 1; }

// The cells of an 8^3 tile as seen from the part at (0, y0, z0)
template <typename Addr>
struct PartAddr : Addr {
    int y0, z0;
    __device__ __forceinline__ long long at(int x, int y, int z) const { return Addr::at(x, y + y0, z + z0); }
    __device__ __forceinline__ int entry(int x, int y, int z) const { return Addr::entry(x, y + y0, z + z0); }
    __device__ __forceinline__ int local(int x, int y, int z) const { return Addr::local(x, y + y0, z + z0); }
};

__device__ __forceinline__ int wrap_cell(int i, int n)
{
    // i >= -2; past the first period only on grids narrower than a tile
    if (i < 0) return i + n;
    if (i >= n) {
        i -= n;
        if (i >= n) i %= n;
    }
    return i;
}

// two consecutive elements, loaded and stored as one 2 sizeof(T) access
template <typename T>
struct alignas(2 * sizeof(T)) Pair {
    T a, b;
};

template <typename T>
struct NoCoarse {
    static constexpr bool active = false;
    __device__ __forceinline__ void load() {}
    __device__ __forceinline__ void stage() {}
    __device__ __forceinline__ T add(int, int, int, int, T v) const { return v; }
};

// Element at a byte offset from a wavefront-uniform base: the offset stays a
// 32-bit VGPR and the base an SGPR pair, so the 3 components and eta share one
// address computation.  The launchers check that every level array fits in
// 4 GiB.
template <typename T>
__device__ __forceinline__ T load_at(const T *base, unsigned off)
{
    return *(const T *)((const char *)base + off);
}
template <typename T>
__device__ __forceinline__ Pair<T> load_pair(const T *base, unsigned off)
{
    return *(const Pair<T> *)((const char *)base + off);
}
template <typename T>
__device__ __forceinline__ void store_at(T *base, unsigned off, T v)
{
    *(T *)((char *)base + off) = v;
}

// Trilinear correction (27/9/3/1 over 64) from the next coarser grid, a dense
// grid q, for the tile of fine origin (i, j, k): the coarse cells that hold the
// parents of the tile's cells and their neighbours (origin (i, j, k) / 2 - 2,
// periodic) are staged in LDS; the weights and the order of the sum are those
// of the stand-alone prolongation kernels.
template <typename T, typename Tl = WholeTile>
struct TileCoarse {
    static constexpr bool active = true;
    static constexpr int N = 3 * Tl::NCOARSE, PER = (N + Tl::THREADS - 1) / Tl::THREADS;
    const T *coarse;
    long long ccs;
    DenseProbDev q;
    int i0, j0, k0;
    T *sC;      // [N] in LDS
    T r[PER];
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            unsigned t = threadIdx.x + Tl::THREADS * k;
            if (N % Tl::THREADS) t = min(t, (unsigned)N - 1);
            const unsigned c = t / Tl::NCOARSE, m = t % Tl::NCOARSE;
            const int i = wrap_cell(i0 + (int)(m & 7), q.nx), j = wrap_cell(j0 + (int)((m >> 3) % Tl::CY), q.ny),
                      kk = wrap_cell(k0 + (int)(m / (8 * Tl::CY)), q.nz);
            r[k] = coarse[c * ccs + q.off + i + (long long)q.nx * (j + (long long)q.ny * kk)];
        }
    }
    __device__ __forceinline__ void stage()
    {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (N % Tl::THREADS == 0 || (int)threadIdx.x + Tl::THREADS * k < N) sC[threadIdx.x + Tl::THREADS * k] = r[k];
    }
    __device__ __forceinline__ T add(int x, int y, int z, int c, T base) const
    {
        const int i = (x >> 1) + 2, j = (y >> 1) + 2, k = (z >> 1) + 2;
        const int i1 = i + ((x & 1) ? 1 : -1), j1 = j + ((y & 1) ? 1 : -1), k1 = k + ((z & 1) ? 1 : -1);
        const T *C = sC + Tl::NCOARSE * c;
        auto at = [](int a, int bb, int cc) { return a + 8 * (bb + Tl::CY * cc); };
        const T v = trilinear<T>(C[at(i, j, k)], C[at(i1, j, k)] + C[at(i, j1, k)] + C[at(i, j, k1)],
                           C[at(i1, j1, k)] + C[at(i1, j, k1)] + C[at(i, j1, k1)], C[at(i1, j1, k1)]);
        return base + v;
    }
};

// The result goes to `out` as TO (T, or double from an FP32 sweep), with the
// same element offsets and component stride as the input.
// 16 bytes from global memory straight into LDS: lane l of the wavefront
// writes dst + 16 l bytes (dst uniform over the wavefront)
__device__ __forceinline__ void lds_load16(const void *src, void *dst)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                     (void __attribute__((address_space(3))) *)dst, 16, 0, 0);
}

template <typename T, bool ZERO, typename Addr, typename Coarse = NoCoarse<T>, typename TO = T,
          typename Tl = WholeTile, int TS = Tl::N, bool DIRECT = false>
__device__ __forceinline__ void fused_sweep_tile(const Addr &A, const T *__restrict__ B, long long cs,
                                                 const T *__restrict__ S, const T *__restrict__ eta,
                                                 TO *__restrict__ out, const T cih2, T (*sB)[TS], T *sE,
                                                 Coarse cor = Coarse())
{
    constexpr int TY = Tl::TY, TZ = Tl::TZ, THREADS = Tl::THREADS;
    const int u = threadIdx.x;
    const T *B0 = B, *B1 = ZERO ? B : B + cs, *B2 = ZERO ? B : B + 2 * cs;
    const T *S0 = S, *S1 = S + cs, *S2 = S + 2 * cs;
    constexpr int HALF = Tl::HALF;
    const T c8 = cih2 * T(0.125), c2 = cih2 * T(0.5);
    auto load_s = [&] __device__(T v[3], int x, int y, int z) {
        const unsigned off = (unsigned)A.at(x, y, z) * (unsigned)sizeof(T);
        v[0] = load_at(S0, off);
        v[1] = load_at(S1, off);
        v[2] = load_at(S2, off);
    };
    // This thread's black cell (u < HALF) and its red one (as red_cell) in the
    // tile (-1: none) with their S.  A part of a tile requests S together with
    // the tile: a launch of parts has too few groups to hide a cold load
    // behind another group's updates.
    T srd[3], sbk[3], red[3];
    int rp = -1, pb = -1;
    auto red_start = [&] __device__() {
        int x, y, z;
        Tl::red_cell(u, x, y, z);
        if constexpr (Addr::ghosts)
            if (u >= HALF && A.entry(x, y, z) < 0) return;
        rp = Tl::at(x, y, z);
        load_s(srd, x, y, z);
    };
    auto red_update = [&] __device__() {
        T al[3];
        if (ZERO) {
            alpha_all<T, Tl::W, Tl::P>(sE, rp, al);
#pragma unroll
            for (int c = 0; c < 3; ++c) red[c] = relax_div(srd[c], fma(c2, al[c], T(1)));
        } else {
            T dv[3];
            divF_all<T, Tl::W, Tl::P>(sB[0], sB[1], sB[2], sE, rp, dv, al);
#pragma unroll
            for (int c = 0; c < 3; ++c) red[c] = relax_point(sB[c][rp], srd[c], dv[c], al[c], c8, c2);
        }
    };
    auto black_start = [&] __device__() {
        const int z = u / (4 * TY), y = (u >> 2) % TY, x = 2 * (u & 3) + (1 - ((y + z) & 1));
        pb = Tl::at(x, y, z);
        load_s(sbk, x, y, z);
    };
    if constexpr (!Tl::whole) {
        if (u < Tl::NRED) red_start();
        if (u < HALF) black_start();
    }
    if constexpr (DIRECT) {
        // FP64 tile pairs loaded straight into LDS: pair P = u + THREADS k of
        // the NP (plane-major, as the tile lays them out) lands at element 2 P,
        // which is lane order within each wavefront; lanes past the last pair
        // (of the 864 of a whole tile) reload it into 64 elements of padding
        constexpr int NPC = Tl::P / 2, NP = Tl::N / 2;
        static_assert(sizeof(T) == 8 && !ZERO && !Addr::ghosts && !Coarse::active &&
                          TS >= Tl::N + (NP % 64 ? 64 : 0),
                      "direct tile loads are for plain FP64 sweeps");
        const int w = u >> 6;
        // the waves of a group that issues its tile's loads take precedence
        // over the other resident group's updates until the loads are out
        __builtin_amdgcn_s_setprio(3);
#pragma unroll
        for (int k = 0; k < (NP + THREADS - 1) / THREADS; ++k) {
            const int first = THREADS * k + 64 * w;
            if (first < NP) {
                const int P = min(u + THREADS * k, NP - 1);
                const int pc = P % NPC, z = P / NPC - 2;
                const int x = 2 * (pc % (Tl::W / 2)) - 2, y = pc / (Tl::W / 2) - 2;
                const unsigned off = (unsigned)A.at(x, y, z) * (unsigned)sizeof(T);
                lds_load16((const char *)B0 + off, &sB[0][2 * first]);
                lds_load16((const char *)B1 + off, &sB[1][2 * first]);
                lds_load16((const char *)B2 + off, &sB[2][2 * first]);
                lds_load16((const char *)eta + off, &sE[2 * first]);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    } else {
    // tile load in pairs of x-neighbours (x even, so a pair never straddles a
    // block or a periodic wrap and is 2 sizeof(T) aligned): a loader (the
    // first 432 threads of a whole tile) owns pair column (px, y) = u mod NPC
    // and EACH planes; all global loads first, then the LDS stores
    constexpr int NPC = Tl::P / 2;           // pair columns per plane
    constexpr int EACH = NPC * (TZ + 4) > THREADS ? 2 : 1;
    const bool loader = u < (TZ + 4) / EACH * NPC;
    const int pc = u % NPC, zq = u / NPC;
    const int x = 2 * (pc % (Tl::W / 2)) - 2, y = pc / (Tl::W / 2) - 2;
    Pair<T> v[EACH][4];
    if (Coarse::active) cor.load();
    if (loader) {
#pragma unroll
        for (int k = 0; k < EACH; ++k) {
            const int z = EACH * zq + k - 2;
            if constexpr (Addr::ghosts) {
                const int n = A.entry(x, y, z);
                const bool g = n < 0;
                const unsigned off = ((unsigned)(g ? -1 - n : n) * (unsigned)NC + (unsigned)A.local(x, y, z)) *
                                     (unsigned)sizeof(T);
                if (!ZERO) {
                    v[k][0] = load_pair(g ? A.G : B0, off);
                    v[k][1] = load_pair(g ? A.G + A.gcs : B1, off);
                    v[k][2] = load_pair(g ? A.G + 2 * A.gcs : B2, off);
                }
                v[k][3] = load_pair(g ? A.EG : eta, off);
            } else {
                const unsigned off = (unsigned)A.at(x, y, z) * (unsigned)sizeof(T);
                if (!ZERO) {
                    v[k][0] = load_pair(B0, off);
                    v[k][1] = load_pair(B1, off);
                    v[k][2] = load_pair(B2, off);
                }
                v[k][3] = load_pair(eta, off);
            }
        }
    }
    if (Coarse::active) {
        cor.stage();
        __syncthreads();
    }
    if (loader) {
#pragma unroll
        for (int k = 0; k < EACH; ++k) {
            const int z = EACH * zq + k - 2;
            const int t = Tl::at(x, y, z);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                Pair<T> w;
                w.a = cor.add(x, y, z, c, ZERO ? T(0) : v[k][c].a);
                w.b = cor.add(x + 1, y, z, c, ZERO ? T(0) : v[k][c].b);
                *(Pair<T> *)&sB[c][t] = w;
            }
            *(Pair<T> *)&sE[t] = v[k][3];
        }
    }
    __syncthreads();
    }
    // red half-sweep; a whole tile requests the black cells' S here, to overlap
    // with it
    if constexpr (Tl::whole) {
        if (u < HALF) black_start();
        if (u < Tl::NRED) {
            red_start();
            if (!Addr::ghosts || rp >= 0) red_update();
        }
    } else if (rp >= 0) {
        red_update();
    }
    __syncthreads();
    if (rp >= 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) sB[c][rp] = red[c];
    __syncthreads();
    // black half-sweep on the tile
    {
        T blk[3];
        if (u < HALF) {
            T dv[3], al[3];
            divF_all<T, Tl::W, Tl::P>(sB[0], sB[1], sB[2], sE, pb, dv, al);
#pragma unroll
            for (int c = 0; c < 3; ++c) blk[c] = relax_point(sB[c][pb], sbk[c], dv[c], al[c], c8, c2);
        }
        __syncthreads();
        if (u < HALF)
#pragma unroll
            for (int c = 0; c < 3; ++c) sB[c][pb] = blk[c];
    }
    __syncthreads();
    if (Tl::whole || u < 8 * TY * TZ) {
        const int x = u & 7, y = (u >> 3) % TY, z = u / (8 * TY);
        const int p = Tl::at(x, y, z);
        const unsigned off = (unsigned)A.at(x, y, z) * (unsigned)sizeof(TO);
        store_at(out, off, TO(sB[0][p]));
        store_at(out + cs, off, TO(sB[1][p]));
        store_at(out + 2 * cs, off, TO(sB[2][p]));
    }
}

// ---------------------------------------------------------------------------
// The way down from a level of few tiles, by parts of a tile as the sweeps: the
// residual S - L e with its restriction, with ZERO behind one sweep from a zero
// guess (whose result is stored), which computes e one cell around the part.
// Same operations on the same values as the sweep and the residual kernels.
//
// Such a launch is its chain of loads and updates; the sweep's launch, its
// stores and the reload of e and eta are what putting it in front saves.  FP64
// levels of 16^3 and 8^3: 4.1 + 6.0 -> 6.7 and 4.0 + 4.6 -> 5.7 us; without the
// sweep (base level of 32^3) 6.0 -> 3.7 us against the kernel of whole blocks.
// ---------------------------------------------------------------------------
template <typename Tl>
struct DownTile {
    // tile and halo in LDS: rows of 16 (x from -4), y and z from -3
    static constexpr int W = 16, P = W * (Tl::TY + 6), N = P * (Tl::TZ + 6), CELLS = 8 * Tl::TY * Tl::TZ,
                         NC8 = CELLS / 8;   // coarse cells
    static __device__ __forceinline__ int at(int x, int y, int z) { return (x + 4) + W * ((y + 3) + (Tl::TY + 6) * (z + 3)); }
};

// the residual goes to sR[component][cell of the part], x fastest
template <typename T, bool ZERO, typename Tl, typename Addr>
__device__ __forceinline__ void down_tile(const Addr &A, T *e, long long cs, const T *__restrict__ S,
                                          const T *__restrict__ eta, const T cih2, T (*sB)[DownTile<Tl>::N], T *sE,
                                          T (*sR)[DownTile<Tl>::CELLS])
{
    using Dn = DownTile<Tl>;
    constexpr int TY = Tl::TY, TZ = Tl::TZ, THREADS = Tl::THREADS;
    const int u = threadIdx.x;
    auto off = [&] __device__(int x, int y, int z) { return (unsigned)A.at(x, y, z) * (unsigned)sizeof(T); };
    auto load_s = [&] __device__(T v[3], int x, int y, int z) {
        const unsigned o = off(x, y, z);
        v[0] = load_at(S, o);
        v[1] = load_at(S + cs, o);
        v[2] = load_at(S + 2 * cs, o);
    };
    // eta (and e) in pairs of x-neighbours: three cells around the part (one
    // without the sweep)
    constexpr int H = ZERO ? 3 : 1, PW = ZERO ? 8 : 6, X0 = ZERO ? -4 : -2;
    constexpr int NP = PW * (TY + 2 * H) * (TZ + 2 * H), PER = (NP + THREADS - 1) / THREADS;
    Pair<T> ve[PER], vb[ZERO ? 1 : PER][3];
    int tp[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = min(u + THREADS * k, NP - 1);
        const int x = X0 + 2 * (t % PW), y = t / PW % (TY + 2 * H) - H, z = t / (PW * (TY + 2 * H)) - H;
        const unsigned o = off(x, y, z);
        tp[k] = Dn::at(x, y, z);
        ve[k] = load_pair(eta, o);
        if (!ZERO)
#pragma unroll
            for (int c = 0; c < 3; ++c) vb[k][c] = load_pair(e + c * cs, o);
    }
    // S of the cells this thread updates: red cells two around the part, black
    // ones one around it, then a cell of the part
    constexpr int NR = ZERO ? 6 * (TY + 4) * (TZ + 4) : 0, RPER = (NR + THREADS - 1) / THREADS, NK = 5 * (TY + 2) * (TZ + 2);
    static_assert(NK <= THREADS && Dn::CELLS <= THREADS, "one black cell and one cell of the part per thread");
    T sr[RPER ? RPER : 1][3], sk[3], so[3];
    int rp[RPER ? RPER : 1], pk = 0;
    if constexpr (ZERO) {
#pragma unroll
        for (int k = 0; k < RPER; ++k) {
            const int t = min(u + THREADS * k, NR - 1);
            const int y = t / 6 % (TY + 4) - 2, z = t / (6 * (TY + 4)) - 2, x = -2 + 2 * (t % 6) + ((y + z) & 1);
            rp[k] = Dn::at(x, y, z);
            load_s(sr[k], x, y, z);
        }
        const int t = min(u, NK - 1);
        const int y = t / 5 % (TY + 2) - 1, z = t / (5 * (TY + 2)) - 1, x = -1 + 2 * (t % 5) + ((y + z) & 1);
        pk = Dn::at(x, y, z);
        load_s(sk, x, y, z);
    }
    const int cell = min(u, Dn::CELLS - 1), x = cell & 7, y = (cell >> 3) % TY, z = cell / (8 * TY);
    const int po = Dn::at(x, y, z);
    load_s(so, x, y, z);
#pragma unroll
    for (int k = 0; k < PER; ++k) {   // (threads past the last pair store it again)
        *(Pair<T> *)&sE[tp[k]] = ve[k];
        if (!ZERO)
#pragma unroll
            for (int c = 0; c < 3; ++c) *(Pair<T> *)&sB[c][tp[k]] = vb[k][c];
    }
    const T c8 = cih2 * T(0.125), c2 = cih2 * T(0.5);
    __syncthreads();
    if constexpr (ZERO) {
        // red: S over the diagonal; the other cell of the pair is still zero
#pragma unroll
        for (int k = 0; k < RPER; ++k) {
            T al[3];
            alpha_all<T, Dn::W, Dn::P>(sE, rp[k], al);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                sB[c][rp[k]] = relax_div(sr[k][c], fma(c2, al[c], T(1)));
                sB[c][rp[k] ^ 1] = T(0);
            }
        }
        __syncthreads();
        T blk[3], dv[3], al[3];
        divF_all<T, Dn::W, Dn::P>(sB[0], sB[1], sB[2], sE, pk, dv, al);
#pragma unroll
        for (int c = 0; c < 3; ++c) blk[c] = relax_point(T(0), sk[c], dv[c], al[c], c8, c2);
        __syncthreads();
        if (u < NK)
#pragma unroll
            for (int c = 0; c < 3; ++c) sB[c][pk] = blk[c];
        __syncthreads();
    }
    {
        T dv[3], al[3];
        divF_all<T, Dn::W, Dn::P>(sB[0], sB[1], sB[2], sE, po, dv, al);
        if (u < Dn::CELLS) {
            const unsigned o = off(x, y, z);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                sR[c][u] = so[c] - fma(c8, dv[c], sB[c][po]);
                if (ZERO) store_at(e + c * cs, o, sB[c][po]);
            }
        }
    }
    __syncthreads();
}

// mean of the residual over the children of coarse cell t of the part
template <typename T, typename Tl>
__device__ __forceinline__ T restrict_part(const T *r, int t)
{
    const int i = t & 3, j = (t >> 2) % (Tl::TY / 2), k = t / (2 * Tl::TY);
    T a = T(0);
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) a += r[(2 * i + dx) + 8 * ((2 * j + dy) + Tl::TY * (2 * k + dz))];
    return a * T(0.125);
}

}  // namespace ohm
