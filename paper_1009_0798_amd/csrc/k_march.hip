// Plane-marching fused red-black sweep (eq. 19) of the base level.
//
// A workgroup takes a column segment of 16 x 16 cells and marches along z.  At
// step q plane q of B and eta, with a halo of two cells, goes to LDS, the red
// cells of plane q - 1 and the black cells of plane q - 2 are updated, and
// plane q - 2 is written: the operations of the sweep per 8^3 block (sweep.h)
// on the same values, hence the same bits.  A cell's neighbours above and
// below are its own thread's registers, the others come from rings of planes
// in LDS, kept by colour so that consecutive lanes read consecutive elements.
//
// What bounds it: on large levels HBM, on the smallest it takes the issue of
// the wavefronts that update both colours (a step is about 300 vector
// instructions and 60 LDS reads of theirs, 1.1 us in FP64).  Against the sweep
// per block it loads 1.56 instead of 3.4 cells per cell (plus four planes per
// segment) and asks the L2 for 2.5 instead of 6.7 lines per line, and its
// loads run two planes ahead instead of in front of each block's updates.
// Measured per launch on one box, us, sweep per block -> this kernel: FP64
// 128^3 47.6 -> 39.2, 160x128x192 110 -> 79, 256^3 505 -> 307 (2.7 -> 4.4 TB/s of
// algorithmic bytes; other boxes up to 344); FP32 28.3 -> 24.4, 49 -> 39, 284 -> 189.
#include <type_traits>

#include "march.h"
#include "stencil.h"
#include "sweep.h"

namespace ohm {

namespace {

// B (3 components) and eta of a pair of x-neighbours on one plane, and S on
// the plane before
template <typename T>
struct Stage {
    Pair<T> b[3], e, s[3];
    T co;   // a coarse value (see CoarseRing)
};

// a value every lane holds, kept in scalar registers
__device__ __forceinline__ float uniform(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)b),
                   hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// waits for this wave's LDS accesses only: global loads stay in flight
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Two consecutive results at a byte offset; an offset past the array (lanes
// without a result) is dropped by the buffer's bounds check, so the store
// stays outside any branch and the loads in flight are counted exactly.
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, unsigned off, Pair<double> v)
{
    typedef unsigned __attribute__((ext_vector_type(4))) u4;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, off, 0, 0);
}
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, unsigned off, Pair<float> v)
{
    typedef unsigned __attribute__((ext_vector_type(2))) u2;
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, 0, 0);
}

__device__ __forceinline__ void store_one(__amdgpu_buffer_rsrc_t r, unsigned off, double v)
{
    typedef unsigned __attribute__((ext_vector_type(2))) u2;
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, 0, 0);
}
__device__ __forceinline__ void store_one(__amdgpu_buffer_rsrc_t r, unsigned off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 0);
}

// LDS rings of planes, plane q in slot (q - first plane) mod 4 (mod 2 for the
// updated red cells): red and black cells before the sweep, red cells after
// it, resistivity at the red and at the black cells
constexpr int RB = MNP;                               // elements per ring row (one component of one plane)
constexpr int O_ER = 0, O_EK = O_ER + 4 * RB, O_R1 = O_EK + 4 * RB, O_R0 = O_R1 + 2 * 3 * RB, O_K0 = O_R0 + 4 * 3 * RB,
              N_ZERO = O_R0, N_FULL = O_K0 + 4 * 3 * RB;

// With a coarse correction the tile's values are B + P(coarse): the coarse cells
// under the tile and its halo, with one more layer around (12 x 12 cells from
// half the tile's origin less 2), of the planes K = q/2 - 1 to q/2 + 2 are kept
// in a ring in LDS.  At step q every thread requests one of the 216 values of
// half (q mod 2) of plane q/2 + 3, and stores it two steps later: plane K is
// complete at step 2 K - 3 and first read at step 2 K - 1.  (36 LDS reads and 54
// operations a pair; us against the prolongation's launch and a sweep, FP64
// 128^3 24.2 + 39.5 -> 51.7, FP32 160x128x192 29.9 + 39.9 -> 53.8; against a
// sweep per block with the correction, 64 FP32 problems, 82 -> 73.)
constexpr int CW = MT / 2 + 4, CP = 3 * CW * CW;      // edge, and elements of a plane
template <typename T>
struct CoarseRing {
    T *lds;                  // [4][CP]
    const T *src;
    unsigned off[2];         // this thread's value of each half on plane 0: byte offset ...
    int at[2];               // ... and place in the plane
    unsigned plane;          // bytes from plane to plane
    int nz;
    __device__ __forceinline__ T load(int half, int K) const
    {
        K = K < 0 ? K + nz : (K >= nz ? K - nz : K);
        return load_at(src, off[half] + (unsigned)K * plane);
    }
    __device__ __forceinline__ T *slot(int K) const { return lds + (K & 3) * CP; }
};

// hardware placement of a wavefront: bits 0-3 its slot on the SIMD, 4-5 the SIMD
constexpr int HWREG_PLACE = 4 | (5 << 11);

// Wavefronts of a group: two update the tile's 128 pairs of x-neighbours (a
// pair holds one red and one black cell on every plane), one the red cells of
// the first halo layer that face the tile, one only loads the rest of the halo
enum { ROLE_INNER = 0, ROLE_RING = 1, ROLE_LOAD = 2 };

template <typename T, typename TO, int ROLE, bool ZERO, bool CO>
__device__ __forceinline__ void march_loop(T *sh, const int *ids, const T *__restrict__ B, long long cs,
                                           const T *__restrict__ S, const T *__restrict__ eta, TO *__restrict__ out,
                                           unsigned obytes, T cih2, int x, int y, int z0, int n, bool in,
                                           const CoarseRing<T> &co)
{
    constexpr bool RED = ROLE != ROLE_LOAD, BLACK = ROLE == ROLE_INNER;
    const T c8 = uniform(cih2 * T(0.125)), c2 = uniform(cih2 * T(0.5));
    const int u = (x + 2) / 2 + MHW * (y + 2);
    const T *B0 = B, *B1 = ZERO ? B : B + cs, *B2 = ZERO ? B : B + 2 * cs;
    const T *S0 = S, *S1 = S + cs, *S2 = S + 2 * cs;
    const __amdgpu_buffer_rsrc_t O0 = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)obytes, 0x00027000),
                                 O1 = __builtin_amdgcn_make_buffer_rsrc(out + cs, 0, (int)obytes, 0x00027000),
                                 O2 = __builtin_amdgcn_make_buffer_rsrc(out + 2 * cs, 0, (int)obytes, 0x00027000);

    Stage<T> st[2];
    // block of the pair on plane P
    auto block = [&](int P) {
        int v = u;
        asm volatile("" : "+v"(v));   // formed when needed, once in 8 planes: not held in registers
        const int ry = v / MHW, hx = v - ry * MHW;
        return (unsigned)ids[((hx + 3) >> 2) + 4 * ((ry + 6) >> 3) + 16 * (((P - z0) >> 3) + 1)];
    };
    // byte offset of the pair on plane P, given the one on plane P - 1
    auto offset = [&](int P, unsigned before) -> unsigned {
        constexpr unsigned PLANE = 64 * (unsigned)sizeof(T);
        return (P & 7) == 0 ? block(P) * 8u * PLANE + before % PLANE : before + PLANE;
    };
    auto issue = [&](Stage<T> &v, unsigned off, unsigned offs, int half, int K) {
        if (CO) v.co = co.load(half, K);
        if (!ZERO) {
            v.b[0] = load_pair(B0, off);
            v.b[1] = load_pair(B1, off);
            v.b[2] = load_pair(B2, off);
        }
        v.e = load_pair(eta, off);
        if (RED) {
            v.s[0] = load_pair(S0, offs);
            v.s[1] = load_pair(S1, offs);
            v.s[2] = load_pair(S2, offs);
        }
    };
    const int zs = z0 - 2, zend = z0 + n + 2;                   // planes zs .. zend - 1
    const unsigned o_p0 = (block(zs) * (unsigned)NC + (unsigned)((x & 7) + 8 * (y & 7) + 64 * (zs & 7))) * (unsigned)sizeof(T),
                   o_p1 = offset(zs + 1, o_p0);
    // (as in the loop, each plane's loads are followed by three stores, here
    // dropped ones: the waits count the accesses behind the plane they need)
    const Pair<TO> none = {TO(0), TO(0)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        issue(st[h], h ? o_p1 : o_p0, o_p0, h, (zs >> 1) + 2);
        __builtin_amdgcn_sched_barrier(0);
        if (BLACK) {
            store_pair(O0, 0xFFFFFFF0u, none);
            store_pair(O1, 0xFFFFFFF0u, none);
            store_pair(O2, 0xFFFFFFF0u, none);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // register history of this thread's column, by plane mod 4 (a pair holds
    // one red and one black cell on every plane): values before the sweep,
    // resistivity, red values after it, S of the black cell, offset, and what
    // a plane's red (black) cells contribute to the planes around it
    T k[4][3], er[4], nw[4][3], sk[4][3];
    unsigned off[4] = {o_p0, o_p1, 0u, 0u};
    PlaneEdges<T> xk[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        er[h] = T(0);
        xk[h] = PlaneEdges<T>{T(0), T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int c = 0; c < 3; ++c) k[h][c] = nw[h][c] = sk[h][c] = T(0);
    }
    int q0 = zs;
    do {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int q = q0 + h;
            constexpr int m = 3;
            const int h1 = (h + 3) & m, h2 = (h + 2) & m, h3 = (h + 1) & m;   // planes q - 1, q - 2, q - 3
            const bool par = ((y + h) & 1) != 0;                // red is the pair's second cell on plane q (zs is even)
            // plane q (and S of plane q - 1) arrive
            Stage<T> &v = st[h & 1];
            if constexpr (CO) {
                co.slot((q >> 1) + 2)[co.at[h & 1]] = v.co;
                // the prolongation kernels' weights and order of the sum
                const T *ck = co.slot(q >> 1), *c1 = co.slot((q >> 1) + ((h & 1) ? 1 : -1));
                const int row = ((y + 2) >> 1) + 1, A = CW * row + ((x + 2) >> 1) + 1, A1 = A + ((y & 1) ? CW : -CW);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T *a0 = ck + CW * CW * c + A, *a1 = ck + CW * CW * c + A1, *b0 = c1 + CW * CW * c + A,
                            *b1 = c1 + CW * CW * c + A1;
                    const T va = trilinear<T>(a0[0], a0[-1] + a1[0] + b0[0], a1[-1] + b0[-1] + b1[0], b1[-1]);
                    const T vb = trilinear<T>(a0[0], a0[1] + a1[0] + b0[0], a1[1] + b0[1] + b1[0], b1[1]);
                    v.b[c].a = v.b[c].a + va;
                    v.b[c].b = v.b[c].b + vb;
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (ZERO) continue;
                sh[O_R0 + (h * 3 + c) * RB + u] = par ? v.b[c].b : v.b[c].a;
                k[h][c] = par ? v.b[c].a : v.b[c].b;
                sh[O_K0 + (h * 3 + c) * RB + u] = k[h][c];
            }
            const T ek0 = par ? v.e.a : v.e.b;
            sh[O_ER + h * RB + u] = par ? v.e.b : v.e.a;
            sh[O_EK + h * RB + u] = ek0;
            T sr[3];
            if (RED) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {                   // plane q - 1 has the other parity
                    sr[c] = par ? v.s[c].a : v.s[c].b;
                    sk[h1][c] = par ? v.s[c].b : v.s[c].a;
                }
            }
            const unsigned o_m2 = off[h2];
            off[h2] = q + 2 < zend ? offset(q + 2, off[h3]) : off[h3];   // plane q + 2
            issue(v, off[h2], off[h3], h & 1, (q >> 1) + 3);    // ... and S of q + 1
            lds_barrier();
            // x-neighbours: of the red cell at q - 1 and of the black cell at
            // q - 2 alike, the same-row (and row +-1, plane +-1) partner on
            // the right at pair ix, on the left at ix - 1
            const int ix = u + (par ? 0 : 1);
            er[h1] = sh[O_ER + h1 * RB + u];
            const T ek2 = sh[O_EK + h2 * RB + u];
            if (RED) {
                const T *E0 = sh + O_EK + h1 * RB;
                if (ZERO) {
                    // S over the diagonal
                    Nbr<T> nb;
                    nb.e0 = er[h1], nb.e_zp = ek0, nb.e_zm = ek2;
                    nb.e_xp = E0[ix], nb.e_xm = E0[ix - 1], nb.e_yp = E0[u + MHW], nb.e_ym = E0[u - MHW];
                    T al[3];
                    alpha_core(nb, al);
#pragma unroll
                    for (int c = 0; c < 3; ++c) nw[h1][c] = relax_div(sr[c], fma(c2, al[c], T(1)));
                } else {
                    const T *R = sh + O_R0 + h1 * 3 * RB;
                    const T r0[3] = {R[u], R[RB + u], R[2 * RB + u]};
                    Nbr<T> nb;
                    nb.x0 = r0[0], nb.y0 = r0[1], nb.z0 = r0[2], nb.e0 = er[h1];
                    nb.e_zp = ek0, nb.e_zm = ek2;
                    nb.x_zp = k[h][0], nb.x_zm = k[h2][0], nb.y_zp = k[h][1], nb.y_zm = k[h2][1];
                    fill_faces<T, MHW, RB>(nb, sh + O_K0 + h1 * 3 * RB, E0, u, ix);
                    fill_corners<T, MHW, RB>(nb, R, u, ix);
                    nb.p = plane_edges<T, MHW, RB>(sh + O_R0 + h * 3 * RB, u, ix);
                    nb.m = plane_edges<T, MHW, RB>(sh + O_R0 + h2 * 3 * RB, u, ix);
                    T dv[3], al[3];
                    divF_core(nb, dv, al);
#pragma unroll
                    for (int c = 0; c < 3; ++c) nw[h1][c] = relax_point(r0[c], sr[c], dv[c], al[c], c8, c2);
                }
            }
            if (BLACK) {
                Nbr<T> nb;
                nb.x0 = k[h2][0], nb.y0 = k[h2][1], nb.z0 = k[h2][2], nb.e0 = ek2;
                nb.e_zp = er[h1], nb.e_zm = er[h3];
                nb.x_zp = nw[h1][0], nb.x_zm = nw[h3][0], nb.y_zp = nw[h1][1], nb.y_zm = nw[h3][1];
                fill_faces<T, MHW, RB>(nb, sh + O_R1 + (h & 1) * 3 * RB, sh + O_ER + h2 * RB, u, ix);
                if (ZERO) {
                    nb.x_xpyp = nb.x_xpym = nb.x_xmyp = nb.x_xmym = T(0);
                    nb.y_xpyp = nb.y_xpym = nb.y_xmyp = nb.y_xmym = T(0);
                } else {
                    fill_corners<T, MHW, RB>(nb, sh + O_K0 + h2 * 3 * RB, u, ix);
                    xk[h1] = plane_edges<T, MHW, RB>(sh + O_K0 + h1 * 3 * RB, u, ix);
                }
                nb.p = xk[h1], nb.m = xk[h3];
                T dv[3], al[3];
                divF_core(nb, dv, al);
                // plane q - 2 (its offset is in the slot that q + 2 takes)
                const unsigned oo = in && q - 2 >= z0 ? o_m2 / (unsigned)sizeof(T) * (unsigned)sizeof(TO) : 0xFFFFFFF0u;
                Pair<TO> o[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T kv = relax_point(k[h2][c], sk[h2][c], dv[c], al[c], c8, c2);
                    o[c].a = TO(par ? kv : nw[h2][c]);         // plane q - 2 has plane q's parity
                    o[c].b = TO(par ? nw[h2][c] : kv);
                }
                store_pair(O0, oo, o[0]);
                store_pair(O1, oo, o[1]);
                store_pair(O2, oo, o[2]);
            }
            // (after the black update's reads, which may then be issued early)
            if (RED) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sh[O_R1 + ((h1 & 1) * 3 + c) * RB + u] = nw[h1][c];
            }
        }
        q0 += 4;
    } while (q0 < zend);
}

template <typename T, typename TO, bool ZERO, bool CO>
__global__ void __launch_bounds__(MARCH_THREADS, 2)
k_march_sweep(MarchLists lists, const MarchTile *__restrict__ tiles, const int *__restrict__ bmap,
              const int *__restrict__ active, const double *__restrict__ inv_h2_p,
              const double *__restrict__ coef_p, double coef_v,
              const T *__restrict__ B, long long cs, const T *__restrict__ S, const T *__restrict__ eta,
              TO *__restrict__ out, unsigned obytes, const DenseProbDev *__restrict__ dp,
              const T *__restrict__ coarse, long long ccs)
{
    __shared__ T sh[ZERO ? N_ZERO : N_FULL];
    __shared__ T sco[CO ? 4 * CP : 1];
    __shared__ int place[MARCH_THREADS / 64];
    __shared__ int ids[16 * (MARCH_MAX_NBZ + 2)];
    const int xc = blockIdx.x % NXCD, seg = lists.first[xc] + (int)blockIdx.x / NXCD;
    if (seg >= lists.first[xc + 1]) return;
    const MarchTile &M = tiles[seg];
    const int pr = M.prob;
    if (active && !active[pr]) return;
    const T cih2 = T(coef_of(coef_p[pr], coef_v)) * T(inv_h2_p[pr]);
    const int nbx = M.nx, nby = M.ny, nbz = M.nz;
    const int ex = min(MT, 8 * (nbx - M.bx)), ey = min(MT, 8 * (nby - M.by));   // cells of the tile inside the box
    const int z0 = 8 * M.bz, n = 8 * M.nbz;
    // block at each position along the segment (one layer more on each side)
    // of the 4 x 4 columns the tile and its halo touch
    for (int t = threadIdx.x; t < 16 * (M.nbz + 2); t += MARCH_THREADS) {
        int i = M.bx - 1 + (t & 3), j = M.by - 1 + ((t >> 2) & 3), k = M.bz - 1 + (t >> 4);
        i = i < 0 ? i + nbx : i % nbx;
        j = j < 0 ? j + nby : j % nby;
        k = k < 0 ? k + nbz : k % nbz;
        ids[t] = bmap[M.map + i + nbx * (j + nby * k)];
    }
    CoarseRing<T> co{};
    if constexpr (CO) {
        const DenseProbDev g = dp[pr];
        auto wrap = [](int i, int n) { return i < 0 ? i + n : (i >= n ? i % n : i); };
        auto place_of = [&](int e) {     // element e of a plane: component, row, cell
            const int c = e / (CW * CW), m = e % (CW * CW);
            return (unsigned)(c * ccs + g.off + wrap(4 * M.bx - 2 + m % CW, g.nx) +
                              (long long)g.nx * wrap(4 * M.by - 2 + m / CW, g.ny)) * (unsigned)sizeof(T);
        };
        co.lds = sco;
        co.src = coarse;
        co.plane = (unsigned)(g.nx * g.ny) * (unsigned)sizeof(T);
        co.nz = g.nz;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            co.at[h] = CP / 2 * h + min((int)threadIdx.x, CP / 2 - 1);
            co.off[h] = place_of(co.at[h]);
        }
        // planes z0/2 - 2 to z0/2
        T first[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) first[m] = co.load(m & 1, z0 / 2 - 2 + m / 2);
#pragma unroll
        for (int m = 0; m < 6; ++m) co.slot(z0 / 2 - 2 + m / 2)[co.at[m & 1]] = first[m];
    }
    if ((threadIdx.x & 63) == 0) place[threadIdx.x >> 6] = __builtin_amdgcn_s_getreg(HWREG_PLACE);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    // the two inner wavefronts go to SIMDs 0 and 2 in a compute unit's first
    // group and to 1 and 3 in its second, so that they do not share one
    const int first = place[0], mine = place[threadIdx.x >> 6] >> 4;
    const bool spread = ((1 << (first >> 4)) | (1 << (place[1] >> 4)) | (1 << (place[2] >> 4)) |
                         (1 << (place[3] >> 4))) == 15;
    const int simd = (spread ? mine : (int)(threadIdx.x >> 6)) ^ (first & 1), role = (simd >> 1) | ((simd & 1) << 1);
    if (__builtin_amdgcn_readfirstlane(role) < 2) {
        // wavefronts of 8 rows of 8 pairs: the rows r, r + 4, r + 8 and r + 12
        // of 32 consecutive lanes start 8 elements apart modulo 32, so that
        // reads of a plane meet no bank twice (rows 0 to 7 and 8 to 15
        // instead: FP32 sweep of 128^3 34.9 instead of 29.2 us)
        const int r = 2 * role + (lane >> 5) + 4 * ((lane >> 3) & 3), x = 2 * (lane & 7);
        march_loop<T, TO, ROLE_INNER, ZERO, CO>(sh, ids, B, cs, S, eta, out, obytes, cih2, min(x, ex - 2), min(r, ey - 1), z0, n,
                                      x < ex && r < ey, co);
    } else if (__builtin_amdgcn_readfirstlane(role) == 2) {
        // red cells of the first halo layer that face the tile
        const int l = min(lane, 47);
        const int x = l < 16 ? min(2 * (l & 7), ex - 2) : (l < 32 ? -2 : ex),
                  y = l < 16 ? (l < 8 ? -1 : ey) : min(l & 15, ey - 1);
        march_loop<T, TO, ROLE_RING, ZERO, CO>(sh, ids, B, cs, S, eta, out, obytes, cih2, x, y, z0, n, false, co);
    } else {
        // the rest of the halo: rows -2 and ey + 1, the corners of rows -1 and ey
        const int l = min(lane, 23);
        const int x = l < 20 ? min(2 * (l % 10) - 2, ex) : ((l & 1) ? ex : -2),
                  y = l < 20 ? (l < 10 ? -2 : ey + 1) : (l < 22 ? -1 : ey);
        march_loop<T, TO, ROLE_LOAD, ZERO, CO>(sh, ids, B, cs, S, eta, out, obytes, cih2, x, y, z0, n, false, co);
    }
}

// ---------------------------------------------------------------------------
// Plane-marching operator (eqs. 8-11) of the base level: L B, the residual and
// what the block stencil kernel computes with them, on the same column
// segments.  At step q plane q of B and eta with a halo of one cell goes to a
// ring of four in LDS, and plane q - 1 is computed and written: a thread's
// own column above and below is in its registers, and a z face's flux is
// formed once for the two planes it separates.  The sums are those of the
// block stencil kernel on the same values, hence the same bits.
//
// A wavefront takes one block's 8 x 8 cells of the plane (its loads and stores
// are whole runs of 64 cells), plus one array's halo cells around the tile.
// Rows of 24 elements in LDS: the rows of 8 consecutive cells that a read
// touches at once start 8 apart modulo 16 (32 in FP32), no bank meets twice.
//
// What bounds it: HBM, at the rate of a large copy.  Per cell it asks for 1.1
// instead of 2.3 lines of each array, two planes ahead.  Per launch on one box,
// us, per block -> this kernel: FP64 128^3 with two dot products 42.3 -> 38.0
// (4.9 TB/s of algorithmic bytes), residual + restriction 33.8 -> 26.7,
// residual 40.7 -> 35.8; 256^3 L B 305 -> 216 (4.4 TB/s); 64 FP32 problems of
// 16^3 to 64^3, residual + restriction 41.2 -> 34.7.  A dot product adds up per
// lane over a block's eight planes: one reduction over the lanes per block (one
// per plane instead: 40.0 us).
// ---------------------------------------------------------------------------
constexpr int SW = 24, SP = SW * (MT + 2);   // row and plane of one array in LDS

// the value of lane l ^ 1 (quad permutation 1, 0, 3, 2) or l ^ 8 (rotation of
// the 16 lanes of a row by 8)
constexpr int LANES_XOR1 = 0xB1, LANES_XOR8 = 0x128;
template <int CTRL>
__device__ __forceinline__ float lanes(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double lanes(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true),
                   hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// this thread's cell of a plane, and the z face below it: differences of B_x and
// B_y across it and along x and y, sum of the resistivity
template <typename T>
struct Plane {
    T b[3], e, fx, fy, Ez;
};

template <typename T, int MODE, bool DOTS>
__global__ void __launch_bounds__(MARCH_THREADS, 2)
k_march_stencil(MarchLists lists, const MarchTile *__restrict__ tiles, const int *__restrict__ bmap,
                const int *__restrict__ active, const double *__restrict__ inv_h2_p,
              const double *__restrict__ coef_p, double coef_v,
                const T *__restrict__ B, long long cs, const T *S, const T *__restrict__ eta, T *out, unsigned obytes,
                StencilDots dots, unsigned pbytes, const int *__restrict__ dense_map,
                const DenseProbDev *__restrict__ dp, long long ccs)
{
    constexpr bool HAS_S = MODE != MODE_APPLY || DOTS, RESTRICT = MODE == MODE_RESID_RESTRICT;
    constexpr int NID = 16 * (MARCH_MAX_NBZ + 2);
    __shared__ T sh[4][4][SP];
    __shared__ int ids[NID];
    __shared__ int cmap[RESTRICT ? NID : 1];
    const int xc = blockIdx.x % NXCD, seg = lists.first[xc] + (int)blockIdx.x / NXCD;
    if (seg >= lists.first[xc + 1]) return;
    const MarchTile &M = tiles[seg];
    const int pr = M.prob;
    const int nbx = M.nx, nby = M.ny, nbz = M.nz;
    const bool on = !(active && !active[pr]);
    const int ex = min(MT, 8 * (nbx - M.bx)), ey = min(MT, 8 * (nby - M.by));
    const int z0 = 8 * M.bz, n = 8 * M.nbz;
    for (int t = threadIdx.x; t < 16 * (M.nbz + 2); t += MARCH_THREADS) {
        int i = M.bx - 1 + (t & 3), j = M.by - 1 + ((t >> 2) & 3), k = M.bz - 1 + (t >> 4);
        i = i < 0 ? i + nbx : i % nbx;
        j = j < 0 ? j + nby : j % nby;
        k = k < 0 ? k + nbz : k % nbz;
        const int b = bmap[M.map + i + nbx * (j + nby * k)];
        ids[t] = b;
        if (RESTRICT) cmap[t] = dense_map[b];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool in = 8 * (wv & 1) < ex && 8 * (wv >> 1) < ey;   // this wavefront's block is in the box
    const int x = (in ? 8 * (wv & 1) : 0) + (lane & 7), y = (in ? 8 * (wv >> 1) : 0) + (lane >> 3);
    if (!on) {   // an inactive problem contributes nothing
        if (DOTS && in)
            for (int t = lane; t < M.nbz * dots.ndot; t += 64)
                dots.dot_part[(long long)ids[((x + 8) >> 3) + 4 * ((y + 8) >> 3) + 16 * (t / dots.ndot + 1)] * dots.ndot +
                              t % dots.ndot] = 0.0;
        return;
    }
    const T c8 = uniform(T(coef_of(coef_p[pr], coef_v)) * T(inv_h2_p[pr]) * T(0.125));
    // halo cells: the lanes of wavefront k load array k around the tile, four
    // lanes (of each, for B_x and B_y) the tile's edges
    const int l = lane & 15;
    const int hx = lane < 32 ? min(l, ex - 1) : (lane < 48 ? -1 : ex), hy = lane < 32 ? (lane < 16 ? -1 : ey) : min(l, ey - 1);
    const int cx = (lane & 1) ? ex : -1, cy = (lane & 2) ? ey : -1;
    const T *H = wv == 3 ? eta : B + wv * cs, *C = B + (wv & 1) * cs;
    const int u = (x + 1) + SW * (y + 1), uh = (hx + 1) + SW * (hy + 1), uc = (cx + 1) + SW * (cy + 1);
    const T *B0 = B, *B1 = B + cs, *B2 = B + 2 * cs, *S0 = S, *S1 = S + cs, *S2 = S + 2 * cs;
    const long long os = RESTRICT ? ccs : cs;
    const __amdgpu_buffer_rsrc_t O0 = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)obytes, 0x00027000),
                                 O1 = __builtin_amdgcn_make_buffer_rsrc(out + os, 0, (int)obytes, 0x00027000),
                                 O2 = __builtin_amdgcn_make_buffer_rsrc(out + 2 * os, 0, (int)obytes, 0x00027000),
                                 OP = __builtin_amdgcn_make_buffer_rsrc(dots.dot_part, 0, (int)pbytes, 0x00027000);
    struct Stage1 {
        T b[3], e, h, c, s[3];
    } st[2];
    struct Off {
        unsigned own, halo, edge;
    };
    const int zs = z0 - 1, zend = z0 + n + 1;                  // planes zs .. zend - 1
    constexpr unsigned PLANE = 64 * (unsigned)sizeof(T);
    auto column = [](int a, int b) { return ((a + 8) >> 3) + 4 * ((b + 8) >> 3); };
    const int io = column(x, y), ih = column(hx, hy), ic = column(cx, cy);
    auto at = [&](int i, int cell, int P) {
        const unsigned b = (unsigned)ids[i + 16 * (((P - z0) >> 3) + 1)];
        return (b * (unsigned)NC + (unsigned)(cell + 64 * (P & 7))) * (unsigned)sizeof(T);
    };
    auto cell = [](int a, int b) { return (a & 7) + 8 * (b & 7); };
    const int lo = cell(x, y), lh = cell(hx, hy), lc = cell(cx, cy);
    auto next = [&](Off o, int P) -> Off {                     // offsets on plane P, given those on plane P - 1
        if ((P & 7) == 0) return {at(io, lo, P), at(ih, lh, P), at(ic, lc, P)};
        return {o.own + PLANE, o.halo + PLANE, o.edge + PLANE};
    };
    auto issue = [&](Stage1 &v, const Off &o, unsigned offs) {
        v.b[0] = load_at(B0, o.own);
        v.b[1] = load_at(B1, o.own);
        v.b[2] = load_at(B2, o.own);
        v.e = load_at(eta, o.own);
        v.h = load_at(H, o.halo);
        v.c = load_at(C, o.edge);
        if (HAS_S) {
            v.s[0] = load_at(S0, offs);
            v.s[1] = load_at(S1, offs);
            v.s[2] = load_at(S2, offs);
        }
    };
    Off o1 = {at(io, lo, zs), at(ih, lh, zs), at(ic, lc, zs)};
    unsigned own[4];                                           // offset of the thread's cell by plane mod 4
    own[0] = o1.own;
    issue(st[0], o1, own[0]);
    __builtin_amdgcn_sched_barrier(0);
    o1 = next(o1, zs + 1);
    own[1] = o1.own;
    issue(st[1], o1, own[0]);
    __builtin_amdgcn_sched_barrier(0);
    own[2] = own[3] = 0;
    Plane<T> pl[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) pl[h] = Plane<T>{};
    double sum[2] = {0.0, 0.0};
    T acc[3] = {T(0), T(0), T(0)};
    const int nd = DOTS ? dots.ndot : 0, qy = DOTS && dots.dot_y[0] ? 0 : 1;
    const int ccell = RESTRICT ? ((lane & 7) >> 1) + dp[pr].nx * (lane >> 4) : 0, cnxy = RESTRICT ? dp[pr].nx * dp[pr].ny : 0;
    int q0 = zs;
    do {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if (h == 2 && q0 + 2 >= zend) break;               // (a segment has 8 n + 2 planes)
            __builtin_amdgcn_sched_barrier(0);
            const int q = q0 + h;
            const int h1 = (h + 3) & 3, h2 = (h + 2) & 3;      // planes q - 1, q - 2
            Stage1 &v = st[h & 1];
            T(*L)[SP] = sh[h];
            Plane<T> &N = pl[h];
            const Plane<T> &P = pl[h1], &Q = pl[h2];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                N.b[c] = v.b[c];
                L[c][u] = N.b[c];
            }
            N.e = v.e;
            L[3][u] = N.e;
            L[wv][uh] = v.h;
            L[wv & 1][uc] = v.c;
            T s[3];
            if (HAS_S)
#pragma unroll
                for (int c = 0; c < 3; ++c) s[c] = v.s[c];
            if (q + 2 < zend) o1 = next(o1, q + 2);
            own[h2] = o1.own;                                  // (plane q - 2's slot)
            issue(v, o1, own[(h + 1) & 3]);
            lds_barrier();
            const T m4 = T(-4);
            const T *Z0 = sh[h][2] + u, *X = sh[h1][0] + u, *Y = sh[h1][1] + u, *Z = sh[h1][2] + u, *E = sh[h1][3] + u;
            const T Exp = P.e + E[1], Exm = E[-1] + P.e, Eyp = P.e + E[SW], Eym = E[-SW] + P.e;
            const T z_xp = Z[1], z_xm = Z[-1], z_yp = Z[SW], z_ym = Z[-SW];
            const T x_yp = X[SW], x_ym = X[-SW], y_xp = Y[1], y_xm = Y[-1];
            N.fx = fma(m4, N.b[0] - P.b[0], (z_xp - z_xm) + (Z0[1] - Z0[-1]));
            N.fy = fma(m4, N.b[1] - P.b[1], (z_yp - z_ym) + (Z0[SW] - Z0[-SW]));
            N.Ez = P.e + N.e;
            T dv[3];
            {
                const T D = y_xp - y_xm;
                const T tp = D + (Y[SW + 1] - Y[SW - 1]), tm = (Y[-SW + 1] - Y[-SW - 1]) + D;
                const T gy = fma(Eyp, fma(m4, x_yp - P.b[0], tp), -(Eym * fma(m4, P.b[0] - x_ym, tm)));
                dv[0] = gy + fma(N.Ez, N.fx, -(P.Ez * P.fx));
            }
            {
                const T D = x_yp - x_ym;
                const T tp = D + (X[SW + 1] - X[-SW + 1]), tm = (X[SW - 1] - X[-SW - 1]) + D;
                const T gx = fma(Exp, fma(m4, y_xp - P.b[1], tp), -(Exm * fma(m4, P.b[1] - y_xm, tm)));
                dv[1] = gx + fma(N.Ez, N.fy, -(P.Ez * P.fy));
            }
            {
                const T *X0 = sh[h][0] + u, *X2 = sh[h2][0] + u, *Y0 = sh[h][1] + u, *Y2 = sh[h2][1] + u;
                const T D = N.b[0] - Q.b[0];
                const T tp = D + (X0[1] - X2[1]), tm = (X0[-1] - X2[-1]) + D;
                const T gx = fma(Exp, fma(m4, z_xp - P.b[2], tp), -(Exm * fma(m4, P.b[2] - z_xm, tm)));
                const T D2 = N.b[1] - Q.b[1];
                const T tp2 = D2 + (Y0[SW] - Y2[SW]), tm2 = (Y0[-SW] - Y2[-SW]) + D2;
                const T gy = fma(Eyp, fma(m4, z_yp - P.b[2], tp2), -(Eym * fma(m4, P.b[2] - z_ym, tm2)));
                dv[2] = gx + gy;
            }
            const int p = q - 1;
            const bool mine = in && p >= z0;
            T r[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T LB = fma(c8, dv[c], P.b[c]);
                r[c] = MODE == MODE_APPLY ? LB : (MODE == MODE_MEAN ? T(0.5) * (s[c] + LB) : s[c] - LB);
            }
            if (RESTRICT) {
                // the mean of 8 children in the order of the restriction kernel
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T r8 = lanes<LANES_XOR8>(r[c]);
                    acc[c] = (h & 1) ? acc[c] + r[c] : r[c];   // plane p is even on even h
                    acc[c] += lanes<LANES_XOR1>(r[c]);
                    acc[c] += r8;
                    acc[c] += lanes<LANES_XOR1>(r8);
                }
                if (h & 1) {
                    const int cell = cmap[io + 16 * (((p - z0) >> 3) + 1)] + ccell + cnxy * ((p & 7) >> 1);
                    const unsigned oc = mine && (lane & 9) == 0 ? (unsigned)cell * (unsigned)sizeof(T) : 0xFFFFFFF0u;
                    store_one(O0, oc, acc[0] * T(0.125));
                    store_one(O1, oc, acc[1] * T(0.125));
                    store_one(O2, oc, acc[2] * T(0.125));
                }
            } else {
                const unsigned oo = mine ? own[h1] : 0xFFFFFFF0u;
                store_one(O0, oo, r[0]);
                store_one(O1, oo, r[1]);
                store_one(O2, oo, r[2]);
            }
            if (DOTS) {
                // each lane its column of the block, then the 64 lanes
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    if (d >= nd) continue;
                    double a = 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) a = fma((double)r[c], d == qy ? (double)s[c] : (double)r[c], a);
                    sum[d] = h == 2 && (p & 7) == 0 ? a : sum[d] + a;   // p = z0 - 2 + h + 4 i
                    if (h == 1 && (p & 7) == 7) {
                        double v = sum[d];
                        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
                        store_one(OP, mine && lane == 0 ? (own[h1] / PLANE / 8 * nd + d) * 8u : 0xFFFFFFF0u, v);
                    }
                }
            }
        }
        q0 += 4;
    } while (q0 < zend);
}

}  // namespace

template <typename T, typename TO>
ohm_status launch_march_sweep(const ohm_hier *h, const T *B, long long cs, const T *S, const T *eta,
                              Coef coef_dev, TO *out, const int *active, hipStream_t s, const T *coarse,
                              long long ccs)
{
    const AmrLevelDev &L = h->amr[0];
    const unsigned obytes = (unsigned)((unsigned long long)L.nb * NC * sizeof(TO));   // (the callers allow 4 GiB)
    const MarchTile *tiles = (const MarchTile *)L.march;
#define RUN(zero, co) k_march_sweep<T, TO, zero, co><<<NXCD * L.mlists.longest, MARCH_THREADS, 0, s>>>(L.mlists, tiles, L.bmap, active, \
        L.inv_h2, coef_dev.p, coef_dev.v, B, cs, S, eta, out, obytes, h->dense[1].probs, coarse, ccs)
    if (!B) RUN(true, false);
    else if (coarse) RUN(false, true);
    else RUN(false, false);
#undef RUN
    return check_launch("marching sweep");
}
#define INST(T, TO)                                                                                              \
    template ohm_status launch_march_sweep<T, TO>(const ohm_hier *, const T *, long long, const T *, const T *, \
                                                  Coef, TO *, const int *, hipStream_t, const T *, long long);
INST(double, double)
INST(float, float)
INST(float, double)
#undef INST

template <typename T>
ohm_status launch_march_stencil(const ohm_hier *h, int mode, const T *B, long long cs, const T *S, const T *eta,
                                Coef coef_dev, T *out, long long ccs, const int *active, hipStream_t s,
                                StencilDots dots)
{
    const AmrLevelDev &L = h->amr[0];
    const unsigned long long cells = mode == MODE_RESID_RESTRICT ? ccs : (long long)L.nb * NC;
    const unsigned obytes = (unsigned)(cells * sizeof(T));
    const unsigned pbytes = (unsigned)((unsigned long long)L.nb * dots.ndot * sizeof(double));
    const MarchTile *tiles = (const MarchTile *)L.march;
#define RUN(mode, d, S) k_march_stencil<T, mode, d><<<NXCD * L.mlists.longest, MARCH_THREADS, 0, s>>>(L.mlists, tiles, L.bmap, active, \
        L.inv_h2, coef_dev.p, coef_dev.v, B, cs, S, eta, out, obytes, dots, pbytes, L.dense_map, h->dense[1].probs, ccs)
    switch (mode) {
    case MODE_APPLY:
        if constexpr (std::is_same<T, double>::value)
            if (dots.ndot > 0) {
                RUN(MODE_APPLY, true, (dots.dot_y[0] ? dots.dot_y[0] : dots.dot_y[1]));
                break;
            }
        RUN(MODE_APPLY, false, S);
        break;
    case MODE_RESID: RUN(MODE_RESID, false, S); break;
    case MODE_MEAN: RUN(MODE_MEAN, false, out); break;
    case MODE_RESID_RESTRICT: RUN(MODE_RESID_RESTRICT, false, S); break;
    default: return fail(OHM_ERR_ARG, "unknown marching mode %d", mode);
    }
#undef RUN
    return check_launch("marching stencil");
}
#define INST(T)                                                                                                    \
    template ohm_status launch_march_stencil<T>(const ohm_hier *, int, const T *, long long, const T *, const T *, \
                                                Coef, T *, long long, const int *, hipStream_t, StencilDots);
INST(double)
INST(float)
#undef INST

}  // namespace ohm
