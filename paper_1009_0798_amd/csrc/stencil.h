// Device-side discrete operator of eqs. (8)-(11) and the smoother diagonal of
// eqs. (21)-(23), on a box of cells with rows of W cells and planes of P cells
// (a cube unless given) held in fast memory (LDS tile or registers).
#pragma once

namespace ohm {

// All three components at index p of the box, every neighbour read once:
//   dv[c] = 8 h^2 (div F)_c  and  al[c] = 2 h^2 alpha_c / lam_dt.
// Face fluxes are written without their power-of-two factors: with E the sum of
// the two cell resistivities at a face (twice the mean of eq. 11), t the
// transverse four-point sum (four times the difference of eq. 10) and n the
// normal difference (eq. 9), 8 h F = E (t - 4 n); scaling by 2, 4 or 8 is exact,
// so the callers fold the factors into their coefficients.  (The sums are
// spelled out in fused operations where a compiler could choose which product
// to fuse: every kernel's values are the same.)  The central
// difference of B_d along c at p is shared by the +d and -d faces.
template <typename T, int W, int P = W * W>
__device__ __forceinline__ void divF_all(const T *__restrict__ Bx, const T *__restrict__ By, const T *__restrict__ Bz,
                                         const T *__restrict__ E, int p, T dv[3], T al[3])
{
    constexpr int ox = 1, oy = W, oz = P;
    const T m4 = T(-4);
    const T e0 = E[p];
    const T Exp = e0 + E[p + ox], Exm = E[p - ox] + e0, Eyp = e0 + E[p + oy], Eym = E[p - oy] + e0,
            Ezp = e0 + E[p + oz], Ezm = E[p - oz] + e0;
    const T x0 = Bx[p], y0 = By[p], z0 = Bz[p];
    const T x_yp = Bx[p + oy], x_ym = Bx[p - oy], x_zp = Bx[p + oz], x_zm = Bx[p - oz];
    const T y_xp = By[p + ox], y_xm = By[p - ox], y_zp = By[p + oz], y_zm = By[p - oz];
    const T z_xp = Bz[p + ox], z_xm = Bz[p - ox], z_yp = Bz[p + oy], z_ym = Bz[p - oy];
    {   // component x: faces +-y (transverse d_x B_y) and +-z (d_x B_z)
        const T D = y_xp - y_xm;
        const T tp = D + (By[p + oy + ox] - By[p + oy - ox]), tm = (By[p - oy + ox] - By[p - oy - ox]) + D;
        const T gy = fma(Eyp, fma(m4, x_yp - x0, tp), -(Eym * fma(m4, x0 - x_ym, tm)));
        const T D2 = z_xp - z_xm;
        const T tp2 = D2 + (Bz[p + oz + ox] - Bz[p + oz - ox]), tm2 = (Bz[p - oz + ox] - Bz[p - oz - ox]) + D2;
        const T gz = fma(Ezp, fma(m4, x_zp - x0, tp2), -(Ezm * fma(m4, x0 - x_zm, tm2)));
        dv[0] = gy + gz;
    }
    {   // component y: faces +-x (d_y B_x) and +-z (d_y B_z)
        const T D = x_yp - x_ym;
        const T tp = D + (Bx[p + ox + oy] - Bx[p + ox - oy]), tm = (Bx[p - ox + oy] - Bx[p - ox - oy]) + D;
        const T gx = fma(Exp, fma(m4, y_xp - y0, tp), -(Exm * fma(m4, y0 - y_xm, tm)));
        const T D2 = z_yp - z_ym;
        const T tp2 = D2 + (Bz[p + oz + oy] - Bz[p + oz - oy]), tm2 = (Bz[p - oz + oy] - Bz[p - oz - oy]) + D2;
        const T gz = fma(Ezp, fma(m4, y_zp - y0, tp2), -(Ezm * fma(m4, y0 - y_zm, tm2)));
        dv[1] = gx + gz;
    }
    {   // component z: faces +-x (d_z B_x) and +-y (d_z B_y)
        const T D = x_zp - x_zm;
        const T tp = D + (Bx[p + ox + oz] - Bx[p + ox - oz]), tm = (Bx[p - ox + oz] - Bx[p - ox - oz]) + D;
        const T gx = fma(Exp, fma(m4, z_xp - z0, tp), -(Exm * fma(m4, z0 - z_xm, tm)));
        const T D2 = y_zp - y_zm;
        const T tp2 = D2 + (By[p + oy + oz] - By[p + oy - oz]), tm2 = (By[p - oy + oz] - By[p - oy - oz]) + D2;
        const T gy = fma(Eyp, fma(m4, z_yp - z0, tp2), -(Eym * fma(m4, z0 - z_ym, tm2)));
        dv[2] = gx + gy;
    }
    const T sx = Exm + Exp, sy = Eym + Eyp, sz = Ezm + Ezp;
    al[0] = sy + sz;
    al[1] = sx + sz;
    al[2] = sx + sy;
}

// What one plane contributes to the applications at the cells above and below
// it: of the values around the column's cell on that plane, the differences of
// B_z along x and y, B_x on either side in x and B_y on either side in y.
template <typename T>
struct PlaneEdges {
    T zx, zy, x_xp, x_xm, y_yp, y_ym;
};

// The values one application reads around a cell: B_c at the cell (x0, y0, z0),
// a_bs = component a at the neighbour on side s of axis b, a_bscs at the edge
// neighbour in the plane, the plane above (p) and below (m), and the
// resistivity e at the cell and its six faces.
template <typename T>
struct Nbr {
    T x0, y0, z0, e0, e_xp, e_xm, e_yp, e_ym, e_zp, e_zm;
    T x_yp, x_ym, x_zp, x_zm, y_xp, y_xm, y_zp, y_zm, z_xp, z_xm, z_yp, z_ym;
    T x_xpyp, x_xpym, x_xmyp, x_xmym, y_xpyp, y_xpym, y_xmyp, y_xmym;
    PlaneEdges<T> p, m;
};

// al (as divF_all) from those values
template <typename T>
__device__ __forceinline__ void alpha_core(const Nbr<T> &n, T al[3])
{
    const T sx = (n.e_xm + n.e0) + (n.e0 + n.e_xp), sy = (n.e_ym + n.e0) + (n.e0 + n.e_yp),
            sz = (n.e_zm + n.e0) + (n.e0 + n.e_zp);
    al[0] = sy + sz;
    al[1] = sx + sz;
    al[2] = sx + sy;
}

// dv and al (as divF_all) from those values
template <typename T>
__device__ __forceinline__ void divF_core(const Nbr<T> &n, T dv[3], T al[3])
{
    const T m4 = T(-4);
    const T Exp = n.e0 + n.e_xp, Exm = n.e_xm + n.e0, Eyp = n.e0 + n.e_yp, Eym = n.e_ym + n.e0, Ezp = n.e0 + n.e_zp,
            Ezm = n.e_zm + n.e0;
    {   // component x: faces +-y (transverse d_x B_y) and +-z (d_x B_z)
        const T D = n.y_xp - n.y_xm;
        const T tp = D + (n.y_xpyp - n.y_xmyp), tm = (n.y_xpym - n.y_xmym) + D;
        const T gy = fma(Eyp, fma(m4, n.x_yp - n.x0, tp), -(Eym * fma(m4, n.x0 - n.x_ym, tm)));
        const T D2 = n.z_xp - n.z_xm;
        const T tp2 = D2 + n.p.zx, tm2 = n.m.zx + D2;
        const T gz = fma(Ezp, fma(m4, n.x_zp - n.x0, tp2), -(Ezm * fma(m4, n.x0 - n.x_zm, tm2)));
        dv[0] = gy + gz;
    }
    {   // component y: faces +-x (d_y B_x) and +-z (d_y B_z)
        const T D = n.x_yp - n.x_ym;
        const T tp = D + (n.x_xpyp - n.x_xpym), tm = (n.x_xmyp - n.x_xmym) + D;
        const T gx = fma(Exp, fma(m4, n.y_xp - n.y0, tp), -(Exm * fma(m4, n.y0 - n.y_xm, tm)));
        const T D2 = n.z_yp - n.z_ym;
        const T tp2 = D2 + n.p.zy, tm2 = n.m.zy + D2;
        const T gz = fma(Ezp, fma(m4, n.y_zp - n.y0, tp2), -(Ezm * fma(m4, n.y0 - n.y_zm, tm2)));
        dv[1] = gx + gz;
    }
    {   // component z: faces +-x (d_z B_x) and +-y (d_z B_y)
        const T D = n.x_zp - n.x_zm;
        const T tp = D + (n.p.x_xp - n.m.x_xp), tm = (n.p.x_xm - n.m.x_xm) + D;
        const T gx = fma(Exp, fma(m4, n.z_xp - n.z0, tp), -(Exm * fma(m4, n.z0 - n.z_xm, tm)));
        const T D2 = n.y_zp - n.y_zm;
        const T tp2 = D2 + (n.p.y_yp - n.m.y_yp), tm2 = (n.p.y_ym - n.m.y_ym) + D2;
        const T gy = fma(Eyp, fma(m4, n.z_yp - n.z0, tp2), -(Eym * fma(m4, n.z0 - n.z_ym, tm2)));
        dv[2] = gx + gy;
    }
    const T sx = Exm + Exp, sy = Eym + Eyp, sz = Ezm + Ezp;
    al[0] = sy + sz;
    al[1] = sx + sz;
    al[2] = sx + sy;
}

// The in-plane face values of a cell from its plane f [component][row][pair]
// (rows of W pairs, RB elements per component) and the resistivity plane e:
// ix is the pair of the +x partner, ix - 1 of the -x one, u the cell's own.
template <typename T, int W, int RB>
__device__ __forceinline__ void fill_faces(Nbr<T> &n, const T *f, const T *e, int u, int ix)
{
    n.e_xp = e[ix], n.e_xm = e[ix - 1], n.e_yp = e[u + W], n.e_ym = e[u - W];
    n.x_yp = f[u + W], n.x_ym = f[u - W];
    n.y_xp = f[RB + ix], n.y_xm = f[RB + ix - 1];
    n.z_xp = f[2 * RB + ix], n.z_xm = f[2 * RB + ix - 1], n.z_yp = f[2 * RB + u + W], n.z_ym = f[2 * RB + u - W];
}

// The in-plane edge values of a cell from its plane c, laid out as above.
template <typename T, int W, int RB>
__device__ __forceinline__ void fill_corners(Nbr<T> &n, const T *c, int u, int ix)
{
    n.x_xpyp = c[ix + W], n.x_xpym = c[ix - W], n.x_xmyp = c[ix - 1 + W], n.x_xmym = c[ix - 1 - W];
    n.y_xpyp = c[RB + ix + W], n.y_xpym = c[RB + ix - W], n.y_xmyp = c[RB + ix - 1 + W], n.y_xmym = c[RB + ix - 1 - W];
}

// What plane c contributes to the cells above and below, laid out as above.
template <typename T, int W, int RB>
__device__ __forceinline__ PlaneEdges<T> plane_edges(const T *c, int u, int ix)
{
    return {c[2 * RB + ix] - c[2 * RB + ix - 1], c[2 * RB + u + W] - c[2 * RB + u - W], c[ix], c[ix - 1],
            c[RB + u + W], c[RB + u - W]};
}

// al[c] = 2 h^2 alpha_c / lam_dt alone (same sums as divF_all)
template <typename T, int W, int P = W * W>
__device__ __forceinline__ void alpha_all(const T *__restrict__ E, int p, T al[3])
{
    const T e0 = E[p];
    const T sx = (E[p - 1] + e0) + (e0 + E[p + 1]), sy = (E[p - W] + e0) + (e0 + E[p + W]),
            sz = (E[p - P] + e0) + (e0 + E[p + P]);
    al[0] = sy + sz;
    al[1] = sx + sz;
    al[2] = sx + sy;
}

// n / d for d >= 1 (the smoother's diagonal): hardware reciprocal, Newton steps
// (two in FP64, none in FP32) and one residual correction of the quotient; the
// result is within about one unit in the last place of the rounded quotient.
__device__ __forceinline__ float relax_div(float n, float d)
{
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = n * r;
    return fmaf(fmaf(-d, q, n), r, q);
}
__device__ __forceinline__ double relax_div(double n, double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double q = n * r;
    return fma(fma(-d, q, n), r, q);
}

// One point update of eq. (19) for the three components at p: with
// c8 = lam dt / (8 h^2) and c2 = lam dt / (2 h^2),
// B_c + (S_c - (B_c + c8 dv_c)) / (1 + c2 al_c).
template <typename T>
__device__ __forceinline__ T relax_point(T b, T s, T dv, T al, T c8, T c2)
{
    return b + relax_div(s - fma(c8, dv, b), fma(c2, al, T(1)));
}

// Trilinear prolongation: c the parent, s1, s2 and c3 the sums of its
// neighbours on the child's side across one, two and three axes.
template <typename T>
__device__ __forceinline__ T trilinear(T c, T s1, T s2, T c3)
{
    return (fma(T(3), s2, fma(T(9), s1, T(27) * c)) + c3) * T(1.0 / 64.0);
}

}  // namespace ohm
