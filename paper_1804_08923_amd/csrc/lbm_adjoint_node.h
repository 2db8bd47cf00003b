// Per-node forward recomputation and its vector-Jacobian product (reverse
// mode), for the adjoint of one time step.  Host and device code, templated on
// the arithmetic type R: the adjoint kernels run them in FP32 (the derivative
// coefficients need no cancellation-free sums), a host build runs them in
// FP64 or FP32 for checking.
//
// The node map (Sec. II; the reduced collision of lbm_kernels.h) takes
//   d_i   = f_i - w_i rho_b0        the 27 colour-blind pre-collision deviations
//                                   (through their moments up to second order),
//   phic  = phi at the node          (Eq. order),
//   xr    = rho_r / rho at the node,
//   g     = (grad phi, grad rho)     the isotropic stencil gradients,
// and returns the colour-blind post-collision populations
//   f'_i = f^(e)_i + F'_i/2 + Delta_i + Omega^(2)_i
// (Eq. EES with Eq. Phi, Eq. ketFd, the relaxed deviatoric central moments
// Delta, Eq. perturb) and the recoloured red and blue populations
//   f^r*_i = xr f'_i + (w_i/|c_i|) c_i . V,   f^b*_i = f'_i - f^r*_i,
//   V = beta xr (1 - xr) rho kappa(alpha_bar) grad phi / |grad phi|   (Eqs. op3r/op3b).
// node_vjp() returns, for cotangents (Lr, Lb) of (f^r*, f^b*), the cotangents
// of d, phic, xr and g; perturb_vjp() that of the perturbation strength A.
#pragma once
#include "lbm_kernels.h"

#define CG_HD __host__ __device__ __forceinline__

namespace cglbm {

// one-dimensional inverse central-moment basis over c = -1, 0, 1 (index c + 1)
// for shift u; d h0/du = h1 and d h1/du = 2 h2.
template <class R>
struct Basis1T {
    R h0[3], h1[3];
    CG_HD explicit Basis1T(R u)
    {
        h0[0] = R(0.5) * (u * u - u);
        h0[1] = R(1) - u * u;
        h0[2] = R(0.5) * (u * u + u);
        h1[0] = u - R(0.5);
        h1[1] = R(-2) * u;
        h1[2] = u + R(0.5);
    }
};
template <class R>
CG_HD constexpr R h2r(int j) { return j == 1 ? R(-1) : R(0.5); }  // index j = c + 1

// raw moments of the deviations up to second order
template <class R>
struct MomT {
    R m0 = 0, j[3] = {0, 0, 0}, P[6] = {0, 0, 0, 0, 0, 0};  // P: xx yy zz xy xz yz
    CG_HD void add(int i, R v)
    {
        m0 += v;
        if (kCX[i]) { j[0] += kCX[i] * v; P[0] += v; }
        if (kCY[i]) { j[1] += kCY[i] * v; P[1] += v; }
        if (kCZ[i]) { j[2] += kCZ[i] * v; P[2] += v; }
        if (kCX[i] * kCY[i]) P[3] += (kCX[i] * kCY[i]) * v;
        if (kCX[i] * kCZ[i]) P[4] += (kCX[i] * kCZ[i]) * v;
        if (kCY[i] * kCZ[i]) P[5] += (kCY[i] * kCZ[i]) * v;
    }
};

// forward quantities of one node that the reverse sweep needs
template <class R>
struct NodeFwdT {
    R m0, rho, u[3], F[3], gp[3], gr[3];
    R nub, s2, abar, kap, om;
    R q[6];   // second central moments of f - f^(e) + F'/2: xx, yy, zz, xy, xz, yz
    R tr;     // (q_xx + q_yy + q_zz) / 3
    R kk[6];  // relaxed and scaled: (1 - s2) q_ab (off-diagonal), (1 - s2)(q_aa - tr)
    R gn;     // |grad phi| (0 when switched off)
    R n[3];   // grad phi / |grad phi| (0 when switched off)
    bool on;  // |grad phi|^2 > eps^2
};

template <class R>
CG_HD void node_fwd(const KP& k, const MomT<R>& M, R phic, const double* g, NodeFwdT<R>& f)
{
    f.m0 = M.m0;
    f.rho = (R)k.rho_b0 + M.m0;
    const R hp = R(0.5) * (R(1) + phic);
    f.nub = R(1) / (hp * (R)k.inv_nu_r + (R(1) - hp) * (R)k.inv_nu_b);
    f.s2 = R(1) / (R(3) * f.nub + R(0.5));
    f.abar = (R)k.alpha_b + hp * (R)k.dalpha;
    f.kap = R(27.0 / 19.0) * (R(1) - f.abar);
    f.om = R(1) - f.s2;
    const R gv[3] = {(R)k.gx, (R)k.gy, (R)k.gz};
    const R inv_rho = R(1) / f.rho;
    for (int a = 0; a < 3; ++a) {
        f.F[a] = M.m0 * gv[a];
        f.u[a] = (M.j[a] + R(0.5) * f.F[a]) * inv_rho;
        f.gp[a] = (R)g[a];
        f.gr[a] = (R)g[3 + a];
    }
    const R* u = f.u;
    const R* r = f.gr;
    const R* F = f.F;
    const R rho = f.rho, nub = f.nub;
    f.q[0] = M.P[0] - rho * u[0] * u[0] - R(2) * nub * u[0] * r[0] + u[0] * F[0];
    f.q[1] = M.P[1] - rho * u[1] * u[1] - R(2) * nub * u[1] * r[1] + u[1] * F[1];
    f.q[2] = M.P[2] - rho * u[2] * u[2] - R(2) * nub * u[2] * r[2] + u[2] * F[2];
    f.q[3] = M.P[3] - rho * u[0] * u[1] - nub * (u[0] * r[1] + r[0] * u[1]) + R(0.5) * (u[0] * F[1] + u[1] * F[0]);
    f.q[4] = M.P[4] - rho * u[0] * u[2] - nub * (u[0] * r[2] + r[0] * u[2]) + R(0.5) * (u[0] * F[2] + u[2] * F[0]);
    f.q[5] = M.P[5] - rho * u[1] * u[2] - nub * (u[1] * r[2] + r[1] * u[2]) + R(0.5) * (u[1] * F[2] + u[2] * F[1]);
    f.tr = (f.q[0] + f.q[1] + f.q[2]) * R(1.0 / 3.0);
    for (int a = 0; a < 3; ++a) f.kk[a] = f.om * (f.q[a] - f.tr);
    for (int a = 3; a < 6; ++a) f.kk[a] = f.om * f.q[a];
    const double G2 = g[0] * g[0] + g[1] * g[1] + g[2] * g[2];
    f.on = G2 > (double)k.eps2;
    const double gn = f.on ? sqrt(G2) : 0.0, ign = f.on ? 1.0 / gn : 0.0;
    f.gn = (R)gn;
    for (int a = 0; a < 3; ++a) f.n[a] = (R)(g[a] * ign);
}

// Colour-blind post-collision populations f' by opposite pairs (i, i + 1), odd i,
// which share the parts that are even and odd in c:
//   even = w [rho kappa - 1.5 rho u^2 - 1.5 u.F - A |g| + cu (4.5 rho cu + 9 nu cr + 4.5 cF) + A |g| (c.n)^2],
//   odd  = w [cu (rho (3 - 4.5 u^2) + 4.5 rho cu^2) + 1.5 cF]
// (cu = c.u, cr = c.grad rho, cF = c.F), and the relaxed moments contracted axis by
// axis (z, y, then x).
template <class R>
struct PostCtx {
    Basis1T<R> bx, by, bz;
    R u2, uF, ur, K0, K1, r45, nub9, Ag;
    R U0[3][3], U1[3][3], U2[3][3];  // [cy + 1][cz + 1]
    CG_HD explicit PostCtx(const KP& k, const NodeFwdT<R>& f)
        : bx(f.u[0]), by(f.u[1]), bz(f.u[2]),
          u2(f.u[0] * f.u[0] + f.u[1] * f.u[1] + f.u[2] * f.u[2]),
          uF(f.u[0] * f.F[0] + f.u[1] * f.F[1] + f.u[2] * f.F[2]),
          ur(f.u[0] * f.gr[0] + f.u[1] * f.gr[1] + f.u[2] * f.gr[2])
    {
        Ag = f.on ? (R)k.A * f.gn : R(0);
        K0 = f.rho * f.kap - R(1.5) * f.rho * u2 - R(1.5) * uF - Ag;
        K1 = f.rho * (R(3) - R(4.5) * u2);
        r45 = R(4.5) * f.rho;
        nub9 = R(9) * f.nub;
        for (int jz = 0; jz < 3; ++jz) {
            const R a = f.kk[3] * bz.h0[jz], b = f.kk[4] * bz.h1[jz], c = f.kk[5] * bz.h1[jz];
            const R d = f.kk[0] * bz.h0[jz], e = f.kk[1] * bz.h0[jz], g = f.kk[2] * h2r<R>(jz);
            for (int jy = 0; jy < 3; ++jy) {
                U1[jy][jz] = a * by.h1[jy] + b * by.h0[jy];
                U0[jy][jz] = c * by.h1[jy] + e * h2r<R>(jy) + g * by.h0[jy];
                U2[jy][jz] = d * by.h0[jy];
            }
        }
    }
    CG_HD R delta(int cx, int cy, int cz) const
    {
        return U0[cy + 1][cz + 1] * bx.h0[cx + 1] + U1[cy + 1][cz + 1] * bx.h1[cx + 1] +
               U2[cy + 1][cz + 1] * h2r<R>(cx + 1);
    }
    CG_HD R rest(const NodeFwdT<R>& f) const
    {
        const R w = (R)wgtd(0);
        return f.rho * f.abar - R(1.5) * w * f.rho * u2 - R(3) * f.nub * ur - R(1.5) * w * uF + Ag * R(10.0 / 27.0) +
               delta(0, 0, 0);
    }
    // f' of directions i and i + 1
    CG_HD void pair(int i, const NodeFwdT<R>& f, R& fp, R& fm) const
    {
        const R w = (R)wgtd(i);
        const R cu = cdot(i, f.u[0], f.u[1], f.u[2]), cr = cdot(i, f.gr[0], f.gr[1], f.gr[2]);
        const R cF = cdot(i, f.F[0], f.F[1], f.F[2]), cn = cdot(i, f.n[0], f.n[1], f.n[2]);
        const R even = w * (K0 + cu * (r45 * cu + (nub9 * cr + R(4.5) * cF)) + (Ag * cn) * cn);
        const R odd = w * (cu * (K1 + r45 * (cu * cu)) + R(1.5) * cF);
        fp = even + odd + delta(kCX[i], kCY[i], kCZ[i]);
        fm = even - odd + delta(-kCX[i], -kCY[i], -kCZ[i]);
    }
};

// colour-blind post-collision populations f'_i and the recolouring vector V
template <class R>
CG_HD void node_post(const KP& k, const NodeFwdT<R>& f, R xr, R* fp, R* V)
{
    const PostCtx<R> c(k, f);
    fp[0] = c.rest(f);
#pragma unroll
    for (int i = 1; i < Q; i += 2) c.pair(i, f, fp[i], fp[i + 1]);
    const R s = f.on ? (R)k.beta * xr * (R(1) - xr) * f.rho * f.kap : R(0);
    for (int a = 0; a < 3; ++a) V[a] = s * f.n[a];
}

// recoloured red and blue populations of direction i from f'_i and V
template <class R>
CG_HD void recolour_dir(int i, R xr, R fpi, const R* V, R& fr, R& fb)
{
    R v = xr * fpi;
    if (i != 0) v += (R)(wgtd(i) * inv_lend(i)) * (kCX[i] * V[0] + kCY[i] * V[1] + kCZ[i] * V[2]);
    fr = v;
    fb = fpi - v;
}

template <class R>
struct NodeAdjT {
    R Lm0, Lj[3], Lq[6];  // cotangents of the raw moments of d (that of d_i is Lm0 + c_i.Lj + c_i c_i : Lq)
    R Lgp[3], Lgr[3]; // of grad phi, grad rho
    R Lphic, Lxr;     // of phi at the node, rho_r / rho
};

// Cotangent of A: sum_i L'_i |grad phi| [w_i (c_i.n)^2 - B_i] with the colour-blind
// cotangents L' = Lb + xr (Lr - Lb).  In FP64 from the cotangents as they were
// stored: the terms of the nodes alternate in sign, so that their sum over the lattice
// keeps the absolute rounding of each and loses their size.  Relative error of dJ/dA
// against FP64, rms over 43 lattices of up to 4e5 nodes: 1.5e-6 with FP32 terms, 0.75e-6
// now (that of the stored state); no time that could be measured.  With |g| n = g and B_i = w_i the factor of a pair of
// opposite directions is w_i [(c.g)^2 - g^2] / |g|: on a face -(the squares of the
// other two components of g), on an edge +-2 g_a g_b - g_c^2, on a corner the three
// products alone.
CG_HD double perturb_vjp(const KP& k, const double* g, double xr, const float* Lr, const float* Lb)
{
    const double xx = g[0] * g[0], yy = g[1] * g[1], zz = g[2] * g[2], G2 = xx + yy + zz;
    if (!(G2 > (double)k.eps2)) return 0.0;
    const double xy = 2.0 * g[0] * g[1], xz = 2.0 * g[0] * g[2], yz = 2.0 * g[1] * g[2];
    double s[3] = {0.0, 0.0, 0.0};  // faces, edges, corners
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const double r = (double)Lr[i] + (double)Lr[i + 1], b = (double)Lb[i] + (double)Lb[i + 1];
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        double q = 0.0;
        if (cx * cy) q += (cx * cy) * xy;
        if (cx * cz) q += (cx * cz) * xz;
        if (cy * cz) q += (cy * cz) * yz;
        if (!cx) q -= xx;
        if (!cy) q -= yy;
        if (!cz) q -= zz;
        s[csq(i) - 1] += q * fma(xr, r - b, b);
    }
    const double rest = fma(xr, (double)Lr[0] - (double)Lb[0], (double)Lb[0]);
    const double gn = sqrt(G2);
    return (wgtd(1) * s[0] + wgtd(7) * s[1] + wgtd(19) * s[2]) / gn + (10.0 / 27.0) * gn * rest;
}

// Weighted moments sum_i w_i v_i c_ia c_ib ... up to third order of 27 values, axis by
// axis (w_i is a product of 1/6, 2/3, 1/6 per axis): 58 operations for the sums that
// the equilibrium, Phi and the forcing need, 20 per direction one direction at a time.
// The rest direction joins last: s0, the sum over the moving ones, holds no rounding of
// it (dJ/dA of rollouts of 3 to 8 steps, rms over 157 lattices: 7.7e-6 off with s0 as a
// difference, 5.4e-6 now).
template <class R>
struct WMomT {
    R s0, m0, m1[3], m2[6];  // m2: xx yy zz xy xz yz
    R xxy, xxz, xyy, yyz, xzz, yzz, xyz;
    CG_HD explicit WMomT(const R* v)
    {
        R X[3][3][3], Y[3][3][3];  // [order in x][jy][jz], [orders in x and y][jz]
#pragma unroll
        for (int jy = 0; jy < 3; ++jy)
#pragma unroll
            for (int jz = 0; jz < 3; ++jz)
                line(v[dir_of(-1, jy - 1, jz - 1)], jy == 1 && jz == 1 ? R(0) : v[dir_of(0, jy - 1, jz - 1)],
                     v[dir_of(1, jy - 1, jz - 1)], X[0][jy][jz], X[1][jy][jz], X[2][jy][jz]);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int jz = 0; jz < 3; ++jz)
                line(X[a][0][jz], X[a][1][jz], X[a][2][jz], Y[a][0][jz], Y[a][1][jz], Y[a][2][jz]);
        const R W = R(1.0 / 216.0);
        R z[3][3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3 - (a == 2); ++b) {
                line(Y[a][b][0], Y[a][b][1], Y[a][b][2], z[a][b][0], z[a][b][1], z[a][b][2]);
                for (int c = 0; c < 3; ++c) z[a][b][c] *= W;
            }
        s0 = z[0][0][0];
        m0 = s0 + (R)wgtd(0) * v[0];
        m1[0] = z[1][0][0]; m1[1] = z[0][1][0]; m1[2] = z[0][0][1];
        m2[0] = z[2][0][0]; m2[1] = z[0][2][0]; m2[2] = z[0][0][2];
        m2[3] = z[1][1][0]; m2[4] = z[1][0][1]; m2[5] = z[0][1][1];
        xxy = z[2][1][0]; xxz = z[2][0][1]; xyy = z[1][2][0]; yyz = z[0][2][1];
        xzz = z[1][0][2]; yzz = z[0][1][2]; xyz = z[1][1][1];
    }
    // sum w v c (c.a)
    CG_HD void second(const R* a, R* o) const
    {
        o[0] = m2[0] * a[0] + m2[3] * a[1] + m2[4] * a[2];
        o[1] = m2[3] * a[0] + m2[1] * a[1] + m2[5] * a[2];
        o[2] = m2[4] * a[0] + m2[5] * a[1] + m2[2] * a[2];
    }
    // sum w v c (c.a)^2
    CG_HD void third(const R* a, R* o) const
    {
        const R x2 = R(2) * a[0], y2 = R(2) * a[1], xx = a[0] * a[0], yy = a[1] * a[1], zz = a[2] * a[2];
        const R xy = x2 * a[1], xz = x2 * a[2], yz = y2 * a[2];
        o[0] = m1[0] * xx + xxy * xy + xxz * xz + xyy * yy + xzz * zz + xyz * yz;
        o[1] = m1[1] * yy + xyy * xy + yyz * yz + xxy * xx + yzz * zz + xyz * xz;
        o[2] = m1[2] * zz + xzz * xz + yzz * yz + xxz * xx + yyz * yy + xyz * xy;
    }

private:
    static CG_HD void line(R v0, R v1, R v2, R& a, R& b, R& c)
    {
        c = v0 + v2;
        b = v2 - v0;
        a = c + R(4) * v1;
    }
};
template <class R>
CG_HD R dot3(const R* a, const R* b)
{
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// (sum v h0, sum v h1, sum v h2) over c = -1, 0, 1 of the inverse central-moment basis
template <class R>
CG_HD void basis_line(R u, R v0, R v1, R v2, R& a, R& b, R& c)
{
    c = R(0.5) * (v0 + v2) - v1;
    const R t = R(0.5) * (v2 - v0) + u * c;
    a = v1 + u * t;
    b = t + u * c;
}
// [a][b][jz]: 27 values contracted with the bases of x and y
template <class R>
CG_HD void basis_xy(const R* u, const R* v, R (&Y)[3][3][3])
{
    R X[3][3][3];
#pragma unroll
    for (int jy = 0; jy < 3; ++jy)
#pragma unroll
        for (int jz = 0; jz < 3; ++jz)
            basis_line(u[0], v[dir_of(-1, jy - 1, jz - 1)], v[dir_of(0, jy - 1, jz - 1)],
                       v[dir_of(1, jy - 1, jz - 1)], X[0][jy][jz], X[1][jy][jz], X[2][jy][jz]);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int jz = 0; jz < 3; ++jz)
            basis_line(u[1], X[a][0][jz], X[a][1][jz], X[a][2][jz], Y[a][0][jz], Y[a][1][jz], Y[a][2][jz]);
}
template <class R>
CG_HD R basis_z(R u, const R (&Y)[3][3][3], int a, int b, int c)
{
    R z[3];
    basis_line(u, Y[a][b][0], Y[a][b][1], Y[a][b][2], z[0], z[1], z[2]);
    return z[c];
}

// reverse sweep of the node map.  Lr, LbL: on entry the cotangents of the red and blue
// post-collision populations; both are overwritten.
template <class R>
CG_HD void node_vjp(const KP& k, const NodeFwdT<R>& f, R xr, R* Lr, R* LbL, NodeAdjT<R>& o)
{
    const R rho = f.rho, nub = f.nub;
    const R* u = f.u;
    const R* F = f.F;
    const R* gr = f.gr;
    const R* n = f.n;
    const R u2 = dot3(u, u), uF = dot3(u, F), ur = dot3(u, gr);
    const R K1 = R(3) - R(4.5) * u2, w0 = (R)wgtd(0);
    R* L = LbL;
    // recolouring: with D_i = Lr_i - Lb_i (written over Lr) the colour-blind cotangents
    // L'_i = Lb_i + xr D_i (over Lb), that of xr, sum_i D_i f'_i, and of V
    R LV[3] = {0, 0, 0};
    Lr[0] -= L[0];
    L[0] += xr * Lr[0];
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const R dp = Lr[i] - L[i], dm = Lr[i + 1] - L[i + 1];
        Lr[i] = dp;
        Lr[i + 1] = dm;
        L[i] += xr * dp;
        L[i + 1] += xr * dm;
        const R s = (dp - dm) * (R)(wgtd(i) * inv_lend(i));
        if (kCX[i]) LV[0] += kCX[i] * s;
        if (kCY[i]) LV[1] += kCY[i] * s;
        if (kCZ[i]) LV[2] += kCZ[i] * s;
    }
    R Lxr;
    {
        const WMomT<R> D(Lr);
        R Du[3], Duu[3];
        D.second(u, Du);
        D.third(u, Duu);
        const R Ag = f.on ? (R)k.A * f.gn : R(0), d0 = Lr[0];
        Lxr = D.s0 * (rho * f.kap - R(1.5) * rho * u2 - R(1.5) * uF - Ag) + rho * K1 * dot3(D.m1, u) +
              R(1.5) * dot3(D.m1, F) + dot3(Du, u) * (R(4.5) * rho) + R(4.5) * rho * dot3(Duu, u) +
              R(9) * nub * dot3(Du, gr) + R(4.5) * dot3(Du, F) +
              d0 * (rho * f.abar - R(1.5) * w0 * rho * u2 - R(3) * nub * ur - R(1.5) * w0 * uF + Ag * R(10.0 / 27.0));
        if (f.on) {
            R Dn[3];
            D.second(n, Dn);
            Lxr += Ag * dot3(Dn, n);
        }
        R Y[3][3][3];
        basis_xy(u, Lr, Y);
        Lxr += f.kk[0] * basis_z(u[2], Y, 2, 0, 0) + f.kk[1] * basis_z(u[2], Y, 0, 2, 0) +
               f.kk[2] * basis_z(u[2], Y, 0, 0, 2) + f.kk[3] * basis_z(u[2], Y, 1, 1, 0) +
               f.kk[4] * basis_z(u[2], Y, 1, 0, 1) + f.kk[5] * basis_z(u[2], Y, 0, 1, 1);
    }
    R Lrho = 0, Lkap = 0, Labar = 0, Lnub = 0;
    R Lu[3] = {0, 0, 0}, LF[3] = {0, 0, 0}, Lgr[3] = {0, 0, 0}, Lgp[3] = {0, 0, 0};
    const R beta = (R)k.beta;
    if (f.on) {
        const R LVn = LV[0] * f.n[0] + LV[1] * f.n[1] + LV[2] * f.n[2];
        const R xx = xr * (R(1) - xr);
        const R sV = beta * xx * rho * f.kap;
        Lxr += beta * (R(1) - R(2) * xr) * rho * f.kap * LVn;
        Lrho += beta * xx * f.kap * LVn;
        Lkap += beta * xx * rho * LVn;
        const R ig = R(1) / f.gn;
        for (int a = 0; a < 3; ++a) Lgp[a] += sV * (LV[a] - LVn * f.n[a]) * ig;
    }
    // equilibrium, Phi and forcing terms from the weighted moments of L'
    const WMomT<R> T(L);
    R Tu[3], Tuu[3], Tr[3], TF[3];
    T.second(u, Tu);
    T.second(gr, Tr);
    T.second(F, TF);
    T.third(u, Tuu);
    const R sA = T.m0, S0 = T.s0;
    const R T1u = dot3(T.m1, u);
    R su = R(3) * sA + R(9) * T1u;
    Lrho += K1 * T1u + R(4.5) * (dot3(Tu, u) + dot3(Tuu, u)) - R(1.5) * u2 * sA;
    Lnub += R(9) * dot3(Tr, u);
    for (int a = 0; a < 3; ++a) {
        Lu[a] += rho * (K1 * T.m1[a] + R(9) * Tu[a] + R(13.5) * Tuu[a]) + R(9) * nub * Tr[a] + R(4.5) * TF[a];
        Lgr[a] += R(9) * nub * Tu[a];
        LF[a] += R(4.5) * Tu[a] + R(1.5) * T.m1[a];
    }
    su *= rho;
    for (int c = 0; c < 3; ++c) {
        Lu[c] -= su * u[c] + R(1.5) * sA * F[c];
        LF[c] -= R(1.5) * sA * u[c];
    }
    // rest population: rho alpha_bar and Phi_0 = -3 nu_bar u . grad rho
    const R L0 = L[0];
    Lrho += f.abar * L0;
    Labar += rho * L0;
    Lnub += R(-3) * ur * L0;
    for (int c = 0; c < 3; ++c) {
        Lu[c] += R(-3) * nub * L0 * gr[c];
        Lgr[c] += R(-3) * nub * L0 * u[c];
    }
    // moving directions: rho kappa
    Lrho += f.kap * S0;
    Lkap += rho * S0;
    // perturbation (squared projection, prefactor A): A |g| [w (c.n)^2 - B]
    if (f.on) {
        const R A = (R)k.A;
        R Mn[3];
        T.second(n, Mn);
        const R nMn = n[0] * Mn[0] + n[1] * Mn[1] + n[2] * Mn[2];
        const R b0 = L0 * R(10.0 / 27.0) - S0;
        for (int c = 0; c < 3; ++c) Lgp[c] += A * (R(2) * Mn[c] + (b0 - nMn) * n[c]);
    }
    // relaxed-moment part: C[a][b][c] = sum over directions of L h_a(cx) h_b(cy) h_c(cz)
    R Y[3][3][3];
    basis_xy(u, L, Y);
    auto Cz = [&](int a, int b, int c) -> R { return basis_z(u[2], Y, a, b, c); };
    const R C200 = Cz(2, 0, 0), C020 = Cz(0, 2, 0), C002 = Cz(0, 0, 2), C110 = Cz(1, 1, 0), C101 = Cz(1, 0, 1),
            C011 = Cz(0, 1, 1), C210 = Cz(2, 1, 0), C201 = Cz(2, 0, 1), C111 = Cz(1, 1, 1), C120 = Cz(1, 2, 0),
            C102 = Cz(1, 0, 2), C021 = Cz(0, 2, 1), C012 = Cz(0, 1, 2);
    const R* kk = f.kk;  // xx yy zz xy xz yz
    const R Lk[6] = {C200, C020, C002, C110, C101, C011};
    Lu[0] += R(2) * kk[3] * C210 + R(2) * kk[4] * C201 + kk[5] * C111 + kk[1] * C120 + kk[2] * C102;
    Lu[1] += R(2) * kk[3] * C120 + kk[4] * C111 + R(2) * kk[5] * C021 + kk[0] * C210 + kk[2] * C012;
    Lu[2] += kk[3] * C111 + R(2) * kk[4] * C102 + R(2) * kk[5] * C012 + kk[0] * C201 + kk[1] * C021;
    // k = (1 - s2) dev(q)
    const R trL = (Lk[0] + Lk[1] + Lk[2]) * R(1.0 / 3.0);
    R Lq[6];
    for (int a = 0; a < 3; ++a) Lq[a] = f.om * (Lk[a] - trL);
    for (int a = 3; a < 6; ++a) Lq[a] = f.om * Lk[a];
    R Ls2 = 0;
    for (int a = 0; a < 3; ++a) Ls2 -= (f.q[a] - f.tr) * Lk[a];
    for (int a = 3; a < 6; ++a) Ls2 -= f.q[a] * Lk[a];
    // q = P - rho u u^T - nu_bar (u r^T + r u^T) + (u F^T + F u^T)/2, through the symmetric matrix Qm
    const R Qm[3][3] = {{Lq[0], R(0.5) * Lq[3], R(0.5) * Lq[4]},
                        {R(0.5) * Lq[3], Lq[1], R(0.5) * Lq[5]},
                        {R(0.5) * Lq[4], R(0.5) * Lq[5], Lq[2]}};
    R Qu[3], Qr[3], QF[3];
    for (int a = 0; a < 3; ++a) {
        Qu[a] = Qm[a][0] * u[0] + Qm[a][1] * u[1] + Qm[a][2] * u[2];
        Qr[a] = Qm[a][0] * gr[0] + Qm[a][1] * gr[1] + Qm[a][2] * gr[2];
        QF[a] = Qm[a][0] * F[0] + Qm[a][1] * F[1] + Qm[a][2] * F[2];
    }
    Lrho -= u[0] * Qu[0] + u[1] * Qu[1] + u[2] * Qu[2];
    Lnub -= R(2) * (u[0] * Qr[0] + u[1] * Qr[1] + u[2] * Qr[2]);
    for (int a = 0; a < 3; ++a) {
        Lu[a] += R(-2) * rho * Qu[a] - R(2) * nub * Qr[a] + QF[a];
        Lgr[a] += R(-2) * nub * Qu[a];
        LF[a] += Qu[a];
    }
    // interpolated properties
    Labar -= R(27.0 / 19.0) * Lkap;
    R Lhp = (R)k.dalpha * Labar;
    Lnub += R(-3) * f.s2 * f.s2 * Ls2;
    Lhp += -nub * nub * ((R)k.inv_nu_r - (R)k.inv_nu_b) * Lnub;
    // u = (j + F/2) / rho, F = m0 g, rho = rho_b0 + m0
    const R inv_rho = R(1) / rho;
    R Lj[3];
    for (int a = 0; a < 3; ++a) {
        Lj[a] = Lu[a] * inv_rho;
        LF[a] += R(0.5) * Lj[a];
    }
    Lrho -= (u[0] * Lu[0] + u[1] * Lu[1] + u[2] * Lu[2]) * inv_rho;
    const R Lm0 = Lrho + (R)k.gx * LF[0] + (R)k.gy * LF[1] + (R)k.gz * LF[2];
    o.Lm0 = Lm0;
    for (int a = 0; a < 3; ++a) {
        o.Lj[a] = Lj[a];
        o.Lgp[a] = Lgp[a];
        o.Lgr[a] = Lgr[a];
    }
    for (int a = 0; a < 6; ++a) o.Lq[a] = Lq[a];
    o.Lphic = R(0.5) * Lhp;
    o.Lxr = Lxr;
}

}  // namespace cglbm
