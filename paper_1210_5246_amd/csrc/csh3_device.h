// Device arithmetic of the three-dimensional moment equations: the
// ten-moment system (rho, rho u_i, E_ij = P_ij + rho u_i u_j) with zero heat
// flux (Sec. 2, eqs. (2)-(4) in three dimensions; ten eigenvalues, Sec. 3.3),
// characteristic MUSCL-Hancock with HLL fluxes as in two dimensions.
//
// States are 10-vectors in registers: primitive (rho, u, v, w, Pxx, Pxy, Pxz,
// Pyy, Pyz, Pzz), conserved (rho, rho u, rho v, rho w, Exx, ..., Ezz).  Each
// direction N (0, 1, 2) is a template argument, so every index below is a
// compile-time constant and the vectors stay in registers.  Along axis n with
// transverse axes t1 < t2 the eigen-system is (eigenvalues ascending)
//   u - a, u - c (t1), u - c (t2), u (rho, P_t1t1, P_t1t2, P_t2t2),
//   u + c (t1), u + c (t2), u + a,    a = sqrt(3 P_nn / rho), c = sqrt(P_nn / rho),
// projected and back-projected in closed form (q_t = P_nt / P_nn); the
// tracing uses the collapsed form of eqs. (27)-(32) with the HLL terms, which
// needs only the extreme speeds u -+ a.  As in two dimensions the kernels carry
// half slopes (the face-state coefficients take the factor 2) and form each
// wave's amplitude up to a positive per-cell scale.
#pragma once

#include "csh_device.h"

namespace csh {
namespace d3 {

constexpr int NV = 10;

struct V10 {
    double v[NV];
};

// index of P_ij / E_ij
CSH_HD constexpr int P(int i, int j)
{
    return (i == 0) ? 4 + j : (i == 1) ? (j == 0 ? 5 : 6 + j) : (j == 0 ? 6 : j == 1 ? 8 : 9);
}

template <int N>
struct Axes {
    static constexpr int t1 = (N == 0) ? 1 : 0;
    static constexpr int t2 = (N == 2) ? 1 : 2;
};

CSH_HD V10 to_prim(const V10& U, double ir)
{
    V10 w;
    w.v[0] = U.v[0];
#pragma unroll
    for (int i = 0; i < 3; ++i) w.v[1 + i] = U.v[1 + i] * ir;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) w.v[P(i, j)] = U.v[P(i, j)] - U.v[1 + i] * w.v[1 + j];
    return w;
}

CSH_HD V10 to_cons(const V10& w)
{
    V10 U;
    U.v[0] = w.v[0];
#pragma unroll
    for (int i = 0; i < 3; ++i) U.v[1 + i] = w.v[0] * w.v[1 + i];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) U.v[P(i, j)] = w.v[P(i, j)] + U.v[1 + i] * w.v[1 + j];
    return U;
}

// base - k A d with A the primitive Jacobian along N:
//   A d = (u_n d_rho + rho d_un, u_n d_ui + d_Pin / rho,
//          u_n d_Pij + P_ij d_un + P_in d_uj + P_jn d_ui),
// summed before it leaves the base, which is so rounded once (as in two dimensions).
template <int N>
CSH_HD V10 sub_jac(const V10& base, double k, const V10& w, double ir, const V10& d)
{
    constexpr int t1 = Axes<N>::t1, t2 = Axes<N>::t2;
    constexpr int nn = P(N, N), n1 = P(N, t1), n2 = P(N, t2), s11 = P(t1, t1), s12 = P(t1, t2), s22 = P(t2, t2);
    const double un = w.v[1 + N], dn = d.v[1 + N], d1 = d.v[1 + t1], d2 = d.v[1 + t2];
    const double p1 = 2.0 * w.v[n1], p2 = 2.0 * w.v[n2], p3 = 3.0 * w.v[nn];
    V10 o;
    o.v[0] = base.v[0] - k * (un * d.v[0] + w.v[0] * dn);
    o.v[1 + N] = base.v[1 + N] - k * (un * dn + ir * d.v[nn]);
    o.v[1 + t1] = base.v[1 + t1] - k * (un * d1 + ir * d.v[n1]);
    o.v[1 + t2] = base.v[1 + t2] - k * (un * d2 + ir * d.v[n2]);
    o.v[nn] = base.v[nn] - k * (un * d.v[nn] + p3 * dn);
    o.v[n1] = base.v[n1] - k * (un * d.v[n1] + p1 * dn + w.v[nn] * d1);
    o.v[n2] = base.v[n2] - k * (un * d.v[n2] + p2 * dn + w.v[nn] * d2);
    o.v[s11] = base.v[s11] - k * (un * d.v[s11] + w.v[s11] * dn + p1 * d1);
    o.v[s12] = base.v[s12] - k * (un * d.v[s12] + w.v[s12] * dn + w.v[n1] * d2 + w.v[n2] * d1);
    o.v[s22] = base.v[s22] - k * (un * d.v[s22] + w.v[s22] * dn + p2 * d2);
    return o;
}

template <int N>
struct Eig {
    double a, ic, ip, q1, q2;  // a = sqrt(3 Pnn / rho), ic = sqrt(rho / Pnn) = 1/c, ip = 1/Pnn
};

template <int N>
CSH_HD Eig<N> eig(const V10& w, double ir)
{
    constexpr int t1 = Axes<N>::t1, t2 = Axes<N>::t2;
    Eig<N> e;
    const double pnn = w.v[P(N, N)];
    const double t = pnn * ir;
    const double y = rsqrt(t);  // 1 / c
    e.a = 1.7320508075688772935 * (t * y);
    e.ic = y;
    e.ip = y * y * ir;          // (rho / Pnn) / rho
    e.q1 = w.v[P(N, t1)] * e.ip;
    e.q2 = w.v[P(N, t2)] * e.ip;
    return e;
}

// Half the MC limiter, mc(dl, dr) / 2, from order statistics: with
// q = (dl + dr) / 4 the result is the median of (min(dl, dr, q), 0,
// max(dl, dr, q)).
CSH_HD double mc_half(double dl, double dr)
{
    const double q = 0.25 * (dl + dr);
    const double A = fmin(fmin(dl, dr), q), B = fmax(fmax(dl, dr), q);
    return fmax(A, fmin(B, 0.0));
}

// Half the characteristic MC-limited slope along N (eqs. (19)-(26)).  The
// limiter commutes with a positive factor common to its two arguments, so the
// amplitudes are formed up to per-cell positive scales:
//   u -+ a:          dPnn -+ rho a du_n                          (6 Pnn times l . d)
//   u -+ c (t):      (dPnt - q_t dPnn) -+ rho c (q_t du_n - du_t)  (2 Pnn times)
//   u (4 waves):     drho - rho dPnn / (3 Pnn) and the three transverse-stress
//                    combinations, unscaled;
// the back-projection divides the scales out.  The coefficients come from 1/c
// and 1/Pnn as in two dimensions: rho c = Pnn / c, c / Pnn = 1 / (rho c), and
// with h = S / 2 the S terms of the density and the transverse stresses are
// kr h and (P_tt' / Pnn + 2 q_t q_t') h / 3.
template <int N>
CSH_HD V10 half_slope(const V10& w, double ir, const Eig<N>& e, const V10& wm, const V10& wp)
{
    constexpr int t1 = Axes<N>::t1, t2 = Axes<N>::t2;
    constexpr int nn = P(N, N), n1 = P(N, t1), n2 = P(N, t2), s11 = P(t1, t1), s12 = P(t1, t2), s22 = P(t2, t2);
    const double rc = w.v[nn] * e.ic, ra = 1.7320508075688772935 * rc;
    const double ip3 = e.ip * (1.0 / 3.0), kr = w.v[0] * ip3;
    const double g11 = w.v[s11] * ip3, g12 = w.v[s12] * ip3, g22 = w.v[s22] * ip3;
    const double r1 = w.v[n1] * ip3, r2 = w.v[n2] * ip3;
    const double qq11 = e.q1 * r1, qq12 = e.q1 * r2, qq22 = e.q2 * r2;
    const double k11 = 4.0 * qq11 - g11, k12 = 4.0 * qq12 - g12, k22 = 4.0 * qq22 - g22;
    const double q1x2 = e.q1 + e.q1, q2x2 = e.q2 + e.q2;
    auto project = [&](const V10& d, double (&al)[NV]) {
        const double dnn = d.v[nn], dun = d.v[1 + N];
        al[0] = dnn - ra * dun;
        al[9] = dnn + ra * dun;
        const double s1 = d.v[n1] - e.q1 * dnn, h1 = e.q1 * dun - d.v[1 + t1];
        const double s2 = d.v[n2] - e.q2 * dnn, h2 = e.q2 * dun - d.v[1 + t2];
        al[1] = s1 + rc * h1;
        al[7] = s1 - rc * h1;
        al[2] = s2 + rc * h2;
        al[8] = s2 - rc * h2;
        al[3] = d.v[0] - kr * dnn;
        al[4] = d.v[s11] - q1x2 * d.v[n1] + k11 * dnn;
        al[5] = d.v[s12] - e.q2 * d.v[n1] - e.q1 * d.v[n2] + k12 * dnn;
        al[6] = d.v[s22] - q2x2 * d.v[n2] + k22 * dnn;
    };
    double l[NV], r[NV], m[NV];
    {
        V10 dl, dr;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            dl.v[k] = w.v[k] - wm.v[k];
            dr.v[k] = wp.v[k] - w.v[k];
        }
        project(dl, l);
        project(dr, r);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) m[k] = mc_half(l[k], r[k]);
    const double S = m[0] + m[9], D = m[9] - m[0];
    const double S1 = m[1] + m[7], D1 = m[7] - m[1];
    const double S2 = m[2] + m[8], D2 = m[8] - m[2];
    const double z = e.ic * ir, bu = 0.28867513459481288225 * z, bc = 0.5 * z;  // a / (6 Pnn), c / (2 Pnn)
    const double h = 0.5 * S, h1 = 0.5 * S1, h2 = 0.5 * S2;
    V10 d;
    d.v[0] = kr * h + m[3];
    d.v[1 + N] = bu * D;
    d.v[1 + t1] = e.q1 * d.v[1 + N] + bc * D1;
    d.v[1 + t2] = e.q2 * d.v[1 + N] + bc * D2;
    d.v[nn] = h;
    d.v[n1] = e.q1 * h + h1;
    d.v[n2] = e.q2 * h + h2;
    d.v[s11] = (2.0 * qq11 + g11) * h + (q1x2 * h1 + m[4]);
    d.v[s12] = (2.0 * qq12 + g12) * h + (e.q2 * h1 + (e.q1 * h2 + m[5]));
    d.v[s22] = (2.0 * qq22 + g22) * h + (q2x2 * h2 + m[6]);
    return d;
}

// One side of the HLL flux along N: w (F - s U), formed from the primitive state:
// with s' = u_n - s and m = rho s', F - s U is X_rho = m, X_i = m u_i + P_in,
// X_ij = u_j X_i + s' P_ij + P_nj u_i (for i = n: u_j X_n + P_nj (s' + u_n)), linear
// in (s', P_in) at fixed velocities, so the weight scales those alone.  The
// stresses accumulate onto `add` (the other side, of opposite weight).
template <int N, bool ADD>
CSH_HD V10 weighted_flux(const V10& w, double s, double weight, const V10& add)
{
    const double un = w.v[1 + N], sp = un - s, g = sp + un, ws = weight * sp, m = w.v[0] * ws;
    double pn[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) pn[i] = weight * w.v[P(i, N)];
    V10 X;
    X.v[0] = ADD ? add.v[0] + m : m;
    double xi[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        xi[i] = m * w.v[1 + i] + pn[i];
        X.v[1 + i] = ADD ? add.v[1 + i] + xi[i] : xi[i];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) {
            const double a = ADD ? add.v[P(i, j)] : 0.0;
            if (i == N) X.v[P(i, j)] = ADD ? a + w.v[1 + j] * xi[N] + pn[j] * g : w.v[1 + j] * xi[N] + pn[j] * g;
            else if (j == N) X.v[P(i, j)] = ADD ? a + w.v[1 + i] * xi[N] + pn[i] * g : w.v[1 + i] * xi[N] + pn[i] * g;
            else
                X.v[P(i, j)] = ADD ? a + w.v[1 + j] * xi[i] + ws * w.v[P(i, j)] + pn[j] * w.v[1 + i]
                                   : w.v[1 + j] * xi[i] + ws * w.v[P(i, j)] + pn[j] * w.v[1 + i];
        }
    return X;
}

// HLL flux along N between face states (Davis speeds); with the clamped
// outer speeds S_L' = min(S_L, 0), S_R' = max(S_R, 0) it is
// (S_R' X_L - S_L' X_R) / (S_R' - S_L'), X_K = F_K - S_K' U_K.
template <int N>
CSH_HD V10 hll(const V10& wl, const V10& wr)
{
    constexpr double s3 = 1.7320508075688772935;
    const double pl = wl.v[P(N, N)], pr = wr.v[P(N, N)];
    const double cl = pl * rsqrt(pl * wl.v[0]), cr = pr * rsqrt(pr * wr.v[0]);
    const double sl = fmin(fmin(wl.v[1 + N] - s3 * cl, wr.v[1 + N] - s3 * cr), 0.0);
    const double sr = fmax(fmax(wl.v[1 + N] + s3 * cl, wr.v[1 + N] + s3 * cr), 0.0);
    const double inv = rcp(sr - sl);
    return weighted_flux<N, true>(wr, sr, -sl * inv, weighted_flux<N, false>(wl, sl, sr * inv, V10{}));
}

// CFL rate: sum over the axes of (|u_k| + sqrt(3 P_kk / rho)) / h_k
CSH_HD double signal_rate(const V10& w, const double ih[3])
{
    const double ir3 = 3.0 * rcp(w.v[0]);
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) s = s + fabs(w.v[1 + k]) * ih[k] + sqrt_pos(w.v[P(k, k)] * ir3) * ih[k];
    return s;
}

// CFL rate of a new state together with the test of physical(): a finite rate
// means finite velocities and P_kk >= 0 with rho > 0 (each under a square root,
// NaN at <= 0); an infinite or NaN P_ij, i != j, fails one of the minors.
CSH_HD double checked_rate(const V10& w, const double ih[3], bool& bad)
{
    const double pxx = w.v[4], pxy = w.v[5], pxz = w.v[6], pyy = w.v[7], pyz = w.v[8], pzz = w.v[9];
    const double m2 = pxx * pyy - pxy * pxy;
    const double det = pxx * (pyy * pzz - pyz * pyz) - pxy * (pxy * pzz - pyz * pxz) + pxz * (pxy * pyz - pyy * pxz);
    const double s = signal_rate(w, ih);
    bad |= !((w.v[0] > 0.0) & (m2 > 0.0) & (det > 0.0) & __builtin_isfinite(s + w.v[0]));
    return s;
}

CSH_HD bool physical(const V10& w)
{
    const double pxx = w.v[4], pxy = w.v[5], pxz = w.v[6], pyy = w.v[7], pyz = w.v[8], pzz = w.v[9];
    const double m2 = pxx * pyy - pxy * pxy;
    const double det = pxx * (pyy * pzz - pyz * pyz) - pxy * (pxy * pzz - pyz * pxz) + pxz * (pxy * pyz - pyy * pxz);
    double sum = 0.0;
#pragma unroll
    for (int m = 0; m < NV; ++m) sum += w.v[m];
    return (w.v[0] > 0.0) & (pxx > 0.0) & (m2 > 0.0) & (det > 0.0) & __builtin_isfinite(sum);
}

}  // namespace d3
}  // namespace csh
