// Reverse-mode pieces of the sweep (FP64): vector-Jacobian products of every
// stage of csh_device.h, written out by hand statement by statement in reverse
// order, and the per-cell bodies of the adjoint kernels.
//
// Conventions: a function foo_vjp(inputs..., ybar, xbar...) ADDS the
// contribution of ybar to the adjoints xbar of foo's inputs.  At the kinks of
// min/max/|.| the subgradient of one branch is taken: MC takes the centred
// difference first, then 2|dl|, then 2|dr| (first minimal argument); the
// tracing coefficients have zero slope where their eigenvalue is exactly 0;
// HLL speed estimates take the first argument on ties and zero slope where
// they are clipped at 0.  All __host__ __device__, so the tests can run them
// on the CPU.
#pragma once

#include "csh_device.h"
#include "csh_xcd.h"

namespace csh {

using P = Prim<double>;
using C = Cons<double>;

CSH_HD void acc(P& a, const P& b)
{
    a.r += b.r; a.u += b.u; a.v += b.v; a.pxx += b.pxx; a.pxy += b.pxy; a.pyy += b.pyy;
}
CSH_HD P scale(double s, const P& a) { return {s * a.r, s * a.u, s * a.v, s * a.pxx, s * a.pxy, s * a.pyy}; }
CSH_HD double dot(const P& a, const P& b)
{
    return a.r * b.r + a.u * b.u + a.v * b.v + a.pxx * b.pxx + a.pxy * b.pxy + a.pyy * b.pyy;
}
CSH_HD P zero_p() { return {0, 0, 0, 0, 0, 0}; }
CSH_HD C zero_c() { return {0, 0, 0, 0, 0, 0}; }

// The limiter m = mc_half(dl, dr) with the weights of its two arguments in the
// branch it takes: 1/4 and 1/4 centred, 1 and 0 or 0 and 1 one-sided, 0 and 0
// off.  m is one of (dl + dr) / 4, dl, dr and 0 itself, so comparing it tells the
// branch (the centred one first); written without branches, so the adjoints stay
// in registers.
struct McVjp {
    double m, wl, wr;
};
CSH_HD McVjp mc_half_vjp(double dl, double dr)
{
    const double q = 0.25 * (dl + dr);
    const double A = fmin(fmin(dl, dr), q), B = fmax(fmax(dl, dr), q);
    const double m = fmax(A, fmin(B, 0.0));
    const bool on = m != 0.0, cen = on & (m == q), left = on & !cen & (m == dl), right = on & !cen & !left;
    return {m, cen ? 0.25 : (left ? 1.0 : 0.0), cen ? 0.25 : (right ? 1.0 : 0.0)};
}

CSH_HD P swapb(const P& a) { return swap(a); }  // the adjoint of a permutation that is its own inverse

// face_states<TWOD>(W0, Wl, Wr, Wm, Wp, kx, ky): adjoints of the five input states
// The reverse pass of face_states in two parts that add up to it: the y part
// (the y slope, its tracing coefficients and transverse term; adjoints of Wm,
// Wp and its share of W0) and the x part (the rest: the x slope, its
// coefficients and term, and the identity part of base; Wl, Wr and the rest of
// W0).  Both need the summed face adjoints of base; each adds its own 1/rho
// term.  W0b accumulates y first, then x.
CSH_HD P base_adjoint(const Faces<double>& fb, bool twod)
{
    P baseb = zero_p();
    // xhi = base + chix dxm ; xlo = base - clox dxm ; the same for y
    acc(baseb, fb.xhi);
    acc(baseb, fb.xlo);
    if (twod) {
        acc(baseb, fb.yhi);
        acc(baseb, fb.ylo);
    }
    return baseb;
}

// The reverse pass of one direction of face_states (normal direction x): from
// the adjoints of the high and low face states (fhi, flo) and of their common
// centre (baseb), with the slope's differences dl, dr and k2 = dt / dx; adds to
// wb and irb what goes to the cell's state and 1/rho other than through the
// differences and the identity part of the centre, and returns the adjoints of
// dl and dr.  The forward part is half_slope's scaled form, whose coefficients
// are differentiated as they are formed there.
CSH_HD void direction_vjp(const P& w, double ir, const P& dl, const P& dr, double k2, const P& fhi, const P& flo,
                          const P& baseb, P& wb, double& irb, P& dlb, P& drb)
{
    constexpr double s3 = 1.7320508075688772935, ka = 0.28867513459481288225, third = 1.0 / 3.0;
    // ---- forward: half_slope and the tracing coefficients ----
    const double t = w.pxx * ir, y = rsqrt(t), c = t * y, a = s3 * c;  // y = 1 / c
    const double ip = y * y * ir, q = w.pxy * ip, rc = w.pxx * y, ra = s3 * rc, q2 = q + q;
    const double ip3 = ip * third, kr = w.r * ip3, g3 = w.pyy * ip3, p3 = w.pxy * ip3, qq3 = q * p3;
    const double k4 = 4.0 * qq3 - g3, cp = 2.0 * qq3 + g3;
    const double z = y * ir, bu = ka * z, hz = 0.5 * z;
    auto project = [&](const P& d, double (&al)[6]) {
        const double s = d.pxy - q * d.pxx, h = q * d.u - d.v;
        al[0] = d.pxx - ra * d.u;
        al[5] = d.pxx + ra * d.u;
        al[1] = s + rc * h;
        al[4] = s - rc * h;
        al[2] = d.r - kr * d.pxx;
        al[3] = d.pyy - q2 * d.pxy + k4 * d.pxx;
    };
    double l[6], r[6], m[6], wl[6], wr[6];
    project(dl, l);
    project(dr, r);
    for (int n = 0; n < 6; ++n) {
        const McVjp v = mc_half_vjp(l[n], r[n]);
        m[n] = v.m;
        wl[n] = v.wl;
        wr[n] = v.wr;
    }
    const double S = m[0] + m[5], D = m[5] - m[0], S2 = m[1] + m[4], D2 = m[4] - m[1];
    P h;
    h.pxx = 0.5 * S;
    h.r = kr * h.pxx + m[2];
    h.u = bu * D;
    h.v = q * h.u + hz * D2;
    h.pxy = q * h.pxx + 0.5 * S2;
    h.pyy = cp * h.pxx + (q * S2 + m[3]);
    const double up = w.u + a, um = w.u - a;
    const double chi = 1.0 + k2 * fmin(up, 0.0), clo = 1.0 - k2 * fmax(um, 0.0);
    // ---- reverse: hi = base + chi h, lo = base - clo h, base -= k2 A h ----
    const double chib = up < 0.0 ? k2 * dot(h, fhi) : 0.0, clob = um > 0.0 ? k2 * dot(h, flo) : 0.0;
    wb.u += chib + clob;
    double ab = chib - clob;
    const P o = scale(-k2, baseb);
    wb.u += dot(h, o);
    wb.r += h.u * o.r;
    wb.pxx += 3.0 * h.u * o.pxx + h.v * o.pxy;
    wb.pxy += 2.0 * (h.u * o.pxy + h.v * o.pyy);
    wb.pyy += h.u * o.pyy;
    irb += h.pxx * o.u + h.pxy * o.v;
    P hb = axpy(w.u, o, axpy(chi, fhi, scale(-clo, flo)));
    hb.u += w.r * o.r + 3.0 * w.pxx * o.pxx + 2.0 * w.pxy * o.pxy + w.pyy * o.pyy;
    hb.v += w.pxx * o.pxy + 2.0 * w.pxy * o.pyy;
    hb.pxx += ir * o.u;
    hb.pxy += ir * o.v;
    // the back-projection
    const double hub = hb.u + q * hb.v;
    const double hpb = hb.pxx + cp * hb.pyy + q * hb.pxy + kr * hb.r;
    double qb = S2 * hb.pyy + h.pxx * hb.pxy + h.u * hb.v;
    double krb = h.pxx * hb.r;
    const double cpb = h.pxx * hb.pyy;
    const double Sb = 0.5 * hpb, Db = bu * hub, S2b = q * hb.pyy + 0.5 * hb.pxy, D2b = hz * hb.v;
    const double zb = ka * (D * hub) + 0.5 * (D2 * hb.v);
    const double mb[6] = {Sb - Db, S2b - D2b, hb.r, hb.pyy, S2b + D2b, Sb + Db};
    // the limiter and the two projections
    double rcb = 0.0, rab = 0.0, k4b = 0.0;
    auto project_vjp = [&](const P& d, const double (&wk)[6], P& db) {
        const double a0 = wk[0] * mb[0], a1 = wk[1] * mb[1], a2 = wk[2] * mb[2], a3 = wk[3] * mb[3];
        const double a4 = wk[4] * mb[4], a5 = wk[5] * mb[5];
        const double sb = a1 + a4, eb = a1 - a4, fb = a5 - a0, hh = rc * eb;
        rcb += (q * d.u - d.v) * eb;
        rab += d.u * fb;
        qb += d.u * hh - d.pxx * sb - 2.0 * d.pxy * a3;
        krb -= d.pxx * a2;
        k4b += d.pxx * a3;
        db = {a2, q * hh + ra * fb, -hh, a0 + a5 - q * sb - kr * a2 + k4 * a3, sb - q2 * a3, a3};
    };
    project_vjp(dl, wl, dlb);
    project_vjp(dr, wr, drb);
    // the coefficients
    const double qq3b = 2.0 * cpb + 4.0 * k4b, g3b = cpb - k4b, p3b = q * qq3b;
    qb += p3 * qq3b;
    wb.pyy += ip3 * g3b;
    wb.r += ip3 * krb;
    wb.pxy += ip3 * p3b + ip * qb;
    const double ipb = third * (w.pxy * p3b + w.pyy * g3b + w.r * krb) + w.pxy * qb;
    rcb += s3 * rab;
    const double yb = w.pxx * rcb + ir * zb - (s3 * ab) * (c * c);  // a = s3 / y
    const double tb = -0.5 * (y * (y * y)) * yb;                    // y = t^(-1/2)
    wb.pxx += y * rcb - ip * ip * ipb + ir * tb;
    irb += y * zb + w.pxx * tb;
}

CSH_HD void face_states_vjp_y(const P& W0, const P& Wm, const P& Wp, double ky, const Faces<double>& fb, P& W0b,
                              P& Wmb, P& Wpb)
{
    const double ir = rcp(W0.r);
    P wb = zero_p(), dlb, drb;
    double irb = 0.0;
    direction_vjp(swap(W0), ir, swap(sub(W0, Wm)), swap(sub(Wp, W0)), ky + ky, swapb(fb.yhi), swapb(fb.ylo),
                  swapb(base_adjoint(fb, true)), wb, irb, dlb, drb);
    // dl = W0 - Wm, dr = Wp - W0, ir = 1 / W0.r
    wb.r -= ir * ir * irb;
    acc(W0b, swapb(sub(axpy(1.0, wb, dlb), drb)));
    acc(Wmb, swapb(scale(-1.0, dlb)));
    acc(Wpb, swapb(drb));
}

template <bool TWOD>
CSH_HD void face_states_vjp_x(const P& W0, const P& Wl, const P& Wr, double kx, const Faces<double>& fb, P& W0b,
                              P& Wlb, P& Wrb)
{
    const double ir = rcp(W0.r);
    const P baseb = base_adjoint(fb, TWOD);
    P wb = baseb, dlb, drb;  // base = W0 + ...
    double irb = 0.0;
    direction_vjp(W0, ir, sub(W0, Wl), sub(Wr, W0), kx + kx, fb.xhi, fb.xlo, baseb, wb, irb, dlb, drb);
    // dl = W0 - Wl, dr = Wr - W0, ir = 1 / W0.r
    wb.r -= ir * ir * irb;
    acc(W0b, sub(axpy(1.0, wb, dlb), drb));
    acc(Wlb, scale(-1.0, dlb));
    acc(Wrb, drb);
}

// reverse of face_states<double, TWOD>(W0, ir, Wl, Wr, Wm, Wp, kx, ky)
template <bool TWOD>
CSH_HD void face_states_vjp(const P& W0, const P& Wl, const P& Wr, const P& Wm, const P& Wp, double kx, double ky,
                            const Faces<double>& fb, P& W0b, P& Wlb, P& Wrb, P& Wmb, P& Wpb)
{
    if constexpr (TWOD) face_states_vjp_y(W0, Wm, Wp, ky, fb, W0b, Wmb, Wpb);
    face_states_vjp_x<TWOD>(W0, Wl, Wr, kx, fb, W0b, Wlb, Wrb);
}

// to_cons(w): mx = r u, my = r v, exx = pxx + mx u, exy = pxy + mx v, eyy = pyy + my v
CSH_HD void to_cons_vjp(const P& w, const C& Ub, P& wb)
{
    const double mx = w.r * w.u, my = w.r * w.v;
    wb.pxx += Ub.exx;
    wb.pxy += Ub.exy;
    wb.pyy += Ub.eyy;
    const double mxb = Ub.mx + w.u * Ub.exx + w.v * Ub.exy;
    const double myb = Ub.my + w.v * Ub.eyy;
    wb.u += mx * Ub.exx + w.r * mxb;
    wb.v += mx * Ub.exy + my * Ub.eyy + w.r * myb;
    wb.r += Ub.r + w.u * mxb + w.v * myb;
}

// to_prim(U): u = mx ir, v = my ir, pxx = exx - mx u, pxy = exy - mx v, pyy = eyy - my v
CSH_HD void to_prim_vjp(const C& U, const P& wb, C& Ub)
{
    const double ir = rcp(U.r);
    const double u = U.mx * ir, v = U.my * ir;
    Ub.exx += wb.pxx;
    Ub.exy += wb.pxy;
    Ub.eyy += wb.pyy;
    const double ub = wb.u - U.mx * wb.pxx;
    const double vb = wb.v - U.mx * wb.pxy - U.my * wb.pyy;
    Ub.mx += -u * wb.pxx - v * wb.pxy + ir * ub;
    Ub.my += -v * wb.pyy + ir * vb;
    const double irb = U.mx * ub + U.my * vb;
    Ub.r += wb.r - ir * ir * irb;
}

// w (F - s U) of one side (moving_flux_x), reversed: from the adjoint Xb of
// F - s U, adds to the state's adjoint and returns that of s.  X1, X2: its
// momentum components.
CSH_HD double moving_flux_vjp(const P& w, double s, double X1, double X2, const C& Xb, P& wb)
{
    const double sp = w.u - s, m = w.r * sp, g = sp + w.u;
    const double X2b = Xb.my + w.v * Xb.eyy, X1b = Xb.mx + w.u * Xb.exx + w.v * Xb.exy;
    const double gb = w.pxx * Xb.exx + w.pxy * Xb.exy;
    const double mb = Xb.r + w.v * X2b + w.u * X1b;
    const double spb = w.pyy * Xb.eyy + w.r * mb + gb;
    wb.r += sp * mb;
    wb.u += X1 * Xb.exx + m * X1b + gb + spb;
    wb.v += (X2 + w.pxy) * Xb.eyy + X1 * Xb.exy + m * X2b;
    wb.pxx += g * Xb.exx + X1b;
    wb.pxy += w.v * Xb.eyy + g * Xb.exy + X2b;
    wb.pyy += sp * Xb.eyy;
    return -spb;
}

// hll_x(make_face_x(wl), make_face_x(wr)): adjoints of the two primitive face
// states.  F = a X_L - b X_R with a = S_R' / (S_R' - S_L'), b = S_L' / (S_R' - S_L')
// (a - b = 1) and X_K = F_K - S_K' U_K, whose dependence on S_K' is reversed with
// the rest of X_K.
CSH_HD void hll_vjp(const P& wl, const P& wr, const C& Fb, P& wlb, P& wrb)
{
    constexpr double s3 = 1.7320508075688772935;
    const double yl = rsqrt(wl.pxx * wl.r), yr = rsqrt(wr.pxx * wr.r);
    const double cl = wl.pxx * yl, cr = wr.pxx * yr;  // sqrt(Pxx / rho)
    const double A1 = wl.u - s3 * cl, B1 = wr.u - s3 * cr;
    const double C1 = wl.u + s3 * cl, D1 = wr.u + s3 * cr;
    const double sl = fmin(fmin(A1, B1), 0.0);
    const double sr = fmax(fmax(C1, D1), 0.0);
    const double inv = rcp(sr - sl);
    const double a = sr * inv, b = sl * inv;
    const C XL = moving_flux_x(wl, sl), XR = moving_flux_x(wr, sr);
    const double t = inv * ((XL.r - XR.r) * Fb.r + (XL.mx - XR.mx) * Fb.mx + (XL.my - XR.my) * Fb.my +
                            (XL.exx - XR.exx) * Fb.exx + (XL.exy - XR.exy) * Fb.exy + (XL.eyy - XR.eyy) * Fb.eyy);
    auto weighted = [&](double k) -> C {
        return {k * Fb.r, k * Fb.mx, k * Fb.my, k * Fb.exx, k * Fb.exy, k * Fb.eyy};
    };
    const double slb = a * t + moving_flux_vjp(wl, sl, XL.mx, XL.my, weighted(a), wlb);
    const double srb = moving_flux_vjp(wr, sr, XR.mx, XR.my, weighted(-b), wrb) - b * t;
    // the speed estimates: the first argument on ties, no slope where clipped at 0
    const bool ll = A1 <= B1, rl = C1 >= D1;
    const double sbl = fmin(A1, B1) < 0.0 ? slb : 0.0, sbr = fmax(C1, D1) > 0.0 ? srb : 0.0;
    const double l1 = ll ? sbl : 0.0, l2 = ll ? 0.0 : sbl, r1 = rl ? sbr : 0.0, r2 = rl ? 0.0 : sbr;
    wlb.u += l1 + r1;
    wrb.u += l2 + r2;
    // a = s3 sqrt(Pxx / rho): da/dPxx = s3 y / 2, da/drho = -s3 y (Pxx / rho) / 2
    const double hl = 0.5 * s3 * yl * (r1 - l1), hr = 0.5 * s3 * yr * (r2 - l2);
    wlb.pxx += hl;
    wlb.r -= hl * (cl * cl);
    wrb.pxx += hr;
    wrb.r -= hr * (cr * cr);
}

// the fixed-field kick is affine in U with a constant Jacobian K; lam' = K^T lam
CSH_HD C kick_vjp(const C& lb, double h, double ax, double ay)
{
    C o = lb;
    o.r += h * ax * lb.mx + h * ay * lb.my + h * h * (ax * ax * lb.exx + ax * ay * lb.exy + ay * ay * lb.eyy);
    o.mx += 2.0 * h * ax * lb.exx + h * ay * lb.exy;
    o.my += h * ax * lb.exy + 2.0 * h * ay * lb.eyy;
    return o;
}

// ---- per-cell bodies of the adjoint kernels ----------------------------------------------

struct AdjArgs {
    int nx, ny, bcx, bcy;
    int ex, ey;          // extended grid: ex = nx + 2, ey = ny + 2 (1-D: 1)
    double dx, dy, dt;
    double kx, ky;       // dt / (2 dx), dt / (2 dy) (1-D: ky = 0)
    double cx, cy;       // dt / dx, dt / dy
    double vc2, rc2, x0, y0;
    const double* U;     // [6][ny][nx]
    const double* lam1;  // lam^{n+1}
    double* lam0;        // lam^n
    double* FS;          // [4 faces][6][ext]
    double* FSb;         // [4][6][ext]
    double* Cs;          // [3 roles][6][ext]: the y part's shares (SELF, DOWN, UP)
    double* XS;          // [6][ey][nx + 4]: per padded position (column -2 .. nx + 1 of an extended
                         // row), SELF and the x part's shares summed
};

// the step factors of AdjArgs from dt, dx, dy (IEEE divisions, once per call)
CSH_HD void set_step_factors(AdjArgs& a)
{
    a.kx = a.dt / (2.0 * a.dx);
    a.ky = a.ey > 1 ? a.dt / (2.0 * a.dy) : 0.0;
    a.cx = a.dt / a.dx;
    a.cy = a.ey > 1 ? a.dt / a.dy : 0.0;
}

// the workspace of a 1-D grid: the two x-face states of every extended cell, their
// adjoints, the sums per padded position
CSH_HD size_t workspace_1d(int nx) { return 24 * (size_t)(nx + 2) + 6 * (size_t)(nx + 4); }
CSH_HD void set_workspace_1d(AdjArgs& a, double* ws)
{
    a.FS = ws;
    a.FSb = ws + 12 * (size_t)a.ex;
    a.XS = ws + 24 * (size_t)a.ex;
}

enum { XHI = 0, XLO = 1, YHI = 2, YLO = 3 };
enum { SELF = 0, DOWN = 1, UP = 2 };

CSH_HD P load_p(const double* B, size_t plane, size_t slot, size_t idx)
{
    const double* b = B + slot * 6 * plane;
    return {b[idx], b[plane + idx], b[2 * plane + idx], b[3 * plane + idx], b[4 * plane + idx], b[5 * plane + idx]};
}
CSH_HD void store_p(double* B, size_t plane, size_t slot, size_t idx, const P& v)
{
    double* b = B + slot * 6 * plane;
    b[idx] = v.r;
    b[plane + idx] = v.u;
    b[2 * plane + idx] = v.v;
    b[3 * plane + idx] = v.pxx;
    b[4 * plane + idx] = v.pxy;
    b[5 * plane + idx] = v.pyy;
}

// map_index for -2n <= i < 3n (the reverse pass reads at most two cells past
// the extended ring, so any n >= 1 is covered): no division
CSH_HD int map_wide(int i, int n, int bc)
{
    if (bc == 0) {
        if (i < 0) i += n;
        if (i < 0) i += n;
        if (i >= n) i -= n;
        if (i >= n) i -= n;
        return i;
    }
    return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// primitive state of the (possibly ghost) cell (i, j)
CSH_HD P prim_at(const AdjArgs& a, int i, int j, bool twod)
{
    const int gi = map_wide(i, a.nx, a.bcx);
    const int gj = twod ? map_wide(j, a.ny, a.bcy) : 0;
    return to_prim(load_cons<double>(a.U, (size_t)a.nx * a.ny, (size_t)gj * a.nx + gi));
}

CSH_HD size_t ext_index(const AdjArgs& a, int i, int j) { return (size_t)(j + (a.ey > 1 ? 1 : 0)) * a.ex + (i + 1); }

// lam' of interior cell (i, j): the kick's transpose applied to lam^{n+1}
CSH_HD C lam_prime(const AdjArgs& a, int i, int j, bool twod)
{
    const C l = load_cons<double>(a.lam1, (size_t)a.nx * a.ny, (size_t)j * a.nx + i);
    if (a.vc2 == 0.0) return l;
    const double x = a.x0 + (i + 0.5) * a.dx;
    const double y = twod ? a.y0 + (j + 0.5) * a.dy : 0.0;
    const double f = -a.vc2 * rcp(x * x + y * y + a.rc2);
    return kick_vjp(l, a.dt, f * x, f * y);
}

template <bool TWOD>
CSH_HD void faces_cell(const AdjArgs& a, int i, int j)
{
    const double kx = a.kx, ky = TWOD ? a.ky : 0.0;
    const P W0 = prim_at(a, i, j, TWOD);
    const P Wl = prim_at(a, i - 1, j, TWOD), Wr = prim_at(a, i + 1, j, TWOD);
    const P Wm = TWOD ? prim_at(a, i, j - 1, TWOD) : W0, Wp = TWOD ? prim_at(a, i, j + 1, TWOD) : W0;
    const Faces<double> f = face_states<double, TWOD>(W0, rcp(W0.r), Wl, Wr, Wm, Wp, kx, ky);
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    store_p(a.FS, ne, XHI, e, f.xhi);
    store_p(a.FS, ne, XLO, e, f.xlo);
    if (TWOD) {
        store_p(a.FS, ne, YHI, e, f.yhi);
        store_p(a.FS, ne, YLO, e, f.ylo);
    }
}

CSH_HD C csub(const C& p, const C& q, double s)
{
    return {s * (p.r - q.r), s * (p.mx - q.mx), s * (p.my - q.my), s * (p.exx - q.exx), s * (p.exy - q.exy),
            s * (p.eyy - q.eyy)};
}

template <bool TWOD>
CSH_HD void hll_cell(const AdjArgs& a, int i, int j)
{
    const size_t ne = (size_t)a.ex * a.ey;
    const size_t e = ext_index(a, i, j);
    const C z = zero_c();
    // face-state adjoint slots of this cell that no face writes (the outer
    // faces of the ring) are cleared here; every other slot is written by the
    // one face that uses that state
    const bool jin = !TWOD || (j >= 0 && j < a.ny), iin = i >= 0 && i < a.nx;
    if (!(i <= a.nx - 1 && jin)) store_p(a.FSb, ne, XHI, e, zero_p());
    if (!(i >= 0 && jin)) store_p(a.FSb, ne, XLO, e, zero_p());
    if (TWOD) {
        if (!(j <= a.ny - 1 && iin)) store_p(a.FSb, ne, YHI, e, zero_p());
        if (!(j >= 0 && iin)) store_p(a.FSb, ne, YLO, e, zero_p());
    }
    // x face i + 1/2 in an interior row: between extended cells (i, j) and (i + 1, j)
    if (i <= a.nx - 1 && (!TWOD || (j >= 0 && j < a.ny))) {
        const int jj = TWOD ? j : 0;
        const C lp = (i + 1 <= a.nx - 1) ? lam_prime(a, i + 1, jj, TWOD) : z;
        const C lm = (i >= 0) ? lam_prime(a, i, jj, TWOD) : z;
        const C Fb = csub(lp, lm, a.cx);
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(load_p(a.FS, ne, XHI, e), load_p(a.FS, ne, XLO, e + 1), Fb, wlb, wrb);
        store_p(a.FSb, ne, XHI, e, wlb);
        store_p(a.FSb, ne, XLO, e + 1, wrb);
    }
    if (TWOD && j <= a.ny - 1 && i >= 0 && i < a.nx) {
        const C lp = (j + 1 <= a.ny - 1) ? lam_prime(a, i, j + 1, true) : z;
        const C lm = (j >= 0) ? lam_prime(a, i, j, true) : z;
        const C Gb = csub(lp, lm, a.cy);
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(swap(load_p(a.FS, ne, YHI, e)), swap(load_p(a.FS, ne, YLO, e + a.ex)), swap(Gb), wlb, wrb);
        store_p(a.FSb, ne, YHI, e, swapb(wlb));
        store_p(a.FSb, ne, YLO, e + a.ex, swapb(wrb));
    }
}

CSH_HD Faces<double> load_face_adjoints(const AdjArgs& a, size_t ne, size_t e, bool twod)
{
    Faces<double> fb;
    fb.xhi = load_p(a.FSb, ne, XHI, e);
    fb.xlo = load_p(a.FSb, ne, XLO, e);
    if (twod) {
        fb.yhi = load_p(a.FSb, ne, YHI, e);
        fb.ylo = load_p(a.FSb, ne, YLO, e);
    } else {
        fb.yhi = fb.ylo = zero_p();
    }
    return fb;
}

// y part of the face-state adjoint of extended cell (i, j) (2-D): slots SELF
// (its share), DOWN, UP
CSH_HD void cells_cell_y(const AdjArgs& a, int i, int j)
{
    const double ky = a.ky;
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    const P W0 = prim_at(a, i, j, true);
    const P Wm = prim_at(a, i, j - 1, true), Wp = prim_at(a, i, j + 1, true);
    const Faces<double> fb = load_face_adjoints(a, ne, e, true);
    P b0 = zero_p(), bm = zero_p(), bp = zero_p();
    face_states_vjp_y(W0, Wm, Wp, ky, fb, b0, bm, bp);
    store_p(a.Cs, ne, SELF, e, b0);
    store_p(a.Cs, ne, DOWN, e, bm);
    store_p(a.Cs, ne, UP, e, bp);
}

// x part of extended cell (i, j): b0 = its SELF share (2-D: the y part's plus
// this part's), bl, br its LEFT and RIGHT shares (to positions i - 1, i + 1)
template <bool TWOD>
CSH_HD void cells_x_vjp(const AdjArgs& a, int i, int j, P& b0, P& bl, P& br)
{
    const double kx = a.kx;
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    const P W0 = prim_at(a, i, j, TWOD);
    const P Wl = prim_at(a, i - 1, j, TWOD), Wr = prim_at(a, i + 1, j, TWOD);
    const Faces<double> fb = load_face_adjoints(a, ne, e, TWOD);
    b0 = TWOD ? load_p(a.Cs, ne, SELF, e) : zero_p();
    bl = zero_p();
    br = zero_p();
    face_states_vjp_x<TWOD>(W0, Wl, Wr, kx, fb, b0, bl, br);
}

// index of padded position (px, j), px in [-2, nx + 1], j an extended row, in XS
CSH_HD size_t xs_index(const AdjArgs& a, int px, int j) { return (size_t)(j + (a.ey > 1 ? 1 : 0)) * (a.nx + 4) + (px + 2); }

// positions p in [-2, n+1] (the ghost-padded range the stencil reads) with
// map(p) == i; returns their count (at most 5)
CSH_HD int preimages(int i, int n, int bc, int* p)
{
    int k = 0;
    if (bc == 0) {  // periodic: p = i + m n
        for (int m = -3; m <= 3; ++m) {
            const int q = i + m * n;
            if (q >= -2 && q <= n + 1) p[k++] = q;
        }
    } else {        // outflow: clamp(p) == i
        const int lo = (i == 0) ? -2 : i, hi = (i == n - 1) ? n + 1 : i;
        for (int q = lo; q <= hi; ++q) p[k++] = q;
    }
    return k;
}

// sum of the shares that land on padded position (pi, pj): the x-part sum of
// its row (extended rows only) and the y part's DOWN and UP shares of the
// extended cells above and below
template <bool TWOD>
CSH_HD P pad_sum(const AdjArgs& a, int pi, int pj)
{
    const size_t ne = (size_t)a.ex * a.ey, nxs = (size_t)(a.nx + 4) * a.ey;
    auto in_ext = [&](int i, int j) { return i >= -1 && i <= a.nx && (!TWOD || (j >= -1 && j <= a.ny)); };
    P s = zero_p();
    if (!TWOD || (pj >= -1 && pj <= a.ny)) acc(s, load_p(a.XS, nxs, 0, xs_index(a, pi, pj)));
    if (TWOD) {
        if (in_ext(pi, pj + 1)) acc(s, load_p(a.Cs, ne, DOWN, ext_index(a, pi, pj + 1)));
        if (in_ext(pi, pj - 1)) acc(s, load_p(a.Cs, ne, UP, ext_index(a, pi, pj - 1)));
    }
    return s;
}

template <bool TWOD>
CSH_HD void gather_cell(const AdjArgs& a, int i, int j)
{
    int px[5], py[5];
    const int nx_ = preimages(i, a.nx, a.bcx, px);
    const int ny_ = TWOD ? preimages(j, a.ny, a.bcy, py) : 1;
    if (!TWOD) py[0] = 0;
    P wb = zero_p();
    for (int u = 0; u < nx_; ++u)
        for (int v = 0; v < ny_; ++v) acc(wb, pad_sum<TWOD>(a, px[u], py[v]));
    const size_t plane = (size_t)a.nx * a.ny, c = (size_t)j * a.nx + i;
    C out = lam_prime(a, i, j, TWOD);
    to_prim_vjp(load_cons<double>(a.U, plane, c), wb, out);
    store_cons(a.lam0, plane, c, out);
}

// ---- the reverse pass by tiles, on the CPU (2-D) -----------------------------------------
//
// The phases of a tiled reverse pass in two kernels, A (faces and fluxes) and B
// (face states and gather), as bodies a CPU loop over tiles, phases and threads
// runs (tests/host).  The device runs both phases in one kernel with the same
// treatment of the boundaries; these bodies show it equal to the per-cell
// reference above.  Only the face-state adjoints (FSb) pass from A to B.
//
// Periodic axes are treated as a pure wrap: a virtual cell outside [0, n) is
// the wrapped cell (its state, its lam' and its face-state adjoints), every
// face is a real face, and an output cell gathers only the shares that land on
// itself.  Outflow axes keep the extended ring (cells -1 and n, lam' = 0
// outside [0, n)), and the shares landing on ghost positions (-2, -1, n,
// n + 1) are folded into the boundary cell.  Both are the transpose of the
// same forward step; they differ from the five-stage pass only in the order
// of the sums.
//
// kernel A: a tile of kA_TX x kA_TY extended cells, one thread per cell
constexpr int kA_TX = 32, kA_TY = 8, kA_THREADS = kA_TX * kA_TY;
constexpr int kA_WX = kA_TX + 3, kA_WY = kA_TY + 3;  // states: cells [X0 - 1, X0 + TX + 2)
constexpr int kA_FX = kA_TX + 1, kA_FY = kA_TY + 1;  // face states: cells [X0, X0 + TX + 1)
constexpr int kA_NW = kA_WX * kA_WY, kA_NF = kA_FX * kA_FY;
constexpr int kA_LDS = 6 * kA_NW + 12 * kA_NF;       // doubles of LDS: states, low x and y face states

// kernel B: a tile of kB_W x kB_H virtual cells (four rows per wavefront),
// the outputs its inner (kB_W - 2) x (kB_H - 2) cells
constexpr int kB_W = 16, kB_H = 16, kB_THREADS = kB_W * kB_H;
constexpr int kB_OX = kB_W - 2, kB_OY = kB_H - 2;
enum { SH_LEFT = 0, SH_RIGHT = 1, SH_DOWN = 2, SH_UP = 3, SH_TOT = 4 };
constexpr int kB_SX = kB_W + 2, kB_SY = kB_H + 2, kB_NS = kB_SX * kB_SY;  // states: the tile and a ring
constexpr int kB_LDS = 5 * 6 * kB_THREADS + 6 * kB_NS;  // doubles of LDS (the states after the shares)

CSH_HD void lds_put(double* L, int stride, int base, int k, const P& v)
{
    L[base + 0 * stride + k] = v.r;
    L[base + 1 * stride + k] = v.u;
    L[base + 2 * stride + k] = v.v;
    L[base + 3 * stride + k] = v.pxx;
    L[base + 4 * stride + k] = v.pxy;
    L[base + 5 * stride + k] = v.pyy;
}
CSH_HD P lds_get(const double* L, int stride, int base, int k)
{
    return {L[base + k], L[base + stride + k], L[base + 2 * stride + k], L[base + 3 * stride + k],
            L[base + 4 * stride + k], L[base + 5 * stride + k]};
}

// lam' of a virtual cell: wrapped on periodic axes; zero outside the grid on outflow ones
CSH_HD C lam_prime_virtual(const AdjArgs& a, int i, int j)
{
    if (a.bcx != 0 && (i < 0 || i >= a.nx)) return zero_c();
    if (a.bcy != 0 && (j < 0 || j >= a.ny)) return zero_c();
    return lam_prime(a, map_wide(i, a.nx, a.bcx), map_wide(j, a.ny, a.bcy), true);
}

// A1: primitive states of the cells [X0 - 1, X0 + TX + 2) x [Y0 - 1, Y0 + TY + 2)
// (coordinates past [-2, n + 1] are clamped into it: those cells only feed
// face states of cells beyond the extended ring, which no face uses)
CSH_HD void tileA_states(const AdjArgs& a, int X0, int Y0, int t, double* L)
{
    for (int k = t; k < kA_NW; k += kA_THREADS) {
        const int i0 = X0 - 1 + k % kA_WX, j0 = Y0 - 1 + k / kA_WX;
        const int i = i0 < -2 ? -2 : (i0 > a.nx + 1 ? a.nx + 1 : i0);
        const int j = j0 < -2 ? -2 : (j0 > a.ny + 1 ? a.ny + 1 : j0);
        lds_put(L, kA_NW, 0, k, prim_at(a, i, j, true));
    }
}

// face states of cell k of the face-state block [X0, X0 + TX + 1) x [Y0, Y0 + TY + 1)
CSH_HD Faces<double> tileA_face_states(const AdjArgs& a, int k, const double* L)
{
    const int lx = k % kA_FX + 1, ly = k / kA_FX + 1;  // position in the state block
    const int c = ly * kA_WX + lx;
    const P W0 = lds_get(L, kA_NW, 0, c);
    return face_states<double, true>(W0, rcp(W0.r), lds_get(L, kA_NW, 0, c - 1), lds_get(L, kA_NW, 0, c + 1),
                                     lds_get(L, kA_NW, 0, c - kA_WX), lds_get(L, kA_NW, 0, c + kA_WX), a.kx, a.ky);
}

// A2: the face states of the thread's own cell e = (X0 + t % TX, Y0 + t / TX):
// the high ones kept (returned), the low ones written to LDS for the faces of
// the cells to the left and below; then the low x face states of the column
// to the right of the tile and the low y face states of the row above it
CSH_HD void tileA_faces(const AdjArgs& a, int t, double* L, P& xhi, P& yhi)
{
    double* X = L + 6 * kA_NW;
    double* Y = X + 6 * kA_NF;
    const int k = (t / kA_TX) * kA_FX + t % kA_TX;
    const Faces<double> f = tileA_face_states(a, k, L);
    xhi = f.xhi;
    yhi = f.yhi;
    lds_put(X, kA_NF, 0, k, f.xlo);
    lds_put(Y, kA_NF, 0, k, f.ylo);
    if (t < kA_TY + kA_TX) {
        const bool col = t < kA_TY;  // the column x = X0 + TX, else the row y = Y0 + TY
        const int k2 = col ? t * kA_FX + kA_TX : kA_TY * kA_FX + (t - kA_TY);
        const Faces<double> g = tileA_face_states(a, k2, L);
        if (col) lds_put(X, kA_NF, 0, k2, g.xlo);
        else lds_put(Y, kA_NF, 0, k2, g.ylo);
    }
}

// A3: the extended cell e of the thread: the flux adjoints of its high x and
// y faces, through HLL into the adjoints of the two face states of each
// (written to FSb); the slots of the ring that no face writes are cleared
CSH_HD void tileA_fluxes(const AdjArgs& a, int X0, int Y0, int t, const double* L, const P& xhi, const P& yhi)
{
    const double* X = L + 6 * kA_NW;
    const double* Y = X + 6 * kA_NF;
    const int i = X0 + t % kA_TX, j = Y0 + t / kA_TX;
    if (i > a.nx || j > a.ny) return;  // outside the extended grid
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    const int k = (t / kA_TX) * kA_FX + t % kA_TX;  // e in the face-state block
    if (i == a.nx) store_p(a.FSb, ne, XHI, e, zero_p());
    if (i == -1) store_p(a.FSb, ne, XLO, e, zero_p());
    if (j == a.ny) store_p(a.FSb, ne, YHI, e, zero_p());
    if (j == -1) store_p(a.FSb, ne, YLO, e, zero_p());
    if (i == a.nx && j == a.ny) return;
    const C l0 = lam_prime_virtual(a, i, j);
    if (i <= a.nx - 1) {  // x face i + 1/2
        const C Fb = csub(lam_prime_virtual(a, i + 1, j), l0, a.cx);
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(xhi, lds_get(X, kA_NF, 0, k + 1), Fb, wlb, wrb);
        store_p(a.FSb, ne, XHI, e, wlb);
        store_p(a.FSb, ne, XLO, e + 1, wrb);
    }
    if (j <= a.ny - 1) {  // y face j + 1/2
        const C Gb = csub(lam_prime_virtual(a, i, j + 1), l0, a.cy);
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(swap(yhi), swap(lds_get(Y, kA_NF, 0, k + kA_FX)), swap(Gb), wlb, wrb);
        store_p(a.FSb, ne, YHI, e, swapb(wlb));
        store_p(a.FSb, ne, YLO, e + a.ex, swapb(wrb));
    }
}

// index of a virtual cell in the extended face-state arrays, -1 for a cell
// beyond the ring [-1, n] (its shares reach no output: on an outflow axis its
// face states feed no face, on a periodic one it is not next to an output);
// a ring cell of a periodic axis is the wrapped cell
CSH_HD long ext_of_virtual(const AdjArgs& a, int i, int j)
{
    if (i < -1 || i > a.nx || j < -1 || j > a.ny) return -1;
    if (a.bcx == 0) i = map_wide(i, a.nx, 0);
    if (a.bcy == 0) j = map_wide(j, a.ny, 0);
    return (long)ext_index(a, i, j);
}

// B0: primitive states of the tile and its ring, cells [X0 - 2, X0 + kB_W) x
// [Y0 - 2, Y0 + kB_H) (coordinates clamped into [-2, n + 1], as in A1)
CSH_HD void tileB_states(const AdjArgs& a, int X0, int Y0, int t, double* L)
{
    double* S = L + 5 * 6 * kB_THREADS;
    for (int k = t; k < kB_NS; k += kB_THREADS) {
        const int i0 = X0 - 2 + k % kB_SX, j0 = Y0 - 2 + k / kB_SX;
        const int i = i0 < -2 ? -2 : (i0 > a.nx + 1 ? a.nx + 1 : i0);
        const int j = j0 < -2 ? -2 : (j0 > a.ny + 1 ? a.ny + 1 : j0);
        lds_put(S, kB_NS, 0, k, prim_at(a, i, j, true));
    }
}

// the face-state adjoints of the thread's cell; zero beyond the ring
CSH_HD Faces<double> tileB_face_adjoints(const AdjArgs& a, int X0, int Y0, int t)
{
    const long e = ext_of_virtual(a, X0 - 1 + t % kB_W, Y0 - 1 + t / kB_W);
    if (e < 0) return {zero_p(), zero_p(), zero_p(), zero_p()};
    return load_face_adjoints(a, (size_t)a.ex * a.ey, (size_t)e, true);
}

// B1: the face-state reverse pass of the virtual cell at column l, row w of the
// tile (X0 - 1 + l, Y0 - 1 + w) from its face-state adjoints fb: its own share
// returned, the four it gives its neighbours written to LDS
CSH_HD P tileB_shares(const AdjArgs& a, int X0, int Y0, int t, double* L, const Faces<double>& fb)
{
    const double* S = L + 5 * 6 * kB_THREADS;
    const int l = t % kB_W, w = t / kB_W;
    const int i = X0 - 1 + l, j = Y0 - 1 + w;
    const int c = (w + 1) * kB_SX + (l + 1);  // the cell in the state block
    P b0 = zero_p();
    const long e = ext_of_virtual(a, i, j);
    // the y part first, its two neighbour shares stored before the x part
    // starts (fewer values live at once)
    const P W0 = e >= 0 ? lds_get(S, kB_NS, 0, c) : zero_p();
    {
        P bm = zero_p(), bp = zero_p();
        if (e >= 0)
            face_states_vjp_y(W0, lds_get(S, kB_NS, 0, c - kB_SX), lds_get(S, kB_NS, 0, c + kB_SX), a.ky, fb, b0, bm,
                              bp);
        lds_put(L, kB_THREADS, SH_DOWN * 6 * kB_THREADS, t, bm);
        lds_put(L, kB_THREADS, SH_UP * 6 * kB_THREADS, t, bp);
    }
    P bl = zero_p(), br = zero_p();
    if (e >= 0)
        face_states_vjp_x<true>(W0, lds_get(S, kB_NS, 0, c - 1), lds_get(S, kB_NS, 0, c + 1), a.kx, fb, b0, bl, br);
    lds_put(L, kB_THREADS, SH_LEFT * 6 * kB_THREADS, t, bl);
    lds_put(L, kB_THREADS, SH_RIGHT * 6 * kB_THREADS, t, br);
    return b0;
}

// B2: everything that lands on the position of column l, row w from inside the tile
CSH_HD P tileB_total(int t, const P& self, const double* L)
{
    const int l = t % kB_W, w = t / kB_W;
    P s = self;
    if (l + 1 < kB_W) acc(s, lds_get(L, kB_THREADS, SH_LEFT * 6 * kB_THREADS, t + 1));
    if (l >= 1) acc(s, lds_get(L, kB_THREADS, SH_RIGHT * 6 * kB_THREADS, t - 1));
    if (w >= 1) acc(s, lds_get(L, kB_THREADS, SH_UP * 6 * kB_THREADS, t - kB_W));
    if (w + 1 < kB_H) acc(s, lds_get(L, kB_THREADS, SH_DOWN * 6 * kB_THREADS, t + kB_W));
    return s;
}

CSH_HD void tileB_put_total(int t, const P& s, double* L) { lds_put(L, kB_THREADS, SH_TOT * 6 * kB_THREADS, t, s); }

// what lands on tile position (lp, wp), lp in [-1, kB_W], wp in [-1, kB_H]:
// the total inside the tile, or the one share a tile cell gives a position just
// outside it (the cells beyond it feed only ghost positions of outflow axes
// through shares that are zero: they lie past the extended ring)
CSH_HD P tileB_landing(int lp, int wp, const double* L)
{
    const bool xin = lp >= 0 && lp < kB_W, yin = wp >= 0 && wp < kB_H;
    if (xin && yin) return lds_get(L, kB_THREADS, SH_TOT * 6 * kB_THREADS, wp * kB_W + lp);
    if (yin && lp == -1) return lds_get(L, kB_THREADS, SH_LEFT * 6 * kB_THREADS, wp * kB_W);
    if (yin && lp == kB_W) return lds_get(L, kB_THREADS, SH_RIGHT * 6 * kB_THREADS, wp * kB_W + kB_W - 1);
    if (xin && wp == -1) return lds_get(L, kB_THREADS, SH_DOWN * 6 * kB_THREADS, lp);
    if (xin && wp == kB_H) return lds_get(L, kB_THREADS, SH_UP * 6 * kB_THREADS, (kB_H - 1) * kB_W + lp);
    return zero_p();
}

// positions whose shares belong to output coordinate i on one axis: itself, and
// on an outflow axis the ghost positions the boundary cell stands for
CSH_HD int fold_positions(int i, int n, int bc, int* p)
{
    int k = 0;
    p[k++] = i;
    if (bc != 0) {
        if (i == 0) { p[k++] = -1; p[k++] = -2; }
        if (i == n - 1) { p[k++] = n; p[k++] = n + 1; }
    }
    return k;
}

// B3: the output cell at column l, row w (inner cells only): the folded total of
// the shares on its positions, through W(U), plus lam' itself
CSH_HD void tileB_gather(const AdjArgs& a, int X0, int Y0, int t, const double* L)
{
    const int l = t % kB_W, w = t / kB_W;
    if (l < 1 || l > kB_OX || w < 1 || w > kB_OY) return;
    const int i = X0 - 1 + l, j = Y0 - 1 + w;
    if (i >= a.nx || j >= a.ny) return;
    int px[5], py[5];
    const int nx_ = fold_positions(i, a.nx, a.bcx, px), ny_ = fold_positions(j, a.ny, a.bcy, py);
    P wb = zero_p();
    for (int u = 0; u < nx_; ++u)
        for (int v = 0; v < ny_; ++v) acc(wb, tileB_landing(px[u] - (X0 - 1), py[v] - (Y0 - 1), L));
    const size_t plane = (size_t)a.nx * a.ny, c = (size_t)j * a.nx + i;
    C out = lam_prime(a, i, j, true);
    to_prim_vjp(load_cons<double>(a.U, plane, c), wb, out);
    store_cons(a.lam0, plane, c, out);
}

}  // namespace csh
