// Reverse-mode pieces of the sweep (FP64): vector-Jacobian products of every
// stage of csh_device.h, written out by hand statement by statement in reverse
// order, and the bodies of the adjoint kernels: per cell (1-D) and per thread of a
// block (2-D).
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

// ---- bodies of the adjoint kernels ---------------------------------------------------------

struct AdjArgs {
    int nx, ny, bcx, bcy;
    double dx, dy, dt;
    double kx, ky;       // dt / (2 dx), dt / (2 dy) (1-D: ky = 0)
    double cx, cy;       // dt / dx, dt / dy
    double vc2, rc2, x0, y0;
    const double* U;     // [6][ny][nx]
    const double* lam1;  // lam^{n+1}
    double* lam0;        // lam^n
    // 1-D, over the nx + 2 extended cells
    double* FS;          // [high, low][6][nx + 2]: face states
    double* FSb;         // [high, low][6][nx + 2]: their adjoints
    double* XS;          // [6][nx + 4]: per padded position (-2 .. nx + 1), the shares summed
};

// the step factors of AdjArgs from dt, dx, dy (IEEE divisions, once per call)
CSH_HD void set_step_factors(AdjArgs& a)
{
    a.kx = a.dt / (2.0 * a.dx);
    a.ky = a.ny > 1 ? a.dt / (2.0 * a.dy) : 0.0;
    a.cx = a.dt / a.dx;
    a.cy = a.ny > 1 ? a.dt / a.dy : 0.0;
}

// the workspace of a 1-D grid
CSH_HD size_t workspace_1d(int nx) { return 24 * (size_t)(nx + 2) + 6 * (size_t)(nx + 4); }
CSH_HD void set_workspace_1d(AdjArgs& a, double* ws)
{
    const size_t ne = (size_t)a.nx + 2;
    a.FS = ws;
    a.FSb = ws + 12 * ne;
    a.XS = ws + 24 * ne;
}

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

CSH_HD C csub(const C& p, const C& q, double s)
{
    return {s * (p.r - q.r), s * (p.mx - q.mx), s * (p.my - q.my), s * (p.exx - q.exx), s * (p.exy - q.exy),
            s * (p.eyy - q.eyy)};
}

// the transpose of the kick at (x, y)
CSH_HD C kick_adjoint(const AdjArgs& a, const C& l, double x, double y)
{
    const double f = -a.vc2 * rcp(x * x + y * y + a.rc2);
    return kick_vjp(l, a.dt, f * x, f * y);
}

// ---- 1-D, per cell --------------------------------------------------------------------------
//
// Extended cell i in [-1, nx] lies at index i + 1 of the workspace's arrays; XHI and
// XLO are its high and low face.

enum { XHI = 0, XLO = 1 };

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

// primitive state of the (possibly ghost) cell i
CSH_HD P prim_at(const AdjArgs& a, int i)
{
    return to_prim(load_cons<double>(a.U, (size_t)a.nx, (size_t)map_wide(i, a.nx, a.bcx)));
}

// lam' of interior cell i: the kick's transpose applied to lam^{n+1}
CSH_HD C lam_prime(const AdjArgs& a, int i)
{
    const C l = load_cons<double>(a.lam1, (size_t)a.nx, (size_t)i);
    return a.vc2 == 0.0 ? l : kick_adjoint(a, l, a.x0 + (i + 0.5) * a.dx, 0.0);
}

CSH_HD void faces_cell(const AdjArgs& a, int i)
{
    const P W0 = prim_at(a, i);
    const Faces<double> f =
        face_states<double, false>(W0, rcp(W0.r), prim_at(a, i - 1), prim_at(a, i + 1), W0, W0, a.kx, 0.0);
    const size_t ne = (size_t)a.nx + 2, e = (size_t)(i + 1);
    store_p(a.FS, ne, XHI, e, f.xhi);
    store_p(a.FS, ne, XLO, e, f.xlo);
}

CSH_HD void hll_cell(const AdjArgs& a, int i)
{
    const size_t ne = (size_t)a.nx + 2, e = (size_t)(i + 1);
    const C z = zero_c();
    // the outer faces of the ring, which no flux uses; every other slot is written
    // by the one face that uses that state
    if (i > a.nx - 1) store_p(a.FSb, ne, XHI, e, zero_p());
    if (i < 0) store_p(a.FSb, ne, XLO, e, zero_p());
    // face i + 1/2: between extended cells i and i + 1
    if (i <= a.nx - 1) {
        const C lp = (i + 1 <= a.nx - 1) ? lam_prime(a, i + 1) : z;
        const C lm = (i >= 0) ? lam_prime(a, i) : z;
        const C Fb = csub(lp, lm, a.cx);
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(load_p(a.FS, ne, XHI, e), load_p(a.FS, ne, XLO, e + 1), Fb, wlb, wrb);
        store_p(a.FSb, ne, XHI, e, wlb);
        store_p(a.FSb, ne, XLO, e + 1, wrb);
    }
}

// the face-state reverse pass of extended cell i: b0 its share of itself, bl, br its
// shares of positions i - 1, i + 1
CSH_HD void cells_x_vjp(const AdjArgs& a, int i, P& b0, P& bl, P& br)
{
    const size_t ne = (size_t)a.nx + 2, e = (size_t)(i + 1);
    const Faces<double> fb{load_p(a.FSb, ne, XHI, e), load_p(a.FSb, ne, XLO, e), zero_p(), zero_p()};
    b0 = bl = br = zero_p();
    face_states_vjp_x<false>(prim_at(a, i), prim_at(a, i - 1), prim_at(a, i + 1), a.kx, fb, b0, bl, br);
}

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

CSH_HD void gather_cell(const AdjArgs& a, int i)
{
    int px[5];
    const int n = preimages(i, a.nx, a.bcx, px);
    P wb = zero_p();
    for (int u = 0; u < n; ++u) acc(wb, load_p(a.XS, (size_t)a.nx + 4, 0, (size_t)(px[u] + 2)));
    C out = lam_prime(a, i);
    to_prim_vjp(load_cons<double>(a.U, (size_t)a.nx, (size_t)i), wb, out);
    store_cons(a.lam0, (size_t)a.nx, (size_t)i, out);
}

// ---- 2-D, per thread of a block -------------------------------------------------------------

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

// One thread of the 2-D reverse step (adjoint_fused_kernel): a block of BX x 16 cells,
// its inner (BX - 4) x 12 the outputs, cell (lx, ly) of it this thread's.  The methods
// are the phases between the kernel's barriers and lane shifts, in its order; they hold
// all of its indexing (the boundary maps, the ring, the slots in LDS, the ghost folds),
// so that a CPU loop over blocks, phases and threads runs the same code (tests/host).
constexpr int kF_Y = 16, kF_OY = kF_Y - 4;

template <int BX>
struct AdjointThread {
    static constexpr int SX = BX + 2, OX = BX - 4;
    static constexpr int kStates = (kF_Y + 2) * 6 * SX, kRows = kF_Y * 6 * BX;  // doubles of S; of Y and of M

    const AdjArgs& a;
    double* const S;  // states; later the totals of the positions
    double* const Y;  // low y-face states, their adjoints, the shares downwards
    double* const M;  // lam', then the shares upwards
    int X0, Y0, lx, ly, i, j, gi, gj;
    unsigned cell;
    C lam, Uc, lc;
    P W0, self, left, right;
    double ir;
    Faces<double> f, fb;

    CSH_HD AdjointThread(const AdjArgs& args, double* s, double* y, double* m, unsigned block, int tiles_x, int thread)
        : a(args), S(s), Y(y), M(m)
    {
        X0 = (int)(block % (unsigned)tiles_x) * OX;
        Y0 = (int)(block / (unsigned)tiles_x) * kF_OY;
        lx = thread % BX;
        ly = thread / BX;
        i = X0 - 2 + lx;
        j = Y0 - 2 + ly;
        gi = map(i, a.nx, a.bcx);
        gj = map(j, a.ny, a.bcy);
        cell = (unsigned)(gj * a.nx + gi);
    }

    // cells past [-3, n + 2] feed nothing that is used
    static CSH_HD int map(int k, int n, int bc)
    {
        const int c = k < -3 ? -3 : k;
        return map_index(c < n + 2 ? c : n + 2, n, bc);
    }
    CSH_HD C state_of(unsigned c) const { return Planes<double>(a.U, (size_t)a.nx * a.ny).load(c); }
    CSH_HD C lam_of(unsigned c) const { return Planes<double>(a.lam1, (size_t)a.nx * a.ny).load(c); }
    // rows and columns of S are those of the block, shifted by one
    CSH_HD void put_state(int col, int row, const P& v) { lds_put(S + (row + 1) * 6 * SX, SX, 0, col + 1, v); }
    CSH_HD P state(int col, int row) const { return lds_get(S + (row + 1) * 6 * SX, SX, 0, col + 1); }
    CSH_HD double* yrow(int row) const { return Y + row * 6 * BX; }
    CSH_HD double* mrow(int row) const { return M + row * 6 * BX; }
    // lam' of the mapped cell from its lam^{n+1}
    CSH_HD C lam_prime(const C& l) const
    {
        if (a.vc2 == 0.0) return l;
        return kick_adjoint(a, l, a.x0 + (gi + 0.5) * a.dx, a.y0 + (gj + 0.5) * a.dy);
    }

    // states of the cell and of the ring, lam' of the cell
    CSH_HD void load()
    {
        lam = zero_c();
        if ((a.bcx == 0 || (i >= 0 && i < a.nx)) && (a.bcy == 0 || (j >= 0 && j < a.ny))) lam = lam_prime(lam_of(cell));
        W0 = to_prim(state_of(cell));
        ir = rcp(W0.r);
        put_state(lx, ly, W0);
        if (lx == 0 || lx == BX - 1) {
            const int d = lx == 0 ? -1 : 1;
            put_state(lx + d, ly, to_prim(state_of((unsigned)(gj * a.nx + map(i + d, a.nx, a.bcx)))));
        }
        if (ly == 0 || ly == kF_Y - 1) {
            const int d = ly == 0 ? -1 : 1;
            put_state(lx, ly + d, to_prim(state_of((unsigned)(map(j + d, a.ny, a.bcy) * a.nx + gi))));
        }
        lds_put(mrow(ly), BX, 0, lx, {lam.r, lam.mx, lam.my, lam.exx, lam.exy, lam.eyy});
    }

    // face states
    CSH_HD void faces()
    {
        const P dlx = sub(W0, state(lx - 1, ly)), drx = sub(state(lx + 1, ly), W0);
        f = face_states_d<double, true>(W0, ir, dlx, drx, sub(W0, state(lx, ly - 1)), sub(state(lx, ly + 1), W0), a.kx,
                                        a.ky);
        lds_put(yrow(ly), BX, 0, lx, f.ylo);
        fb = {zero_p(), zero_p(), zero_p(), zero_p()};
    }

    // the high x face, from the low face state and lam' of the cell to the right:
    // returns the adjoint of that face state
    CSH_HD P x_face(const P& xlo, const C& lam_right)
    {
        P low = zero_p();
        hll_vjp(f.xhi, xlo, csub(lam_right, lam, a.cx), fb.xhi, low);
        return low;
    }

    // the high y face, through the row above's slots
    CSH_HD void y_face()
    {
        if (ly == kF_Y - 1) return;
        const P l = lds_get(mrow(ly + 1), BX, 0, lx);
        const C above = {l.r, l.u, l.v, l.pxx, l.pxy, l.pyy};
        P low = zero_p(), high = zero_p();
        hll_vjp(swap(f.yhi), swap(lds_get(yrow(ly + 1), BX, 0, lx)), swap(csub(above, lam, a.cy)), low, high);
        fb.yhi = swapb(low);
        lds_put(yrow(ly + 1), BX, 0, lx, swapb(high));
    }

    // the face-state reverse pass of the cells next to an output, inside the extended ring
    CSH_HD void shares()
    {
        if (ly > 0) fb.ylo = lds_get(yrow(ly), BX, 0, lx);
        const bool inner = lx >= 1 && lx <= BX - 2 && ly >= 1 && ly <= kF_Y - 2 && i >= -1 && i <= a.nx && j >= -1 &&
                           j <= a.ny;
        const P Wc = state(lx, ly);  // W0 again: a register set less through the fluxes
        P down = zero_p(), up = zero_p();
        self = left = right = zero_p();
        if (inner) face_states_vjp_y(Wc, state(lx, ly - 1), state(lx, ly + 1), a.ky, fb, self, down, up);
        lds_put(yrow(ly), BX, 0, lx, down);  // at once: kept through the x part they would spill
        lds_put(mrow(ly), BX, 0, lx, up);
        if (inner) face_states_vjp_x<true>(Wc, state(lx - 1, ly), state(lx + 1, ly), a.kx, fb, self, left, right);
    }

    // what lands on this position from the cells beside it; the state and lam^{n+1}
    // again from the caches: kept in registers they would spill
    CSH_HD void land_x(const P& from_right, const P& from_left)
    {
        acc(self, from_right);
        acc(self, from_left);
        Uc = state_of(cell);
        lc = lam_of(cell);
    }
    // and from those above and below
    CSH_HD void land_y()
    {
        if (ly < kF_Y - 1) acc(self, lds_get(yrow(ly + 1), BX, 0, lx));
        if (ly > 0) acc(self, lds_get(mrow(ly - 1), BX, 0, lx));
    }

    // outflow axes: the two ghost positions on either side belong to the boundary cell
    // (the conditions are uniform in the block); l1, l2, r1, r2: the totals one and two
    // to the left and right
    CSH_HD bool folds_x() const { return a.bcx != 0 && (X0 == 0 || X0 + OX >= a.nx); }
    CSH_HD void fold_x(const P& l1, const P& l2, const P& r1, const P& r2)
    {
        if (i == 0) {
            acc(self, l1);
            acc(self, l2);
        }
        if (i == a.nx - 1) {
            acc(self, r1);
            acc(self, r2);
        }
    }
    CSH_HD bool folds_y() const { return a.bcy != 0 && (Y0 == 0 || Y0 + kF_OY >= a.ny); }
    CSH_HD void put_total() { put_state(lx, ly, self); }  // over the states, last read before the barrier of land_y
    CSH_HD void fold_y()
    {
        if (j == 0 && ly >= 2) {
            acc(self, state(lx, ly - 1));
            acc(self, state(lx, ly - 2));
        }
        if (j == a.ny - 1 && ly <= kF_Y - 3) {
            acc(self, state(lx, ly + 1));
            acc(self, state(lx, ly + 2));
        }
    }

    // the output cells: W(U) reverse and lam'
    CSH_HD void store() const
    {
        if (lx < 2 || lx >= BX - 2 || ly < 2 || ly >= kF_Y - 2 || i >= a.nx || j >= a.ny) return;
        C out = lam_prime(lc);
        to_prim_vjp(Uc, self, out);
        OutPlanes<double>(a.lam0, (size_t)a.nx * a.ny).store(cell, out);
    }
};

}  // namespace csh
