// The 2-D reverse step cell by cell, the CPU reference of the device's blocks: the
// five stages of the 1-D scheme (csh_adjoint.hip) with a y part, over the extended
// grid of (nx + 2) x (ny + 2) cells, every intermediate in memory and no neighbour
// exchange.  Periodic and outflow axes alike gather over the padded positions that
// the boundary mapping sends to a cell, where the device wraps or folds.
#pragma once

#include "csh_adjoint.h"

namespace csh {
namespace ref {

struct Args : AdjArgs {
    int ex, ey;   // nx + 2, ny + 2
    double* FS;   // [4 faces][6][ext]
    double* FSb;  // [4][6][ext]
    double* Cs;   // [3 roles][6][ext]: the y part's shares (SELF, DOWN, UP)
    double* XS;   // [6][ey][nx + 4]: per padded position (column -2 .. nx + 1 of an extended
                  // row), SELF and the x part's shares summed
};

enum { XHI = 0, XLO = 1, YHI = 2, YLO = 3 };
enum { SELF = 0, DOWN = 1, UP = 2 };

// primitive state of the (possibly ghost) cell (i, j)
inline P prim_at(const Args& a, int i, int j)
{
    const int gi = map_wide(i, a.nx, a.bcx), gj = map_wide(j, a.ny, a.bcy);
    return to_prim(load_cons<double>(a.U, (size_t)a.nx * a.ny, (size_t)gj * a.nx + gi));
}

inline size_t ext_index(const Args& a, int i, int j) { return (size_t)(j + 1) * a.ex + (i + 1); }

// lam' of interior cell (i, j): the kick's transpose applied to lam^{n+1}
inline C lam_prime(const Args& a, int i, int j)
{
    const C l = load_cons<double>(a.lam1, (size_t)a.nx * a.ny, (size_t)j * a.nx + i);
    return a.vc2 == 0.0 ? l : kick_adjoint(a, l, a.x0 + (i + 0.5) * a.dx, a.y0 + (j + 0.5) * a.dy);
}

inline void faces_cell(const Args& a, int i, int j)
{
    const P W0 = prim_at(a, i, j);
    const Faces<double> f = face_states<double, true>(W0, rcp(W0.r), prim_at(a, i - 1, j), prim_at(a, i + 1, j),
                                                      prim_at(a, i, j - 1), prim_at(a, i, j + 1), a.kx, a.ky);
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    store_p(a.FS, ne, XHI, e, f.xhi);
    store_p(a.FS, ne, XLO, e, f.xlo);
    store_p(a.FS, ne, YHI, e, f.yhi);
    store_p(a.FS, ne, YLO, e, f.ylo);
}

inline void hll_cell(const Args& a, int i, int j)
{
    const size_t ne = (size_t)a.ex * a.ey;
    const size_t e = ext_index(a, i, j);
    const C z = zero_c();
    // face-state adjoint slots of this cell that no face writes (the outer
    // faces of the ring) are cleared here; every other slot is written by the
    // one face that uses that state
    const bool jin = j >= 0 && j < a.ny, iin = i >= 0 && i < a.nx;
    if (!(i <= a.nx - 1 && jin)) store_p(a.FSb, ne, XHI, e, zero_p());
    if (!(i >= 0 && jin)) store_p(a.FSb, ne, XLO, e, zero_p());
    if (!(j <= a.ny - 1 && iin)) store_p(a.FSb, ne, YHI, e, zero_p());
    if (!(j >= 0 && iin)) store_p(a.FSb, ne, YLO, e, zero_p());
    // x face i + 1/2 in an interior row: between extended cells (i, j) and (i + 1, j)
    if (i <= a.nx - 1 && jin) {
        const C lp = (i + 1 <= a.nx - 1) ? lam_prime(a, i + 1, j) : z;
        const C lm = (i >= 0) ? lam_prime(a, i, j) : z;
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(load_p(a.FS, ne, XHI, e), load_p(a.FS, ne, XLO, e + 1), csub(lp, lm, a.cx), wlb, wrb);
        store_p(a.FSb, ne, XHI, e, wlb);
        store_p(a.FSb, ne, XLO, e + 1, wrb);
    }
    if (j <= a.ny - 1 && iin) {
        const C lp = (j + 1 <= a.ny - 1) ? lam_prime(a, i, j + 1) : z;
        const C lm = (j >= 0) ? lam_prime(a, i, j) : z;
        P wlb = zero_p(), wrb = zero_p();
        hll_vjp(swap(load_p(a.FS, ne, YHI, e)), swap(load_p(a.FS, ne, YLO, e + a.ex)), swap(csub(lp, lm, a.cy)), wlb,
                wrb);
        store_p(a.FSb, ne, YHI, e, swapb(wlb));
        store_p(a.FSb, ne, YLO, e + a.ex, swapb(wrb));
    }
}

inline Faces<double> load_face_adjoints(const Args& a, size_t ne, size_t e)
{
    return {load_p(a.FSb, ne, XHI, e), load_p(a.FSb, ne, XLO, e), load_p(a.FSb, ne, YHI, e),
            load_p(a.FSb, ne, YLO, e)};
}

// y part of the face-state adjoint of extended cell (i, j): slots SELF (its share), DOWN, UP
inline void cells_cell_y(const Args& a, int i, int j)
{
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    P b0 = zero_p(), bm = zero_p(), bp = zero_p();
    face_states_vjp_y(prim_at(a, i, j), prim_at(a, i, j - 1), prim_at(a, i, j + 1), a.ky,
                      load_face_adjoints(a, ne, e), b0, bm, bp);
    store_p(a.Cs, ne, SELF, e, b0);
    store_p(a.Cs, ne, DOWN, e, bm);
    store_p(a.Cs, ne, UP, e, bp);
}

// x part of extended cell (i, j): b0 = its SELF share (the y part's plus this part's),
// bl, br its LEFT and RIGHT shares (to positions i - 1, i + 1)
inline void cells_x_vjp(const Args& a, int i, int j, P& b0, P& bl, P& br)
{
    const size_t ne = (size_t)a.ex * a.ey, e = ext_index(a, i, j);
    b0 = load_p(a.Cs, ne, SELF, e);
    bl = br = zero_p();
    face_states_vjp_x<true>(prim_at(a, i, j), prim_at(a, i - 1, j), prim_at(a, i + 1, j), a.kx,
                            load_face_adjoints(a, ne, e), b0, bl, br);
}

// index of padded position (px, j), px in [-2, nx + 1], j an extended row, in XS
inline size_t xs_index(const Args& a, int px, int j) { return (size_t)(j + 1) * (a.nx + 4) + (px + 2); }

// sum of the shares that land on padded position (pi, pj): the x-part sum of
// its row (extended rows only) and the y part's DOWN and UP shares of the
// extended cells above and below
inline P pad_sum(const Args& a, int pi, int pj)
{
    const size_t ne = (size_t)a.ex * a.ey, nxs = (size_t)(a.nx + 4) * a.ey;
    auto in_ext = [&](int i, int j) { return i >= -1 && i <= a.nx && j >= -1 && j <= a.ny; };
    P s = zero_p();
    if (pj >= -1 && pj <= a.ny) acc(s, load_p(a.XS, nxs, 0, xs_index(a, pi, pj)));
    if (in_ext(pi, pj + 1)) acc(s, load_p(a.Cs, ne, DOWN, ext_index(a, pi, pj + 1)));
    if (in_ext(pi, pj - 1)) acc(s, load_p(a.Cs, ne, UP, ext_index(a, pi, pj - 1)));
    return s;
}

inline void gather_cell(const Args& a, int i, int j)
{
    int px[5], py[5];
    const int nx_ = preimages(i, a.nx, a.bcx, px), ny_ = preimages(j, a.ny, a.bcy, py);
    P wb = zero_p();
    for (int u = 0; u < nx_; ++u)
        for (int v = 0; v < ny_; ++v) acc(wb, pad_sum(a, px[u], py[v]));
    const size_t plane = (size_t)a.nx * a.ny, c = (size_t)j * a.nx + i;
    C out = lam_prime(a, i, j);
    to_prim_vjp(load_cons<double>(a.U, plane, c), wb, out);
    store_cons(a.lam0, plane, c, out);
}

}  // namespace ref
}  // namespace csh
