// CPU harness for the adjoint: runs the bodies of the adjoint kernels and the forward
// face/flux arithmetic in host loops, so the tests can check the hand-written reverse
// pass against finite differences and the oracle's dense Jacobian without a GPU, and
// the device's 2-D blocks against the reverse step cell by cell.  Test infrastructure
// only.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <vector>

#include "adjoint_reference.h"
#include "csh_adjoint.h"

using namespace csh;

static void set_args(AdjArgs& a, int nx, int ny, int bcx, int bcy, double dx, double dy, double dt, double vc,
                     double rc, double x0, double y0, const double* U)
{
    a.nx = nx;
    a.ny = ny;
    a.bcx = bcx;
    a.bcy = bcy;
    a.dx = dx;
    a.dy = ny > 1 ? dy : 1.0;
    a.dt = dt;
    set_step_factors(a);
    a.vc2 = vc * vc;
    a.rc2 = rc * rc;
    a.x0 = x0;
    a.y0 = y0;
    a.U = U;
}

static P plus3(const P& a, const P& b, const P& c)
{
    return {a.r + b.r + c.r, a.u + b.u + c.u, a.v + b.v + c.v, a.pxx + b.pxx + c.pxx, a.pxy + b.pxy + c.pxy,
            a.pyy + b.pyy + c.pyy};
}

static const double kNan = std::numeric_limits<double>::quiet_NaN();

// the 1-D kernels, a loop per stage; the workspace has the device's size and is
// NaN-filled: every slot the reverse pass reads must have been written by it
static void adjoint_1d(AdjArgs a)
{
    std::vector<double> ws(workspace_1d(a.nx), kNan);
    set_workspace_1d(a, ws.data());
    for (int i = -1; i <= a.nx; ++i) faces_cell(a, i);
    for (int i = -1; i <= a.nx; ++i) hll_cell(a, i);
    // self, left and right shares per extended cell, then one sum per padded position
    // in the kernel's order (self, left share of the cell to the right, right share of
    // the cell to the left; zero outside the range)
    const size_t ne = (size_t)a.nx + 2;
    std::vector<P> b0(ne), bl(ne), br(ne);
    for (int i = -1; i <= a.nx; ++i) cells_x_vjp(a, i, b0[i + 1], bl[i + 1], br[i + 1]);
    auto share = [&](const std::vector<P>& v, int i) { return i >= -1 && i <= a.nx ? v[i + 1] : zero_p(); };
    for (int p = -2; p <= a.nx + 1; ++p)
        store_p(a.XS, (size_t)a.nx + 4, 0, (size_t)(p + 2), plus3(share(b0, p), share(bl, p + 1), share(br, p - 1)));
    for (int i = 0; i < a.nx; ++i) gather_cell(a, i);
}

// the 2-D reference, cell by cell
static void adjoint_2d(ref::Args& a)
{
    a.ex = a.nx + 2;
    a.ey = a.ny + 2;
    const size_t ne = (size_t)a.ex * a.ey, nxs = (size_t)(a.nx + 4) * a.ey;
    std::vector<double> ws(66 * ne + 6 * nxs, kNan);
    a.FS = ws.data();
    a.FSb = ws.data() + 24 * ne;
    a.Cs = ws.data() + 48 * ne;
    a.XS = ws.data() + 66 * ne;
    auto extended = [&](auto body) {
        for (int j = -1; j <= a.ny; ++j)
            for (int i = -1; i <= a.nx; ++i) body(i, j);
    };
    extended([&](int i, int j) { ref::faces_cell(a, i, j); });
    extended([&](int i, int j) { ref::hll_cell(a, i, j); });
    extended([&](int i, int j) { ref::cells_cell_y(a, i, j); });
    std::vector<P> b0(ne), bl(ne), br(ne);
    extended([&](int i, int j) {
        const size_t e = ref::ext_index(a, i, j);
        ref::cells_x_vjp(a, i, j, b0[e], bl[e], br[e]);
    });
    auto share = [&](const std::vector<P>& v, int i, int j) {
        return i >= -1 && i <= a.nx ? v[ref::ext_index(a, i, j)] : zero_p();
    };
    for (int j = -1; j <= a.ny; ++j)
        for (int px = -2; px <= a.nx + 1; ++px)
            store_p(a.XS, nxs, 0, ref::xs_index(a, px, j),
                    plus3(share(b0, px, j), share(bl, px + 1, j), share(br, px - 1, j)));
    for (int j = 0; j < a.ny; ++j)
        for (int i = 0; i < a.nx; ++i) ref::gather_cell(a, i, j);
}

extern "C" int host_adjoint_step(int nx, int ny, int bcx, int bcy, double dx, double dy, double dt, double vc,
                                 double rc, double x0, double y0, const double* U, const double* lam1, double* lam0)
{
    ref::Args a{};
    set_args(a, nx, ny, bcx, bcy, dx, dy, dt, vc, rc, x0, y0, U);
    a.lam1 = lam1;
    a.lam0 = lam0;
    if (ny > 1) adjoint_2d(a);
    else adjoint_1d(a);
    return 0;
}

// The values of a block's threads moved by one lane, D = +1 or -1, within each
// wavefront of 64; 0 where the shift has no source (lane_shift on the device).
template <int D, class V>
static std::vector<V> shifted(const std::vector<V>& x)
{
    std::vector<V> out(x.size(), V{0, 0, 0, 0, 0, 0});
    for (size_t t = 0; t < x.size(); ++t) {
        const int l = (int)(t % 64) + D;
        if (l >= 0 && l < 64 && t + D < x.size()) out[t] = x[t + D];
    }
    return out;
}

// The device's 2-D reverse step on the CPU: per block each phase of adjoint_fused_kernel
// for every thread, heap arrays of the exact sizes standing for LDS (a slot read before
// it is written shows as NaN, one outside under the sanitizer), the lane shifts
// wavefront by wavefront.  False if a cell is not written by exactly one block.
template <int BX>
static bool adjoint_blocks(AdjArgs a)
{
    const double unwritten = -7.25e300;
    const size_t cells = 6 * (size_t)a.nx * a.ny;
    double* const lam0 = a.lam0;
    std::vector<double> own(cells, unwritten);
    std::vector<int> writers(cells, 0);
    a.lam0 = own.data();

    using Thread = AdjointThread<BX>;
    const int tiles_x = (a.nx + Thread::OX - 1) / Thread::OX, tiles_y = (a.ny + kF_OY - 1) / kF_OY;
    const int n = BX * kF_Y;
    for (int block = 0; block < tiles_x * tiles_y; ++block) {
        std::vector<double> S(Thread::kStates, kNan), Y(Thread::kRows, kNan), M(Thread::kRows, kNan);
        std::vector<Thread> t;
        t.reserve(n);
        for (int k = 0; k < n; ++k) t.emplace_back(a, S.data(), Y.data(), M.data(), (unsigned)block, tiles_x, k);
        auto every = [&](auto phase) {
            for (int k = 0; k < n; ++k) phase(t[k], k);
        };
        auto values = [&](auto of) {
            std::vector<decltype(of(t[0]))> v;
            for (int k = 0; k < n; ++k) v.push_back(of(t[k]));
            return v;
        };
        every([](Thread& q, int) { q.load(); });
        every([](Thread& q, int) { q.faces(); });
        {
            const auto xlo = shifted<+1>(values([](const Thread& q) { return q.f.xlo; }));
            const auto lam = shifted<+1>(values([](const Thread& q) { return q.lam; }));
            std::vector<P> low(n);
            every([&](Thread& q, int k) { low[k] = q.x_face(xlo[k], lam[k]); });
            low = shifted<-1>(low);
            every([&](Thread& q, int k) { q.fb.xlo = low[k]; });
        }
        every([](Thread& q, int) { q.y_face(); });
        every([](Thread& q, int) { q.shares(); });
        {
            const auto l = shifted<+1>(values([](const Thread& q) { return q.left; }));
            const auto r = shifted<-1>(values([](const Thread& q) { return q.right; }));
            every([&](Thread& q, int k) { q.land_x(l[k], r[k]); });
        }
        every([](Thread& q, int) { q.land_y(); });
        if (t[0].folds_x()) {
            const auto self = values([](const Thread& q) { return q.self; });
            const auto l1 = shifted<-1>(self), l2 = shifted<-1>(l1), r1 = shifted<+1>(self), r2 = shifted<+1>(r1);
            every([&](Thread& q, int k) { q.fold_x(l1[k], l2[k], r1[k], r2[k]); });
        }
        if (t[0].folds_y()) {
            every([](Thread& q, int) { q.put_total(); });
            every([](Thread& q, int) { q.fold_y(); });
        }
        every([](Thread& q, int) { q.store(); });
        for (size_t c = 0; c < cells; ++c) {
            if (own[c] == unwritten) continue;
            lam0[c] = own[c];
            own[c] = unwritten;
            ++writers[c];
        }
    }
    return std::all_of(writers.begin(), writers.end(), [](int k) { return k == 1; });
}

// blocks of `width` columns (16 or 32)
extern "C" int host_adjoint_step_blocks(int width, int nx, int ny, int bcx, int bcy, double dx, double dy, double dt,
                                        double vc, double rc, double x0, double y0, const double* U,
                                        const double* lam1, double* lam0)
{
    if (ny < 2) return -1;
    AdjArgs a{};
    set_args(a, nx, ny, bcx, bcy, dx, dy, dt, vc, rc, x0, y0, U);
    a.lam1 = lam1;
    a.lam0 = lam0;
    if (width == 16) return adjoint_blocks<16>(a) ? 0 : 2;
    return width == 32 ? (adjoint_blocks<32>(a) ? 0 : 2) : -1;
}

// both widths, which agree to rounding; the narrow one's result
extern "C" int host_adjoint_step_tiled(int nx, int ny, int bcx, int bcy, double dx, double dy, double dt, double vc,
                                       double rc, double x0, double y0, const double* U, const double* lam1,
                                       double* lam0)
{
    std::vector<double> wide(6 * (size_t)nx * ny, kNan);
    const int e = host_adjoint_step_blocks(32, nx, ny, bcx, bcy, dx, dy, dt, vc, rc, x0, y0, U, lam1, wide.data()) |
                  host_adjoint_step_blocks(16, nx, ny, bcx, bcy, dx, dy, dt, vc, rc, x0, y0, U, lam1, lam0);
    if (e) return e;
    double most = 0.0;
    for (size_t k = 0; k < wide.size(); ++k) most = std::max(most, std::fabs(lam0[k]));
    for (size_t k = 0; k < wide.size(); ++k)
        if (!(std::fabs(wide[k] - lam0[k]) <= 1e-12 * most)) return 1;
    return 0;
}

// the forward step with the same face-state, HLL, update and kick arithmetic, from the
// face states of the extended cells: [4 faces][6][ex * ey] in both dimensions
extern "C" int host_step(int nx, int ny, int bcx, int bcy, double dx, double dy, double dt, double vc, double rc,
                         double x0, double y0, const double* U, double* Un)
{
    const bool twod = ny > 1;
    ref::Args a{};
    set_args(a, nx, ny, bcx, bcy, dx, dy, dt, vc, rc, x0, y0, U);
    a.ex = nx + 2;
    a.ey = twod ? ny + 2 : 1;
    const size_t ne = (size_t)a.ex * a.ey, plane = (size_t)nx * ny;
    std::vector<double> fs(24 * ne, 0.0);
    a.FS = a.AdjArgs::FS = fs.data();
    if (twod) {
        for (int j = -1; j <= ny; ++j)
            for (int i = -1; i <= nx; ++i) ref::faces_cell(a, i, j);
    } else {
        for (int i = -1; i <= nx; ++i) faces_cell(a, i);
    }
    for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i) {
            const size_t e = twod ? ref::ext_index(a, i, j) : (size_t)(i + 1);
            auto face = [&](int hi, int lo, size_t below, size_t above) {
                return hll_x(make_face_x(hi == ref::XHI ? load_p(a.FS, ne, hi, below) : swap(load_p(a.FS, ne, hi, below))),
                             make_face_x(lo == ref::XLO ? load_p(a.FS, ne, lo, above) : swap(load_p(a.FS, ne, lo, above))));
            };
            C u = update(load_cons<double>(U, plane, (size_t)j * nx + i), a.cx, face(ref::XHI, ref::XLO, e, e + 1),
                         face(ref::XHI, ref::XLO, e - 1, e));
            if (twod)
                u = update(u, a.cy, swap(face(ref::YHI, ref::YLO, e, e + a.ex)),
                           swap(face(ref::YHI, ref::YLO, e - a.ex, e)));
            if (a.vc2 != 0.0) {
                const double x = a.x0 + (i + 0.5) * a.dx, y = twod ? a.y0 + (j + 0.5) * a.dy : 0.0;
                const double f = -a.vc2 / (x * x + y * y + a.rc2), ax = f * x, ay = f * y, h = a.dt;
                const double mx = u.mx, my = u.my;
                u.mx = mx + h * u.r * ax;
                u.my = my + h * u.r * ay;
                u.exx = u.exx + h * ax * (2.0 * mx + h * u.r * ax);
                u.exy = u.exy + h * (ax * my + mx * ay + h * u.r * ax * ay);
                u.eyy = u.eyy + h * ay * (2.0 * my + h * u.r * ay);
            }
            store_cons(Un, plane, (size_t)j * nx + i, u);
        }
    return 0;
}

// W -> U and its transpose, per cell
extern "C" void host_init_adjoint(int64_t n, const double* W, const double* lamU, double* lamW)
{
    for (int64_t c = 0; c < n; ++c) {
        const P w = {W[c], W[n + c], W[2 * n + c], W[3 * n + c], W[4 * n + c], W[5 * n + c]};
        P wb = zero_p();
        to_cons_vjp(w, load_cons<double>(lamU, (size_t)n, (size_t)c), wb);
        const double v[6] = {wb.r, wb.u, wb.v, wb.pxx, wb.pxy, wb.pyy};
        for (int m = 0; m < 6; ++m) lamW[m * n + c] = v[m];
    }
}

// the adjoint kernels' workgroup renumbering, for the bijection test
extern "C" unsigned host_xcd_block(unsigned b, unsigned nb)
{
    return csh::xcd_block(b, nb);
}
